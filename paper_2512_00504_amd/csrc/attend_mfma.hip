// Decode attention on the matrix cores: bf16 or fp32, head_dim 64 or 128, group size g <= 16.
//
// One workgroup of NW wavefronts per (unit, split).  A wavefront owns slices of 16 (or 32) keys
// of the cache (slice it, it + splits*NW, ...) and keeps flash-decoding state (running max,
// running sum, fp32 accumulators) for all g query heads of the KV group, so K and V are read
// from HBM exactly once per KV head.
//
// Per slice and wavefront (16-key tiles; r = lane % 16, kb = lane / 16):
//   K: in the tiled K format each load of a tile's A operands (lane = key r, 16-byte chunk
//      4c + kb of its row) is one contiguous 1 KiB; the few tiles appended since the last
//      compaction are row-major and load as 16 rows x 64 bytes.
//      S^T[key, head] = K[key, :] . Q[head, :]:
//        bf16: a chunk is 8 channels, one MFMA 16x16x32 per load;
//        fp32: a chunk is 4 channels, four MFMAs 16x16x4 per load, the j-th on the j-th channel of
//        every chunk (any order of the channels serves, as long as K and Q use the same).
//      The result lane (head r, block kb) holds keys 4 kb + e, e = 0..3, of its head per tile.
//   softmax: running max shared by the 4 lanes of a head (2 cross-lane exchanges), exp2.
//   V: lane (r, kb) loads D/16 channels of keys 4 kb + e, so a quarter-wave reads one full row.
//      O^T[channel, head] += V^T[channel, key] . P^T[key, head], with P already in the right lanes:
//        bf16: an in-register transpose (v_perm_b32) makes the A operands, D/16 MFMAs per slice;
//        fp32: the loaded words are the A operands, MFMA 16x16x4 per (e, channel of the lane).
//      bf16 rounds P to bf16 at D = 128; at D = 64 it enters as the sum of three bf16 numbers, which
//      hold its 24 bits; fp32 keeps it as it is.
// Bound: HBM at launches of a few hundred units and more, latency below.  fp32 has 8 KiB (D = 64)
// or 16 KiB (D = 128) per slice against 1024 or 2048 cycles of MFMA, so four wavefronts can take
// 32 B a cycle and CU, four times the CU's share of the HBM rate; bf16 needs a tenth of that.
// Against the plain vector-ALU kernel these shapes used before, per launch: fp32 D = 128, 32 units
// of 528 rows 466 -> 9.6 us (uncut 17.6), 896 units 1614 -> 75.5; bf16 D = 64, 128 units of 528 rows 245 -> 6.9,
// 1152 units 575 -> 28.4; fp32 D = 64, 2 units of 72 rows 25.5 -> 4.5.
// The wavefronts of a workgroup are merged through LDS; splits of one unit are merged by the
// last workgroup to finish (ticket counter), in a fixed order, so results are deterministic.
//
// The newest token's k/v are not read from the cache (another workgroup may be writing that
// row): the lanes that would hold row `len` take them from k_new / v_new instead.
// All stores (output, the appended K/V rows, the window-ring slot) are issued at the end of
// the workgroup and are whole contiguous rows: stores mixed into the read stream, partial-line
// stores and atomics each cost several microseconds per launch on this memory system.
#include "gkv_internal.h"

#include <type_traits>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld16(const void* p) { return *(const u32x4*)p; }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Row geometry of one (element type, head_dim).
template <typename T, int D>
struct Geo {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int ROW_BYTES = D * (int)sizeof(T);
  static constexpr int TILE_BYTES = 16 * ROW_BYTES;
  static constexpr int NL = ROW_BYTES / 64;      // K loads (16 bytes a lane) per tile
  static constexpr int RP = ROW_BYTES / 16;      // 16-byte pieces per row
  static constexpr int NC = D / 16;              // channels per lane, accumulators per lane
  static constexpr int VW = ROW_BYTES / 64;      // 32-bit words of V per lane and key
  static constexpr int OSTR = D + 4;             // padded LDS row of the per-wave partial outputs
  static constexpr int PSTR = D + 2;             // split partial: o[D], m, l
};

// V words of one key for lane r: channels [r*NC, +NC), except fp32 at D = 128, whose lanes take 4
// channels from each half of the row so that both 16-byte loads are contiguous over the lanes.
template <int VW> struct VWords { uint32_t w[VW]; };
template <typename T, int D>
__device__ __forceinline__ void ld_v(VWords<Geo<T, D>::VW>& o, const char* row, int r) {
  if constexpr (Geo<T, D>::VW == 2) {
    const u32x2 a = __builtin_nontemporal_load((const u32x2*)(row + r * 8));
    o.w[0] = a[0]; o.w[1] = a[1];
  } else {
    const u32x4 a = __builtin_nontemporal_load((const u32x4*)(row + r * 16));
#pragma unroll
    for (int i = 0; i < 4; ++i) o.w[i] = a[i];
    if constexpr (Geo<T, D>::VW == 8) {
      const u32x4 b = __builtin_nontemporal_load((const u32x4*)(row + 256 + r * 16));
#pragma unroll
      for (int i = 0; i < 4; ++i) o.w[4 + i] = b[i];
    }
  }
}
template <typename T, int D>
__device__ __forceinline__ void ld_v_lds(VWords<Geo<T, D>::VW>& o, const char* row, int r) {
#pragma unroll
  for (int i = 0; i < Geo<T, D>::VW; ++i)
    o.w[i] = *(const uint32_t*)(row + (Geo<T, D>::VW == 8 ? (i >> 2) * 256 + r * 16 + (i & 3) * 4
                                                           : r * Geo<T, D>::VW * 4 + i * 4));
}

// One wavefront iteration's loads: KT K tiles (A operands) and 4*KT V rows per lane.
template <typename T, int D, int KT>
struct Slice {
  u32x4 kA[KT][Geo<T, D>::NL];
  VWords<Geo<T, D>::VW> vR[4 * KT];
};

// Tiles below n_tiled are in tiled format (lane-contiguous 1 KiB per load); tiles above are
// row-major, where the same operand is 16 rows x 64 bytes per load (only the rows appended since
// the last compaction are in that state).
// K is read with ordinary loads, V with non-temporal loads.  Measured on MI355X with this access
// pattern (bf16, D = 128): both ordinary 67-77% of the HBM peak (worst when K+V exceed the 256 MiB
// memory-side cache), both non-temporal 76%, one stream of each kind 80-85% at every cache size
// tried (0.3 to 10 GB), whichever of the two is the non-temporal one.
template <typename T, int D, int KT>
__device__ __forceinline__ void issue_slice(Slice<T, D, KT>& s, const char* Kh, const char* Vh, int it,
                                            int n_tiled, int lane, int r, int kb) {
  using G = Geo<T, D>;
  const int key0 = it * 16 * KT;
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) {
    const int row0 = key0 + 16 * tt;
    const char* Kt = Kh + (size_t)(row0 >> 4) * G::TILE_BYTES;
    const bool tiled = row0 < n_tiled;                     // wave-uniform
    const int lane_off = tiled ? lane * 16 : r * G::ROW_BYTES + kb * 16;
    const int step_off = tiled ? 1024 : 64;
#pragma unroll
    for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = ld16(Kt + lane_off + c * step_off);
  }
#pragma unroll
  for (int jj = 0; jj < 4 * KT; ++jj) {
    const int key = key0 + (jj & 3) + 4 * kb + (jj >> 2) * 16;
    ld_v<T, D>(s.vR[jj], Vh + (size_t)key * G::ROW_BYTES, r);
  }
}

// Flash-decoding state of one wavefront: lane (head = lane%16, blk = lane/16) holds the running
// max (in log2 units, shared by the 4 lanes of a head), its partial running sum, and in
// oacc[m][e] O[head][channel m of lane 4 blk + e].
template <int NC>
struct Running {
  float m_run, l_run;
  f32x4 oacc[NC];
};

// EDGE = the slice may contain the newest token's row and rows past the end: substitute k/v of
// the newest token from the inputs, mask the rest.  The common path has none of that.
// EXACT: right for every logit and value, infinities and finite ones of any size among them.  Without
// it, which is what a wavefront tries first, a logit of -inf may give NaN (the scale's low part times -inf), a
// huge maximum any weight (see log2_weight), and at bf16, D = 64 an infinite value NaN; all of them show at the end.
template <typename T, int D, int KT, bool EDGE, bool EXACT>
__device__ __forceinline__ void process_slice(Slice<T, D, KT>& s, Running<D / 16>& st,
                                              const u32x4 (&qB)[Geo<T, D>::NL], int it,
                                              float scale_log2, float scale_log2_lo, int r, int kb, bool has_new, int len0,
                                              int n_tot, const char* knew, const char* vnew) {
  // knew / vnew: the newest token's k and v rows, staged in LDS at the start of the workgroup
  using G = Geo<T, D>;
  constexpr int NS = 4 * KT;
  const int key0 = it * 16 * KT;
  if constexpr (EDGE) {
    if (has_new && key0 <= len0) {
      const int tt_new = (len0 - key0) >> 4, rr = len0 & 15;
#pragma unroll
      for (int tt = 0; tt < KT; ++tt)
        if (tt == tt_new && r == rr) {
#pragma unroll
          for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = *(const u32x4*)(knew + (4 * c + kb) * 16);
        }
#pragma unroll
      for (int jj = 0; jj < NS; ++jj) {
        const int key = key0 + (jj & 3) + 4 * kb + (jj >> 2) * 16;
        if (key == len0) ld_v_lds<T, D>(s.vR[jj], vnew, r);
      }
    }
#pragma unroll
    for (int jj = 0; jj < NS; ++jj) {
      const int key = key0 + (jj & 3) + 4 * kb + (jj >> 2) * 16;
      if (key >= n_tot) {                                  // stale rows must not reach the MFMA
#pragma unroll
        for (int i = 0; i < G::VW; ++i) s.vR[jj].w[i] = 0u;
      }
    }
  }

  // scores: sc[tt][e] = q[head r] . k[key0 + 16 tt + 4 kb + e]
  f32x4 sc[KT];
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) {
    sc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < G::NL; ++c) {
      if constexpr (G::F32) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          sc[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(s.kA[tt][c][i]), __uint_as_float(qB[c][i]),
                                                        sc[tt], 0, 0, 0);
      } else {
        sc[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(s.kA[tt][c]), as_bf16x8(qB[c]), sc[tt], 0, 0, 0);
      }
    }
  }
  float sv[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    sv[i] = sc[i >> 2][i & 3];
    if constexpr (EDGE) {
      const int key = key0 + (i >> 2) * 16 + 4 * kb + (i & 3);
      if (key >= n_tot) sv[i] = EXACT ? -INFINITY : -1e30f;
    }
  }
  float mx = sv[0];
#pragma unroll
  for (int i = 1; i < NS; ++i) mx = fmaxf(mx, sv[i]);
  mx = fmaxf(mx, __shfl_xor(mx, 16));
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  const float m_new = fmaxf(st.m_run, mx * scale_log2);       // scale > 0: max commutes with it
  if (__any(m_new > st.m_run)) {
    const float corr = __builtin_amdgcn_exp2f(st.m_run - m_new);
    st.l_run *= corr;
#pragma unroll
    for (int m = 0; m < G::NC; ++m) st.oacc[m] *= corr;
    st.m_run = m_new;
  }
  float pf[NS];
  float psum = 0.f;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    // exponent of 2 = z * (hi + lo) - m: the window-score kernel forms its own from the same
    // logits, so the sums recorded below are the normalisers of its probabilities
    float y;
    if constexpr (EXACT) y = log2_weight(sv[i], scale_log2, scale_log2_lo, st.m_run);
    else y = fmaf(sv[i], scale_log2_lo, fmaf(sv[i], scale_log2, -st.m_run));
    pf[i] = __builtin_amdgcn_exp2f(y);
    psum += pf[i];
  }
  st.l_run += psum;

  // O^T[channel, head] += V^T . P^T
  if constexpr (G::F32) {
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int m = 0; m < G::NC; ++m)
        st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(s.vR[i].w[m]), pf[i], st.oacc[m], 0, 0, 0);
  } else if constexpr (EXACT && D == 64) {       // P whole, V converted word by word
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
      for (int m = 0; m < G::NC; ++m) {
        const uint32_t w = s.vR[i].w[m >> 1];
        st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float((m & 1) ? w & 0xffff0000u : w << 16), pf[i],
                                                          st.oacc[m], 0, 0, 0);
      }
  } else if constexpr (KT == 2) {
    f32x8 p8;
#pragma unroll
    for (int i = 0; i < 8; ++i) p8[i] = pf[i];
    const bf16x8 pB = __builtin_convertvector(p8, bf16x8);
    bf16x8 pM, pL;                               // D = 64: P = pB + pM + pL, all of its 24 bits
    if constexpr (D == 64) {
      const f32x8 r1 = p8 - __builtin_convertvector(pB, f32x8);
      pM = __builtin_convertvector(r1, bf16x8);
      pL = __builtin_convertvector(r1 - __builtin_convertvector(pM, f32x8), bf16x8);
    }
    u32x4 t[G::NC];
#pragma unroll
    for (int m = 0; m < G::NC; ++m) {
#pragma unroll
      for (int y = 0; y < 4; ++y)
        t[m][y] = __builtin_amdgcn_perm(s.vR[2 * y + 1].w[m >> 1], s.vR[2 * y].w[m >> 1],
                                        (m & 1) ? 0x07060302u : 0x05040100u);
      st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t[m]), pB, st.oacc[m], 0, 0, 0);
    }
    if constexpr (D == 64) {                     // term by term: an accumulator's products don't wait for each other
#pragma unroll
      for (int m = 0; m < G::NC; ++m) st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t[m]), pM, st.oacc[m], 0, 0, 0);
#pragma unroll
      for (int m = 0; m < G::NC; ++m) st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t[m]), pL, st.oacc[m], 0, 0, 0);
    }
  } else {
    f32x4 p4;
#pragma unroll
    for (int i = 0; i < 4; ++i) p4[i] = pf[i];
    const bf16x4 pB4 = __builtin_convertvector(p4, bf16x4);
    const s16x4 pB = __builtin_bit_cast(s16x4, pB4);
#pragma unroll
    for (int m = 0; m < G::NC; ++m) {
      u32x2 t;
#pragma unroll
      for (int y = 0; y < 2; ++y)
        t[y] = __builtin_amdgcn_perm(s.vR[2 * y + 1].w[m >> 1], s.vR[2 * y].w[m >> 1],
                                     (m & 1) ? 0x07060302u : 0x05040100u);
      st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, t), pB, st.oacc[m], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void store_row4(float* p, const f32x4& o) { *(f32x4*)p = o; }
__device__ __forceinline__ void store_row4(uint16_t* p, const f32x4& o) {
  uint2 packed;
  packed.x = (uint32_t)float_to_bf16_bits(o[0]) | ((uint32_t)float_to_bf16_bits(o[1]) << 16);
  packed.y = (uint32_t)float_to_bf16_bits(o[2]) | ((uint32_t)float_to_bf16_bits(o[3]) << 16);
  *(uint2*)p = packed;
}
// Two neighbouring floats to and from memory that workgroups on other XCDs share.
__device__ __forceinline__ void store_agent(float* p, float x, float y) {
  const uint64_t v = ((uint64_t)__float_as_uint(y) << 32) | __float_as_uint(x);
  __hip_atomic_store((uint64_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_agent(const float* p) {
  const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}
// 1/l in full precision; `fast`: v_rcp_f32, for uncut bf16 units at D = 128, whose P is rounded to 8
// bits as it is.  Nothing attended to: 0; keys whose logits are all -inf: NaN, as softmax gives.
__device__ __forceinline__ float inv_sum(float l, bool any_key, bool fast) {
  if (!(l > 0.f)) return any_key && l == 0.f ? __builtin_nanf("") : 0.f;
  return fast ? __builtin_amdgcn_rcpf(l) : 1.f / l;
}

// KT = 16-key tiles per wavefront iteration (1 or 2)
template <typename T, int D, int NW, int KT, int OCC>
__global__ __launch_bounds__(NW * 64, OCC) void attend_mfma_kernel(GkvDims dm, AttendArgs a) {
  using G = Geo<T, D>;
  constexpr int KEYS = 16 * KT;             // keys per iteration
  constexpr int RP = G::RP, ROW_BYTES = G::ROW_BYTES, OSTR = G::OSTR, PSTR = G::PSTR;
  extern __shared__ __attribute__((aligned(16))) float smem[];   // behind s_last: 16-byte pieces want the alignment
  __shared__ int s_last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, kb = lane >> 4;
  const int splits = a.splits;
  const int unit = quotient(blockIdx.x, a.by_splits), sp = (int)blockIdx.x - unit * splits;
  const int lb = quotient(unit, dm.by_hkv), j = unit - lb * dm.Hkv;
  const int g = dm.g, cap = dm.cap;
  const char* Kh = (const char*)a.K + (size_t)unit * cap * ROW_BYTES;
  const char* Vh = (const char*)a.V + (size_t)unit * cap * ROW_BYTES;
  const char* knew_g = (const char*)a.k_new + (size_t)unit * ROW_BYTES;
  const char* vnew_g = (const char*)a.v_new + (size_t)unit * ROW_BYTES;
  const char* q_g = (const char*)a.q + ((size_t)lb * dm.Hq + j * g) * ROW_BYTES;
  const bool appender = sp == 0;
  const bool ring_copy = appender && a.copy_q;   // q may already live in its ring slot
  const bool may_grow = a.k_new != nullptr;

  // A launch of few units is one trip to memory after the other, so everything whose address the arguments
  // give is requested before anything is waited for: the state record and the step counter (scalar loads; no
  // branch on whether there is a counter), the group's queries (B operand of the QK product: lane (head r, kb)
  // holds chunks 4c+kb of q[r]) and the rows stored at the end of the workgroup.
  int4 rec = *(const int4*)(a.d_state + 4 * (size_t)lb);
  const int32_t base = *(dm.step_base ? dm.step_base : a.d_state);
  __builtin_amdgcn_sched_barrier(0);
  u32x4 qB[G::NL];
  {
    const char* qh = q_g + min(r, g - 1) * ROW_BYTES;      // (lanes beyond the group repeat its last head and are ignored)
#pragma unroll
    for (int c = 0; c < G::NL; ++c) qB[c] = ld16(qh + (4 * c + kb) * 16);
  }
  // one 16-byte piece per thread and round: pieces [0,RP) k_new, [RP,2RP) v_new (every workgroup: the wavefront
  // that owns the last slice substitutes them for cache row `len`), [2RP, 2RP + RP g) the group's q rows for
  // the window ring (split 0 only); others read a valid address and are not used
  constexpr int AP_ROUNDS = (2 * RP + RP * 16 + NW * 64 - 1) / (NW * 64);
  u32x4 ap[AP_ROUNDS];
#pragma unroll
  for (int rd = 0; rd < AP_ROUNDS; ++rd) {
    const int x = tid + rd * NW * 64;
    const char* src = q_g + (x < 2 * RP + RP * g && x >= 2 * RP ? x - 2 * RP : 0) * 16;
    if (may_grow && x < 2 * RP) src = (x < RP ? knew_g : vnew_g - ROW_BYTES) + x * 16;
    ap[rd] = ld16(src);
  }
  const int it0 = sp * NW + wave;
  Slice<T, D, KT> s;
  __builtin_amdgcn_sched_barrier(0);           // loads come back in order: these before the slice's
  asm volatile("" : "+s"(rec.x), "+s"(rec.y), "+s"(rec.w));   // one load, not one for each of them
  const SeqState seq = state_record(rec);
  if (dm.step_base) a.step += base;

  // The length comes from the state record and the step number; nothing is written back, so
  // the workgroups of a (layer, sequence) need no ordering among themselves.
  const int len0 = length_before_step(seq, a.step, cap);
  const bool has_new = may_grow && (len0 < cap);
  const int n_tot = len0 + (has_new ? 1 : 0);
  const int n_iter = (n_tot + KEYS - 1) / KEYS;
  // Splits this unit is really cut into: as many as its own length fills with `split_iters` slices
  // each (an explicit split count sets split_iters = 0: always all of them).
  int ns = splits;
  if (splits > 1 && a.split_iters > 0) {
    ns = max(1, min(splits, (n_iter + a.split_iters - 1) / a.split_iters));
    if (sp >= ns) return;
  }
  const float scale_log2 = dm.scale_l2_hi, scale_log2_lo = dm.scale_l2_lo;

  Running<G::NC> st;
  st.m_run = GKV_NO_MAX;
  st.l_run = 0.f;
#pragma unroll
  for (int m = 0; m < G::NC; ++m) st.oacc[m] = f32x4{0.f, 0.f, 0.f, 0.f};

  // First slice in flight, then stage k_new / v_new in LDS for whoever owns the last slice.  Every wavefront asks for
  // one, those beyond the unit's end for its last (or, in an empty unit, for rows that are there, and not used): after a
  // request under a condition the compiler cannot know how many loads are younger than the rows to stage, waits for
  // all of them, and the barrier holds every wavefront until the first slices of all have arrived.  us per launch in a
  // graph, with the condition -> without: 128 units x 577 rows 11.3 -> 10.65, 256 x 1056 23.5 -> 22.6, 4 x 577 7.3 -> 6.8; d = 64 128 x
  // 528 7.9 -> 7.2, 512 14.8 -> 14.55; fp32 32 x 528 11.4 -> 10.0, ragged 84 to 464 12.7 -> 11.7; 896 x 576 48.8 both ways.
  // (The first slice, or the first two, requested ahead of the record on a guess of K's format cost more than that wait:
  // 4 x 577 7.2, 32 x 577 8.4 against 7.9, ragged 84 to 464 9.9 / 8.4, 128 x 2112 25.3 / 24.8.)
  const int stride = ns * NW;
  issue_slice<T, D, KT>(s, Kh, Vh, min(it0, max(n_iter - 1, 0)), seq.n_tiled, lane, r, kb);
  // stage: 16-byte pieces [0,RP) k_new, [RP,2RP) v_new, [2RP, 2RP+RP*g) q rows; kept in LDS, not
  // in registers, until they are stored at the end
  char* stage = (char*)(smem + NW * g * OSTR + NW * 16 + NW * 16);
  const char* knew = stage;
  const char* vnew = stage + ROW_BYTES;
#pragma unroll
  for (int rd = 0; rd < AP_ROUNDS; ++rd) {
    const int x = tid + rd * NW * 64;
    if (x < 2 * RP + RP * g) *(u32x4*)(stage + x * 16) = ap[rd];
  }
  __syncthreads();
  // this wavefront's slices, the first one already requested
  auto slices = [&](auto exact) {
    constexpr bool EXACT = decltype(exact)::value;
    int it = it0;
    while (it < n_iter) {
      if ((it + 1) * KEYS > len0) process_slice<T, D, KT, true, EXACT>(s, st, qB, it, scale_log2, scale_log2_lo, r, kb, has_new, len0, n_tot, knew, vnew);
      else process_slice<T, D, KT, false, EXACT>(s, st, qB, it, scale_log2, scale_log2_lo, r, kb, has_new, len0, n_tot, knew, vnew);
      it += stride;
      if (it < n_iter) issue_slice<T, D, KT>(s, Kh, Vh, it, seq.n_tiled, lane, r, kb);
    }
  };
  slices(std::false_type{});
  if (it0 < n_iter) {
    // Seldom: a maximum that the short form of the weights is not right for, or a NaN that may be its
    // doing (a logit of -inf; at bf16, D = 64 an infinite value that met a part of P that is zero or
    // negative).  The slices are gone through again.
    bool again = fabsf(st.m_run) >= GKV_HUGE_LOG2 || st.l_run != st.l_run;
    if constexpr (!G::F32 && D == 64) {
#pragma unroll
      for (int m = 0; m < G::NC; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) again |= st.oacc[m][e] != st.oacc[m][e];
    }
    if (__any(again)) {
      st.m_run = GKV_NO_MAX;
      st.l_run = 0.f;
#pragma unroll
      for (int m = 0; m < G::NC; ++m) st.oacc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
      issue_slice<T, D, KT>(s, Kh, Vh, it0, seq.n_tiled, lane, r, kb);
      slices(std::true_type{});
    }
  }
  const float m_run = st.m_run, l_run = st.l_run;
  f32x4 (&oacc)[G::NC] = st.oacc;

  // ---- merge the wavefronts of this workgroup -------------------------------------------------
  float* so = smem;                         // [NW][g][OSTR]
  float* sm = so + NW * g * OSTR;           // [NW][16]
  float* sl = sm + NW * 16;                 // [NW][16]
  float l_tot = l_run;                      // the 4 lanes of a head hold partial sums
  l_tot += __shfl_xor(l_tot, 16);
  l_tot += __shfl_xor(l_tot, 32);
  if (r < g) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // accumulators m = 4q .. 4q+3 are four neighbouring channels
#pragma unroll
      for (int q4 = 0; q4 < G::NC / 4; ++q4) {
        const int ch = (G::F32 && D == 128) ? 64 * q4 + 4 * (4 * kb + e) : G::NC * (4 * kb + e) + 4 * q4;
        *(f32x4*)(so + (wave * g + r) * OSTR + ch) =
            f32x4{oacc[4 * q4][e], oacc[4 * q4 + 1][e], oacc[4 * q4 + 2][e], oacc[4 * q4 + 3][e]};
      }
    }
    if (kb == 0) { sm[wave * 16 + r] = m_run; sl[wave * 16 + r] = l_tot; }
  }
  __syncthreads();

  // one thread per (head, 4 channels): a single round for g <= 8 with 256 threads
  T* out = (T*)a.out + ((size_t)lb * dm.Hq + j * g) * D;
  float* part = a.ws.partials + (size_t)(unit * splits + sp) * g * PSTR;
  float2* stats = a.ws.stats + ((size_t)(a.step % dm.w) * dm.L * dm.B + lb) * dm.Hq + j * g;
  for (int x = tid; x < g * (D / 4); x += NW * 64) {
    const int h = x / (D / 4), c4 = (x % (D / 4)) * 4;
    float mw[NW];
    float M = GKV_NO_MAX;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) { mw[wv] = sm[wv * 16 + h]; M = fmaxf(M, mw[wv]); }
    float Lsum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float f = __builtin_amdgcn_exp2f(mw[wv] - M);
      Lsum += sl[wv * 16 + h] * f;
      o += *(const f32x4*)(so + (wv * g + h) * OSTR + c4) * f;
    }
    if (ns == 1) {
      store_row4(out + h * D + c4, o * inv_sum(Lsum, n_tot > 0, !G::F32 && D == 128));
      // softmax statistics of this head's row (running max in log2 units, sum), into the ring slot
      // that also receives q: the window score of the next compression reuses them
      if (c4 == 0 && a.write_stats) stats[h] = make_float2(M, Lsum);
    } else {
      float* ph = part + h * PSTR;
      store_agent(ph + c4, o[0], o[1]);
      store_agent(ph + c4 + 2, o[2], o[3]);
      if (c4 == 0) store_agent(ph + D, M, Lsum);
    }
  }

  // ---- append the new row (row-major, one contiguous row each for K and V), push q into the
  //      window ring (contiguous per KV group).  Rows the other workgroups may still be reading
  //      are never the new row's source: they take k_new / v_new from the inputs. ---------------
  if (appender) {
    const int slot = a.step % dm.w;
#pragma unroll
    for (int rd = 0; rd < AP_ROUNDS; ++rd) {
      const int x = tid + rd * NW * 64;
      if (x >= 2 * RP + RP * g) continue;
      const u32x4 piece = *(const u32x4*)(stage + x * 16);
      if (x < RP) {
        if (has_new) *(u32x4*)((char*)a.K + ((size_t)unit * cap + len0) * ROW_BYTES + x * 16) = piece;
      } else if (x < 2 * RP) {
        if (has_new) *(u32x4*)((char*)a.V + ((size_t)unit * cap + len0) * ROW_BYTES + (x - RP) * 16) = piece;
      } else if (ring_copy) {
        *(u32x4*)((char*)a.qwin + ((((size_t)slot * dm.L * dm.B + lb) * dm.Hq + j * g) * ROW_BYTES) + (x - 2 * RP) * 16) = piece;
      }
    }
    if (has_new && tid == NW * 64 - 1) a.pos[(size_t)unit * cap + len0] = a.step;
  }

  // ---- merge the splits of this unit: last workgroup to finish does it ------------------------
  // The partials go through memory with agent-scope accesses (they pass the XCDs' separate L2s
  // by), each thread waits for its own stores, and the ticket follows the barrier: no fence, which
  // would write back the whole L2 of the XCD (4 units of 577 rows in 3 splits: 13.4 us with
  // __threadfence, against 8.9 unsplit).
  if (ns > 1) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      const int old = __hip_atomic_fetch_add(&a.ws.split_ticket[unit], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = old == ns - 1;
      if (old == ns - 1) __hip_atomic_store(&a.ws.split_ticket[unit], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (s_last) {
      const float* pu = a.ws.partials + (size_t)unit * splits * g * PSTR;
      for (int x = tid; x < g * (D / 4); x += NW * 64) {
        const int h = x / (D / 4), c4 = (x % (D / 4)) * 4;
        float M = GKV_NO_MAX, Lsum = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int s2 = 0; s2 < ns; ++s2) {
          const float* ph = pu + (s2 * g + h) * PSTR;
          const float2 ml = load_agent(ph + D), a0 = load_agent(ph + c4), a1 = load_agent(ph + c4 + 2);
          const float Mn = fmaxf(M, ml.x);
          const float f0 = __builtin_amdgcn_exp2f(M - Mn), f = __builtin_amdgcn_exp2f(ml.x - Mn);
          M = Mn;
          Lsum = Lsum * f0 + ml.y * f;
          o = o * f0 + f32x4{a0.x, a0.y, a1.x, a1.y} * f;
        }
        store_row4(out + h * D + c4, o * inv_sum(Lsum, n_tot > 0, false));
        if (c4 == 0 && a.write_stats) stats[h] = make_float2(M, Lsum);
      }
    }
  }
}

}  // namespace

size_t gkv_attend_mfma_lds(int esz, int d, int g, int waves) {
  return sizeof(float) * ((size_t)waves * g * (d + 4) + 2 * 16 * (size_t)waves) + (size_t)(2 + g) * d * esz;
}

template <typename T, int D, int NW, int KT, int OCC>
static hipError_t launch_attend(const GkvLaunch& ln, const GkvDims& dm, AttendArgs a) {
  const int units = dm.L * dm.B * dm.Hkv;
  a.by_splits = gkv_divisor(a.splits);
  const size_t shmem = gkv_attend_mfma_lds(sizeof(T), D, dm.g, NW);
  return gkv_launch(ln, attend_mfma_kernel<T, D, NW, KT, OCC>, dim3(units * a.splits), dim3(NW * 64), shmem, dm, a);
}

hipError_t gkv_launch_attend_mfma(const GkvLaunch& ln, const GkvDims& dm, int dtype, const AttendArgs& a) {
  if (dtype == GKV_F32) {
    if (dm.d == 64) {
      if (a.waves == 16) return launch_attend<float, 64, 16, 1, 4>(ln, dm, a);
      if (a.waves == 8) return launch_attend<float, 64, 8, 1, 4>(ln, dm, a);
      return launch_attend<float, 64, 4, 1, 4>(ln, dm, a);
    }
    if (a.waves >= 8) return launch_attend<float, 128, 8, 1, 2>(ln, dm, a);
    return launch_attend<float, 128, 4, 1, 2>(ln, dm, a);
  }
  if (dm.d == 64) {
    if (a.waves == 16) return launch_attend<uint16_t, 64, 16, 2, 4>(ln, dm, a);
    if (a.waves == 8) return launch_attend<uint16_t, 64, 8, 2, 4>(ln, dm, a);
    return launch_attend<uint16_t, 64, 4, 2, 4>(ln, dm, a);
  }
  if (a.waves == 16) return launch_attend<uint16_t, 128, 16, 1, 2>(ln, dm, a);
  if (a.waves == 8) return launch_attend<uint16_t, 128, 8, 1, 4>(ln, dm, a);
  if (a.tile_keys == 32) return launch_attend<uint16_t, 128, 4, 2, 2>(ln, dm, a);
  return launch_attend<uint16_t, 128, 4, 1, 4>(ln, dm, a);
}
