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
//      bf16 rounds P to bf16 at D = 128, in launches of up to 256 workgroups of 4 wavefronts it enters as the sum of two
//      bf16 numbers (see WHOLE); at D = 64 as the sum of three, which hold its 24 bits; fp32 keeps it as it is.
// Bound: HBM at launches of a few hundred units and more.  fp32 has 8 KiB (D = 64) or 16 KiB (D = 128) per slice
// against 1024 or 2048 cycles of MFMA, so four wavefronts can take 32 B a cycle and CU, four times the CU's share of
// the HBM rate; bf16 needs a tenth of that.  Below that the number of instructions: a wavefront alone on its SIMD issues one every
// five cycles or so, and a launch of few units is a chain of about a thousand of them (by clock stamps, 4 units of 577 rows: 11 000
// cycles from the first argument to the last store, of which trips to memory are a third).  So addresses are a scalar base,
// a lane's constant offset and an immediate (a slice 110 instructions where 64-bit lane addresses made it 215), what goes from
// lane to lane goes through registers, a slice that needs no rescaling or masking branches around it, results are
// rounded to bf16 by the conversion instruction, and launches of 4 wavefronts that leave registers free keep two slices in
// flight.  us per launch in a graph, before -> with that: bf16, D = 128 (P in one part; two add 1 to 2%) 4 units of 577 rows 6.46 -> 5.44, 32 7.25 -> 5.9,
// 32 of 1100 8.9 -> 7.0, 4 of 2113 8.05 -> 6.9, 32 of 91 4.3 -> 3.8; fp32, D = 128 32 of 528 9.6 -> 7.9, D = 64 64 of 528 8.1 -> 7.1, 2 of 72 4.5 -> 4.2;
// 896 units of 577 and 4608 of 1056 the same to 1%.
// The wavefronts of a workgroup are merged through LDS; pieces of one unit are merged by the
// last workgroup to finish (tickets), in a fixed order, so results are deterministic.
//
// The newest token's k/v are not read from the cache (another workgroup may be writing that
// row): the lanes that would hold row `len` load them from k_new / v_new instead.
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
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
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
__device__ __forceinline__ void ld_v(VWords<Geo<T, D>::VW>& o, const char* p) {
  if constexpr (Geo<T, D>::VW == 2) {
    const u32x2 a = __builtin_nontemporal_load((const u32x2*)p);
    o.w[0] = a[0]; o.w[1] = a[1];
  } else {
    const u32x4 a = __builtin_nontemporal_load((const u32x4*)p);
#pragma unroll
    for (int i = 0; i < 4; ++i) o.w[i] = a[i];
    if constexpr (Geo<T, D>::VW == 8) {
      const u32x4 b = __builtin_nontemporal_load((const u32x4*)(p + 256));
#pragma unroll
      for (int i = 0; i < 4; ++i) o.w[4 + i] = b[i];
    }
  }
}
// One wavefront iteration's loads: KT K tiles (A operands) and 4*KT V rows per lane.
template <typename T, int D, int KT>
struct Slice {
  u32x4 kA[KT][Geo<T, D>::NL];
  VWords<Geo<T, D>::VW> vR[4 * KT];
};

// Two bf16 numbers, zero in place of infinities and NaN.
__device__ __forceinline__ uint32_t finite_pair(uint32_t w) {
  if ((w & 0x00007f80u) == 0x00007f80u) w &= 0xffff0000u;
  if ((w & 0x7f800000u) == 0x7f800000u) w &= 0x0000ffffu;
  return w;
}

struct Nothing { __device__ void operator()() const {} };

// Where a wavefront's loads go: the unit's rows (uniform) and this lane's offsets from a slice's first row, one for
// each K format and one for V.  Everything else about an address is scalar or an immediate.
template <typename T, int D>
struct Rows {
  using G = Geo<T, D>;
  const char *Kh, *Vh;
  int n_tiled;
  uint32_t k_tiled, k_rows, v;
  __device__ __forceinline__ Rows(const char* K, const char* V, int tiled, int lane)
      : Kh(K), Vh(V), n_tiled(tiled), k_tiled(lane * 16), k_rows((lane & 15) * G::ROW_BYTES + (lane >> 4) * 16),
        v((lane >> 4) * 4 * G::ROW_BYTES + (lane & 15) * (G::VW == 2 ? 8 : 16)) {}
};

// Tiles below n_tiled are in tiled format (lane-contiguous 1 KiB per load); tiles above are
// row-major, where the same operand is 16 rows x 64 bytes per load (only the rows appended since
// the last compaction are in that state).
// K is read with ordinary loads, V with non-temporal loads.  Measured on MI355X with this access
// pattern (bf16, D = 128): both ordinary 67-77% of the HBM peak (worst when K+V exceed the 256 MiB
// memory-side cache), both non-temporal 76%, one stream of each kind 80-85% at every cache size
// tried (0.3 to 10 GB), whichever of the two is the non-temporal one.
// APART: a branch for each format, whose steps are immediates then (fewer instructions, for launches that they bound); in
// full launches the branch holds the requests back: bf16, D = 64 1200 units of 1560 rows 78.3 us without, 86.8 with it.
template <bool APART, typename T, int D, int KT>
__device__ __forceinline__ void issue_k(Slice<T, D, KT>& s, const Rows<T, D>& at, int it) {
  using G = Geo<T, D>;
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) {
    const int t = it * KT + tt;
    const char* Kt = at.Kh + (uint32_t)(t * G::TILE_BYTES);
    if (!APART) {
      const bool tiled = 16 * t < at.n_tiled;
      const uint32_t off = tiled ? at.k_tiled : at.k_rows, step = tiled ? 1024 : 64;
#pragma unroll
      for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = ld16(Kt + off + c * step);
    } else if (16 * t < at.n_tiled) {                        // wave-uniform
#pragma unroll
      for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = ld16(Kt + at.k_tiled + c * 1024);
      asm volatile("; tiled");                               // (the branches stay apart: the steps are immediates)
    } else {
#pragma unroll
      for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = ld16(Kt + at.k_rows + c * 64);
      asm volatile("; rows");
    }
  }
}
template <typename T, int D, int KT>
__device__ __forceinline__ void issue_v(Slice<T, D, KT>& s, const Rows<T, D>& at, int it) {
  using G = Geo<T, D>;
  const char* Vt = at.Vh + (uint32_t)(it * KT * G::TILE_BYTES);
#pragma unroll
  for (int jj = 0; jj < 4 * KT; ++jj) ld_v<T, D>(s.vR[jj], Vt + at.v + ((jj & 3) + (jj >> 2) * 16) * G::ROW_BYTES);
}

// The unit's last slice: the lanes that hold row `new_row` take it from the newest token's own k and v.
template <typename T, int D, int KT>
__device__ __forceinline__ void issue_last_k(Slice<T, D, KT>& s, const Rows<T, D>& at, int it, int lane, int new_row, const char* knew) {
  using G = Geo<T, D>;
  asm volatile("" : "+v"(lane));                             // its addresses are formed here, not kept in registers from the start
  const int r = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) {
    const int t = it * KT + tt;
    const bool tiled = 16 * t < at.n_tiled, is_new = 16 * t + r == new_row;
    const char* p = is_new ? knew + kb * 16 : at.Kh + (uint32_t)(t * G::TILE_BYTES) + (tiled ? at.k_tiled : at.k_rows);
    const uint32_t step = is_new || !tiled ? 64 : 1024;
#pragma unroll
    for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = ld16(p + c * step);
  }
}
template <typename T, int D, int KT>
__device__ __forceinline__ void issue_last_v(Slice<T, D, KT>& s, const Rows<T, D>& at, int it, int lane, int new_row, const char* vnew) {
  using G = Geo<T, D>;
  asm volatile("" : "+v"(lane));
  const int r = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int jj = 0; jj < 4 * KT; ++jj) {
    const int key = it * 16 * KT + 4 * kb + (jj & 3) + (jj >> 2) * 16;
    ld_v<T, D>(s.vR[jj], (key == new_row ? vnew : at.Vh + (uint32_t)(key * G::ROW_BYTES)) + r * (G::VW == 2 ? 8 : 16));
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

// Maximum and sum over the four lanes of a head (lane % 16), in each of them: the halves and then the quarters of
// the wavefront change places in registers, where an exchange through LDS takes 60 ns.
// The compiler keeps the wait states that results of matrix and vector instructions need, across branches too, but does not look into
// inline assembly.  The maximum here is safe by its place: its operands are results of an exchange, never of an MFMA, and the next
// exchange needs a copy of its result, with the wait states of a copy.  (fmaxf would quiet both operands first, an instruction each.)
__device__ __forceinline__ float over_head(float x, bool max) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t u = __float_as_uint(x);
    const u32x2 y = i == 0 ? __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(u, u, false, false))
                           : __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(u, u, false, false));
    const float a = __uint_as_float(y[0]), b = __uint_as_float(y[1]);
    if (max) asm("v_max_f32 %0, %1, %2" : "=v"(x) : "v"(a), "v"(b));
    else x = a + b;
  }
  return x;
}

// edge: the slice may contain rows past the end, which are masked.  first: the wavefront's first slice, whose
// accumulators are zero.  between: what to do once the products with K are under way, whose registers are free then.
// EXACT: right for every logit and value, infinities and finite ones of any size among them.  Without
// it, which is what a wavefront tries first, a logit of -inf may give NaN (the scale's low part times -inf), a
// huge maximum any weight (see log2_weight), and an infinite value NaN where P enters in parts (bf16, D = 64, and WHOLE); all of
// them show at the end.
// WHOLE (bf16, D = 128): P as the sum of two bf16 numbers.  A P rounded to one has no error where it is 1, at the largest
// logit of those that share a running maximum, and 2^-9 elsewhere, so the error grows as a unit's slices are dealt to fewer
// wavefronts: 128 units of 470 to 3900 rows, 16 running maxima a unit 3.6e-4 of the result beside the 1.657e-3 of its own rounding, 4
// to 8 of them 4.9e-4 (2-norm, against 64 bits).  Launches that are cut, or would be if their units were longer, deal out by what is fastest, and
// with both parts their error is 2e-6.  It costs 26 instructions a slice: 128 steps of 4 units 741 -> 755 us, 128 ragged units 27.7 -> 28.5.
template <typename T, int D, int KT, bool EXACT, bool WHOLE, typename Between>
__device__ __forceinline__ void process_slice(Slice<T, D, KT>& s, Running<D / 16>& st,
                                              const u32x4 (&qB)[Geo<T, D>::NL], int it, bool first, bool edge,
                                              float scale_log2, float scale_log2_lo, int r, int kb, int n_tot,
                                              Between between) {
  using G = Geo<T, D>;
  constexpr int NS = 4 * KT;
  const int key0 = it * 16 * KT;
  // Rows past the end have zeros for K and V (what is stored there must not reach the matrix cores) and start from the
  // logit -1e30, or -inf: all of it before the products, so that the common path has no branch between them and the maximum.
  f32x4 sc[KT];
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) sc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (edge) {
#pragma unroll
    for (int tt = 0; tt < KT; ++tt)
      if (key0 + 16 * tt + r >= n_tot) {
#pragma unroll
        for (int c = 0; c < G::NL; ++c) s.kA[tt][c] = u32x4{0u, 0u, 0u, 0u};
      }
#pragma unroll
    for (int jj = 0; jj < NS; ++jj) {
      const int key = key0 + (jj & 3) + 4 * kb + (jj >> 2) * 16;
      if (key >= n_tot) {
        if constexpr (!EXACT) sc[jj >> 2][jj & 3] = -1e30f;
#pragma unroll
        for (int i = 0; i < G::VW; ++i) s.vR[jj].w[i] = 0u;
      }
    }
  }

  // scores: sc[tt][e] = q[head r] . k[key0 + 16 tt + 4 kb + e]
#pragma unroll
  for (int tt = 0; tt < KT; ++tt) {
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
  if constexpr (!std::is_same_v<Between, Nothing>) {
    __builtin_amdgcn_sched_barrier(0);
    between();
    __builtin_amdgcn_sched_barrier(0);
  }
  float sv[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    sv[i] = sc[i >> 2][i & 3];
    if constexpr (EXACT) {                                 // (zero times an infinite query is no number)
      const int key = key0 + (i >> 2) * 16 + 4 * kb + (i & 3);
      if (key >= n_tot) sv[i] = -INFINITY;
    }
  }
  float mx = sv[0];
#pragma unroll
  for (int i = 1; i < NS; ++i) mx = fmaxf(mx, sv[i]);
  mx = over_head(mx, true);
  const float m_new = fmaxf(st.m_run, mx * scale_log2);       // scale > 0: max commutes with it
  if (__any(m_new > st.m_run)) {
    const float corr = __builtin_amdgcn_exp2f(st.m_run - m_new);
    st.l_run *= corr;
    if (!first) {
#pragma unroll
      for (int m = 0; m < G::NC; ++m) st.oacc[m] *= corr;
    }
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
  } else if constexpr (WHOLE) {
    // P = hi + lo: hi its upper half and lo the rest, each key twice in a product over 32.  lo may be zero where P is not: hi alone
    // makes an infinite value infinite then (EXACT).
    u32x4 pw;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t a = __float_as_uint(pf[2 * i]), b = __float_as_uint(pf[2 * i + 1]);
      pw[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
      const f32x2 lo = {pf[2 * i] - __uint_as_float(a & 0xffff0000u), pf[2 * i + 1] - __uint_as_float(b & 0xffff0000u)};
      pw[2 + i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
    }
#pragma unroll
    for (int m = 0; m < G::NC; ++m) {
      u32x4 t;
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        t[y] = __builtin_amdgcn_perm(s.vR[2 * y + 1].w[m >> 1], s.vR[2 * y].w[m >> 1],
                                     (m & 1) ? 0x07060302u : 0x05040100u);
        t[2 + y] = EXACT ? finite_pair(t[y]) : t[y];
      }
      st.oacc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(t), as_bf16x8(pw), st.oacc[m], 0, 0, 0);
    }
  } else {
    f32x4 p4;
#pragma unroll
    for (int i = 0; i < 4; ++i) p4[i] = pf[i];
    u32x2 pw;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      pw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{p4[2 * i], p4[2 * i + 1]}), bf16x2));
    const s16x4 pB = __builtin_bit_cast(s16x4, pw);
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
  u32x2 packed;
  packed[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{o[0], o[1]}), bf16x2));
  packed[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{o[2], o[3]}), bf16x2));
  *(u32x2*)p = packed;
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
// 1/l in full precision; `fast`: v_rcp_f32 (2^-23), for uncut bf16 units at D = 128, whose P has 8 or 16
// bits.  Nothing attended to: 0; keys whose logits are all -inf: NaN, as softmax gives.
__device__ __forceinline__ float inv_sum(float l, bool any_key, bool fast) {
  if (!(l > 0.f)) return any_key && l == 0.f ? __builtin_nanf("") : 0.f;
  return fast ? __builtin_amdgcn_rcpf(l) : 1.f / l;
}

// What the kernel needs of a call, all of it requested at once.
struct KernelArgs {
  const int32_t* d_state; const int32_t* step_base;      // step_base: d_state where there is none, and not used
  const char *q, *k_new, *v_new;
  char *K, *V; int32_t* pos; char *qwin, *out;
  float2* stats; float* partials; int32_t* ticket;
  GkvDivisor by_splits, by_hkv, by_iters, by_w;
  int32_t splits, split_iters, Hq, Hkv, g, cap, LB, w, step;
  int32_t has_base, copy_q, write_stats;
  float scale_hi, scale_lo;
};

// When a wavefront with one slice in flight asks for the next one: BEHIND the products with this one, or K EARLY, as soon as
// the products with this K are under way, and V behind its own.  IN_STEP: BEHIND, and a workgroup's wavefronts start on their
// first slices together, so that they go on asking for neighbouring ones at about the same time: without that barrier 18432 units of 1056
// rows take 1558.5 us, with it 1554.  PACED: BEHIND, and wavefronts of workgroups alone on their CU wait a little first, see launch_by_size.
enum class Next { BEHIND, IN_STEP, PACED, EARLY };

// KT = 16-key tiles per wavefront iteration (1 or 2); DEPTH = slices in flight (1 or 2: twice the registers, for launches
// that leave them free).  STAGED: the rows to store wait in LDS instead of registers (32 units of 577 rows 6.1 us against 6.2
// in registers, whatever the room; fp32, D = 128 9.15 / 8.8).
template <typename T, int D, int NW, int KT, int OCC, int DEPTH, Next NEXT, bool STAGED>
__global__ __launch_bounds__(NW * 64, OCC) void attend_mfma_kernel(KernelArgs a) {
  using G = Geo<T, D>;
  constexpr int KEYS = 16 * KT;             // keys per iteration
  constexpr bool WHOLE = DEPTH == 2 && !G::F32 && D == 128;
  constexpr int RP = G::RP, ROW_BYTES = G::ROW_BYTES, OSTR = G::OSTR, PSTR = G::PSTR;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kb = lane >> 4;
  const int splits = a.splits, g = a.g, cap = a.cap;
  const int unit = quotient(blockIdx.x, a.by_splits), sp = (int)blockIdx.x - unit * splits;
  const int lb = quotient(unit, a.by_hkv), j = unit - lb * a.Hkv;
  const size_t head0 = (size_t)lb * a.Hq + j * g;          // the group's first query head
  const char* q_g = a.q + head0 * ROW_BYTES;
  const char* knew_g = a.k_new + (size_t)unit * ROW_BYTES;
  const char* vnew_g = a.v_new + (size_t)unit * ROW_BYTES;
  const bool may_grow = a.k_new != nullptr;
  const bool alone = blockIdx.x < 256 && blockIdx.x + 256 >= gridDim.x;   // on its CU, as workgroups are dealt out (only speed depends on it)

  // A launch of few units is one trip to memory after the other, so everything whose address the arguments
  // give is requested before anything is waited for: the state record and the step counter (scalar loads; no
  // branch on whether there is a counter), the group's queries (B operand of the QK product: lane (head r, kb)
  // holds chunks 4c+kb of q[r]) and the rows stored at the end of the workgroup.
  int4 rec = *(const int4*)(a.d_state + 4 * (size_t)lb);
  const int32_t base = *a.step_base;
  __builtin_amdgcn_sched_barrier(0);
  u32x4 qB[G::NL];
  {
    const uint32_t at = min(r, g - 1) * ROW_BYTES + kb * 16;   // (lanes beyond the group repeat its last head and are ignored)
#pragma unroll
    for (int c = 0; c < G::NL; ++c) qB[c] = ld16(q_g + at + c * 64);
  }
  // 16-byte pieces stored at the end by piece 0 of a unit: [0,RP) k_new and [RP,2RP) v_new, a thread each, and the group's q
  // rows for the window ring; threads without one read a valid address
  constexpr int Q_ROUNDS = (RP * 16 + NW * 64 - 1) / (NW * 64);
  u32x4 kv_piece, q_piece[Q_ROUNDS];
  {
    const uint32_t x = min(tid, 2 * RP - 1);
    const char* src = x < RP ? knew_g + x * 16 : vnew_g + (x - RP) * 16;
    kv_piece = ld16(may_grow ? src : q_g);
#pragma unroll
    for (int rd = 0; rd < Q_ROUNDS; ++rd) q_piece[rd] = ld16(q_g + (uint32_t)min(tid + rd * NW * 64, RP * g - 1) * 16);
  }
  // what can be had without the record, while that is on its way
  const int it0 = sp * NW + wave;              // this wavefront's slices: it0, it0 + stride, ...
  Rows<T, D> at(a.K + (size_t)unit * cap * ROW_BYTES, a.V + (size_t)unit * cap * ROW_BYTES, 0, lane);
  asm volatile("" : "+v"(at.k_tiled), "+v"(at.k_rows), "+v"(at.v));
  __builtin_amdgcn_sched_barrier(0);           // loads come back in order: these before the slice's
  asm volatile("" : "+s"(rec.x), "+s"(rec.y), "+s"(rec.w));   // one load, not one for each of them
  asm volatile("" :: "s"(a.K), "s"(a.V), "s"(a.by_iters.mul), "s"(a.by_iters.shift), "s"(cap), "s"(a.split_iters));   // no argument is fetched behind it
  const SeqState seq = state_record(rec);
  const int step = a.step + (a.has_base ? base : 0);

  // The length comes from the state record and the step number; nothing is written back, so
  // the workgroups of a (layer, sequence) need no ordering among themselves.
  const int len0 = length_before_step(seq, step, cap);
  const bool has_new = may_grow && len0 < cap;
  const int n_tot = len0 + (has_new ? 1 : 0);
  const int n_iter = (int)((uint32_t)(n_tot + KEYS - 1) / KEYS);
  // Pieces this unit is really cut into: as many as its own length fills with `split_iters` slices
  // each (an explicit split count sets split_iters = 0: always all of them).
  int ns = splits;
  if (splits > 1 && a.split_iters > 0) {
    ns = max(1, min(splits, quotient(n_iter + a.split_iters - 1, a.by_iters)));
    if (sp >= ns) return;
  }

  // The unit's last slice may hold the new row and rows past the end.
  const int stride = ns * NW;
  const int new_row = has_new ? len0 : -1;
  at.n_tiled = seq.n_tiled;
  auto request = [&](Slice<T, D, KT>& s, int it) {
    if (it == n_iter - 1) {
      issue_last_k<T, D, KT>(s, at, it, lane, new_row, knew_g);
      issue_last_v<T, D, KT>(s, at, it, lane, new_row, vnew_g);
    } else {
      issue_k<(DEPTH > 1), T, D, KT>(s, at, it);
      issue_v<T, D, KT>(s, at, it);
    }
  };
  Running<G::NC> st;
  const float scale_log2 = a.scale_hi, scale_log2_lo = a.scale_lo;
  auto process = [&](Slice<T, D, KT>& s, int it, bool edge) {
    process_slice<T, D, KT, false, WHOLE>(s, st, qB, it, it == it0, edge, scale_log2, scale_log2_lo, r, kb, n_tot, Nothing{});
  };
  auto reset = [&]() {
    st.m_run = GKV_NO_MAX;
    st.l_run = 0.f;
#pragma unroll
    for (int m = 0; m < G::NC; ++m) st.oacc[m] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // the rows to store wait in LDS, each piece for the thread that brought it, or in registers where there are enough
  char* stage = (char*)(smem + NW * g * OSTR + NW * 16 + NW * 16);
  auto keep_rows = [&]() {
    if (!STAGED) return;
    if (tid < 2 * RP) *(u32x4*)(stage + tid * 16) = kv_piece;
#pragma unroll
    for (int rd = 0; rd < Q_ROUNDS; ++rd) {
      const int x = tid + rd * NW * 64;
      if (x < RP * g) *(u32x4*)(stage + 2 * RP * 16 + x * 16) = q_piece[rd];
    }
  };

  // The first slice, in wavefronts beyond the unit's end its last one (in an empty unit rows that are there), not used.
  Slice<T, D, KT> s0;
  request(s0, min(it0, max(n_iter - 1, 0)));
  reset();
  keep_rows();
  if constexpr (NEXT == Next::IN_STEP) __syncthreads();
  if (it0 < n_iter) {
    int it = it0;
    if constexpr (DEPTH == 1) {
      auto and_then = [&](auto next) {
        process_slice<T, D, KT, false, WHOLE>(s0, st, qB, it, it == it0, false, scale_log2, scale_log2_lo, r, kb, n_tot, next);
      };
      for (; it + stride < n_iter - 1; it += stride) {
        if constexpr (NEXT == Next::EARLY) and_then([&] { issue_k<false, T, D, KT>(s0, at, it + stride); });
        else {
          and_then(Nothing{});
          if constexpr (NEXT == Next::PACED) {
            __builtin_amdgcn_sched_barrier(0);               // (or the requests move up between the products)
            if (alone) __builtin_amdgcn_s_sleep(8);          // 512 cycles
            __builtin_amdgcn_sched_barrier(0);
          }
          issue_k<false, T, D, KT>(s0, at, it + stride);
        }
        issue_v<T, D, KT>(s0, at, it + stride);
      }
      if (it + stride == n_iter - 1) {
        if constexpr (NEXT == Next::EARLY) and_then([&] { issue_last_k<T, D, KT>(s0, at, it + stride, lane, new_row, knew_g); });
        else {
          and_then(Nothing{});
          issue_last_k<T, D, KT>(s0, at, it + stride, lane, new_row, knew_g);
        }
        issue_last_v<T, D, KT>(s0, at, it += stride, lane, new_row, vnew_g);
      }
      process(s0, it, it == n_iter - 1);
    } else {
      // two slices in turn, the next one always on its way
      Slice<T, D, KT> s1;
      if (it + stride >= n_iter) process(s0, it, it == n_iter - 1);
      else {
        request(s1, it + stride);
        for (;;) {
          process(s0, it, false);
          if ((it += stride) + stride >= n_iter) { process(s1, it, it == n_iter - 1); break; }
          request(s0, it + stride);
          process(s1, it, false);
          if ((it += stride) + stride >= n_iter) { process(s0, it, it == n_iter - 1); break; }
          request(s1, it + stride);
        }
      }
    }
    // Seldom: a maximum that the short form of the weights is not right for, or a NaN that may be its
    // doing (a logit of -inf; where P enters in parts an infinite value that met one that is zero or
    // negative).  The slices are gone through again.  (A NaN passes through this maximum; with a comparison for every two
    // accumulators 128 steps of 4 units took 769 us, so 754.)
    bool again = fabsf(st.m_run) >= GKV_HUGE_LOG2 || st.l_run != st.l_run;
    if constexpr (WHOLE || (!G::F32 && D == 64)) {
      float x = st.l_run;
#pragma unroll
      for (int m = 0; m < G::NC; ++m)
#pragma unroll
        for (int e = 0; e < 4; e += 2)
          x = __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, st.oacc[m][e]), st.oacc[m][e + 1]);
      again |= x != x;
    }
    if (__any(again)) {
      reset();
      for (int it = it0; it < n_iter; it += stride) {
        request(s0, it);
        process_slice<T, D, KT, true, WHOLE>(s0, st, qB, it, false, true, scale_log2, scale_log2_lo, r, kb, n_tot, Nothing{});
      }
    }
  }

  // ---- merge the wavefronts of this workgroup -------------------------------------------------
  float* so = smem;                         // [NW][g][OSTR]
  float* sm = so + NW * g * OSTR;           // [16][NW]
  float* sl = sm + NW * 16;                 // [16][NW]
  const float l_tot = over_head(st.l_run, false);      // the 4 lanes of a head hold partial sums
  if (r < g) {
    float* row = so + (wave * g + r) * OSTR;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // accumulators m = 4q .. 4q+3 are four neighbouring channels
#pragma unroll
      for (int q4 = 0; q4 < G::NC / 4; ++q4) {
        const int ch = (G::F32 && D == 128) ? 64 * q4 + 4 * (4 * kb + e) : G::NC * (4 * kb + e) + 4 * q4;
        *(f32x4*)(row + ch) = f32x4{st.oacc[4 * q4][e], st.oacc[4 * q4 + 1][e], st.oacc[4 * q4 + 2][e], st.oacc[4 * q4 + 3][e]};
      }
    }
    if (kb == 0) { sm[r * NW + wave] = st.m_run; sl[r * NW + wave] = l_tot; }
  }
  __syncthreads();

  // one thread per (head, 4 channels): a single round for g <= 8 with 256 threads
  constexpr int TPH = D / 4;                // threads per head
  T* out = (T*)a.out + head0 * D;
  float* part = a.partials + (size_t)(unit * splits) * g * PSTR;      // [ns][g][PSTR]
  const int slot = step - quotient(step, a.by_w) * a.w;
  float2* stats = a.stats + (size_t)slot * a.LB * a.Hq + head0;
  for (int x = tid; x < g * TPH; x += NW * 64) {
    const int h = x / TPH, c4 = (x % TPH) * 4;
    float mw[NW], lw[NW];
#pragma unroll
    for (int i = 0; i < NW / 4; ++i) {
      const f32x4 m4 = *(const f32x4*)(sm + h * NW + 4 * i), l4 = *(const f32x4*)(sl + h * NW + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) { mw[4 * i + e] = m4[e]; lw[4 * i + e] = l4[e]; }
    }
    float M = GKV_NO_MAX;
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) M = fmaxf(M, mw[wv]);
    float Lsum = 0.f;
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < NW; ++wv) {
      const float f = __builtin_amdgcn_exp2f(mw[wv] - M);
      Lsum += lw[wv] * f;
      o += *(const f32x4*)(so + (wv * g + h) * OSTR + c4) * f;
    }
    if (ns == 1) {
      store_row4(out + (uint32_t)(x * 4), o * inv_sum(Lsum, n_tot > 0, !G::F32 && D == 128));
      // softmax statistics of this head's row (running max in log2 units, sum), into the ring slot
      // that also receives q: the window score of the next compression reuses them
      if (c4 == 0 && a.write_stats) stats[h] = make_float2(M, Lsum);
    } else {
      float* ph = part + (uint32_t)((sp * g + h) * PSTR);
      store_agent(ph + c4, o[0], o[1]);
      store_agent(ph + c4 + 2, o[2], o[3]);
      if (c4 == 0) store_agent(ph + D, M, Lsum);
    }
  }

  // ---- pieces: whoever finishes last merges them ------------------------------------------------
  // A wavefront's outputs are whole heads and need the same heads of the other pieces only, so each
  // wavefront has a ticket of its own and no barrier.  The partials go through memory with agent-scope
  // accesses (they pass the XCDs' separate L2s by), each wavefront waits for its own stores, and its
  // ticket follows: no fence, which would write back the whole L2 of the XCD (4 units of 577 rows in 3
  // pieces: 13.4 us with __threadfence, against 8.9 uncut).  (Results that say by a mark of their own whether they are there,
  // asked for together with the ticket: 6.6 us where this takes 5.5; the marks must be put back, stores that
  // the end of the launch waits for.)
  const bool merges = ns > 1 && wave * 64 < g * TPH;       // uniform
  uint32_t arrived = 0;
  if (merges) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // (counts to ns - 1 and starts over; an addition would be made into one over the active lanes and waited for at once)
    if (lane == 0) arrived = __builtin_amdgcn_atomic_inc32((uint32_t*)a.ticket + (size_t)unit * GKV_TICKETS + wave, (uint32_t)ns - 1u, __ATOMIC_RELAXED, "agent");
  }

  // ---- append the new row (row-major, one contiguous row each for K and V), push q into the
  //      window ring (contiguous per KV group).  Rows the other workgroups may still be reading
  //      are never the new row's source: they take k_new / v_new from the inputs. ---------------
  if (sp == 0) {
    if (has_new) {
      const size_t row = ((size_t)unit * cap + len0) * ROW_BYTES;
      if (tid < 2 * RP) *(u32x4*)((tid < RP ? a.K + row : a.V + row - ROW_BYTES) + tid * 16) = STAGED ? *(const u32x4*)(stage + tid * 16) : kv_piece;
      if (tid == NW * 64 - 1) a.pos[(size_t)unit * cap + len0] = step;
    }
    if (a.copy_q) {                          // (q may already live in its ring slot)
      char* ring = a.qwin + ((size_t)slot * a.LB * a.Hq + head0) * ROW_BYTES;
#pragma unroll
      for (int rd = 0; rd < Q_ROUNDS; ++rd) {
        const int x = tid + rd * NW * 64;
        if (x < RP * g) *(u32x4*)(ring + (uint32_t)(x * 16)) = STAGED ? *(const u32x4*)(stage + 2 * RP * 16 + x * 16) : q_piece[rd];
      }
    }
  }

  if (merges && (int)__builtin_amdgcn_readfirstlane(arrived) == ns - 1) {
    asm volatile("" ::: "memory");
    for (int x = tid; x < g * TPH; x += NW * 64) {
      const int h = x / TPH, c4 = (x % TPH) * 4;
      float M = GKV_NO_MAX, Lsum = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
      constexpr int AT_ONCE = 8;
      for (int s0 = 0; s0 < ns; s0 += AT_ONCE) {
        float2 got[AT_ONCE][3];
        const float* ph = part + (uint32_t)((s0 * g + h) * PSTR);
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i)
          if (s0 + i < ns) {                               // uniform, here and below
            got[i][0] = load_agent(ph + D); got[i][1] = load_agent(ph + c4); got[i][2] = load_agent(ph + c4 + 2);
            ph += (uint32_t)(g * PSTR);
          }
        float Mn = M;
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i)
          if (s0 + i < ns) Mn = fmaxf(Mn, got[i][0].x);
        const float f0 = __builtin_amdgcn_exp2f(M - Mn);
        M = Mn;
        Lsum *= f0;
        o *= f0;
#pragma unroll
        for (int i = 0; i < AT_ONCE; ++i)
          if (s0 + i < ns) {
            const float f = __builtin_amdgcn_exp2f(got[i][0].x - Mn);
            Lsum += got[i][0].y * f;
            o += f32x4{got[i][1].x, got[i][1].y, got[i][2].x, got[i][2].y} * f;
          }
      }
      store_row4(out + (uint32_t)(x * 4), o * inv_sum(Lsum, n_tot > 0, false));
      if (c4 == 0 && a.write_stats) stats[h] = make_float2(M, Lsum);
    }
  }
}

}  // namespace

size_t gkv_attend_mfma_lds(int esz, int d, int g, int waves) {
  return sizeof(float) * ((size_t)waves * g * (d + 4) + 2 * 16 * (size_t)waves) + (size_t)(2 + g) * d * esz;
}

template <typename T, int D, int NW, int KT, int OCC, int DEPTH, Next NEXT, bool STAGED = true>
static hipError_t launch_attend(const GkvLaunch& ln, const GkvDims& dm, const AttendArgs& a) {
  const int units = dm.L * dm.B * dm.Hkv;
  KernelArgs k;
  k.d_state = a.d_state; k.step_base = dm.step_base ? dm.step_base : a.d_state;
  k.q = (const char*)a.q; k.k_new = (const char*)a.k_new; k.v_new = (const char*)a.v_new;
  k.K = (char*)a.K; k.V = (char*)a.V; k.pos = a.pos; k.qwin = (char*)a.qwin; k.out = (char*)a.out;
  k.stats = a.ws.stats; k.partials = a.ws.partials; k.ticket = a.ws.split_ticket;
  k.by_splits = gkv_divisor(a.splits); k.by_hkv = dm.by_hkv; k.by_w = gkv_divisor(dm.w);
  k.by_iters = gkv_divisor(a.split_iters > 0 ? a.split_iters : 1);
  k.splits = a.splits; k.split_iters = a.split_iters;
  k.Hq = dm.Hq; k.Hkv = dm.Hkv; k.g = dm.g; k.cap = dm.cap; k.LB = dm.L * dm.B; k.w = dm.w; k.step = a.step;
  k.has_base = dm.step_base != nullptr; k.copy_q = a.copy_q; k.write_stats = a.write_stats;
  k.scale_hi = dm.scale_l2_hi; k.scale_lo = dm.scale_l2_lo;
  const size_t shmem = gkv_attend_mfma_lds(sizeof(T), D, dm.g, NW);
  return gkv_launch(ln, attend_mfma_kernel<T, D, NW, KT, OCC, DEPTH, NEXT, STAGED>, dim3(units * a.splits), dim3(NW * 64), shmem, k);
}

// The form of a launch of 4 or 8 wavefronts, by its number of workgroups.
template <typename T, int D, int NW, int KT, int OCC>
static hipError_t launch_by_size(const GkvLaunch& ln, const GkvDims& dm, const AttendArgs& a) {
  constexpr bool BF128 = sizeof(T) == 2 && D == 128, F128 = sizeof(T) == 4 && D == 128;
  const int64_t workgroups = (int64_t)dm.L * dm.B * dm.Hkv * a.splits;
  if constexpr (NW == 4) {
    // a workgroup per CU at most: registers for two slices in flight (fp32, D = 128 has none to spare).  Not with 8 wavefronts, which
    // have requests enough (us with two slices -> one: bf16, D = 128 256 units of 3000 rows 64.7 -> 60.7, 200 of 1500 24.9 -> 24.4,
    // 4 of 260 4.9 -> 4.6, D = 64 256 of 1500 17.5 -> 17.0, 128 of 528 7.0 -> 6.45; fp32, D = 64 256 of 1500 32.7 -> 31.9).
    if (workgroups <= 256) return launch_attend<T, D, NW, KT, 2, F128 ? 1 : 2, Next::EARLY, BF128>(ln, dm, a);
    // Up to 512 workgroups some CUs have two and others one, and the CUs with two end last.  The others' wavefronts, alone on their
    // SIMDs, are done with a slice sooner and, the fewer instructions it takes, ask the more often for the memory that all share: what made
    // slices shorter made these launches slower.  So they wait 512 cycles a slice (us, without -> with; 192 and 1024 cycles): bf16, D =
    // 128 270 units of 2000 rows 55.3 -> 50.7 (52.9, 49.5), 400 of 1100 38.8 -> 37.4 (38.0, 36.8), 448 of 577 22.35 -> 22.2, 300 ragged to 2500 43.9
    // -> 44.6 (44.5, 49.2); D = 64 270 of 3000 42.9 -> 38.6 (39.1, 40.4); fp32, D = 64 336 of 1541 47.9 -> 45.7, but D = 128 280 ragged to 470 18.65 ->
    // 19.0, 400 of 900 66.5 -> 66.75.  (K early there: 336 of 1541 49.7, 280 ragged 24.8 where BEHIND took 23.6; 8 wavefronts: 270 of 2000 59.5.)
    if (workgroups <= 512) return launch_attend<T, D, NW, KT, OCC, 1, F128 ? Next::BEHIND : Next::PACED>(ln, dm, a);
    // K early gains where the launch fills the chip (us, without -> with: bf16, D = 128 1200 units of 860 rows 93.7 -> 87.7; fp32,
    // D = 128 800 of 540 84.8 -> 82.4, 32 of 528 8.2 -> 7.9, D = 64 1200 of 860 90.0 -> 88.8).
    return launch_attend<T, D, NW, KT, OCC, 1, Next::EARLY>(ln, dm, a);
  } else {
    // K early loses with 8 wavefronts at bf16, D = 128 (784 ragged to 1227 48.7 -> 49.7)
    if (workgroups <= 256) return launch_attend<T, D, NW, KT, OCC, 1, Next::BEHIND>(ln, dm, a);
    return launch_attend<T, D, NW, KT, OCC, 1, BF128 ? Next::IN_STEP : Next::EARLY>(ln, dm, a);
  }
}

hipError_t gkv_launch_attend_mfma(const GkvLaunch& ln, const GkvDims& dm, int dtype, const AttendArgs& a) {
  if (dtype == GKV_F32) {
    if (dm.d == 64) {
      if (a.waves == 16) return launch_attend<float, 64, 16, 1, 4, 1, Next::EARLY>(ln, dm, a);
      if (a.waves == 8) return launch_by_size<float, 64, 8, 1, 4>(ln, dm, a);
      return launch_by_size<float, 64, 4, 1, 4>(ln, dm, a);
    }
    if (a.waves >= 8) return launch_attend<float, 128, 8, 1, 2, 1, Next::EARLY>(ln, dm, a);
    return launch_by_size<float, 128, 4, 1, 2>(ln, dm, a);
  }
  if (dm.d == 64) {
    if (a.waves == 16) return launch_attend<uint16_t, 64, 16, 2, 4, 1, Next::EARLY>(ln, dm, a);
    if (a.waves == 8) return launch_by_size<uint16_t, 64, 8, 2, 4>(ln, dm, a);
    return launch_by_size<uint16_t, 64, 4, 2, 4>(ln, dm, a);
  }
  if (a.waves == 16) return launch_attend<uint16_t, 128, 16, 1, 2, 1, Next::BEHIND>(ln, dm, a);
  if (a.waves == 8) return launch_by_size<uint16_t, 128, 8, 1, 4>(ln, dm, a);
  if (a.tile_keys == 32) return launch_attend<uint16_t, 128, 4, 2, 2, 1, Next::EARLY>(ln, dm, a);
  return launch_by_size<uint16_t, 128, 4, 1, 4>(ln, dm, a);
}
