// Global-score update, top-(b-w) selection and in-place compaction.  The first two take one workgroup of
// 256 threads per unit, compaction two or more of 256 or 1024; all score arithmetic in fp32, all index
// work in integers.
#include "gkv_internal.h"

namespace {

// 16-byte piece as a native vector (arrays of it stay in registers; the runtime's uint4 class does not)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

// ---- helpers -------------------------------------------------------------------------------
// Across the lanes of a wavefront through registers (an exchange through LDS takes 60 ns): inclusive sums, and the
// maximum of numbers that are not negative in every lane.
#define GKV_DPP_I(v, ctrl, rows) __builtin_amdgcn_update_dpp(0, v, ctrl, rows, 0xF, false)
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += GKV_DPP_I(v, 0x111, 0xF);                 // row_shr 1, 2, 4, 8
  v += GKV_DPP_I(v, 0x112, 0xF);
  v += GKV_DPP_I(v, 0x114, 0xF);
  v += GKV_DPP_I(v, 0x118, 0xF);
  v += GKV_DPP_I(v, 0x142, 0xA);                 // lane 15 of a row to the next row, then lane 31 to the upper half
  v += GKV_DPP_I(v, 0x143, 0xC);
  return v;
}
__device__ __forceinline__ float wave_max_nonneg(float v) {
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const int u = __float_as_int(v);
    const int w = q == 0 ? GKV_DPP_I(u, 0x111, 0xF) : q == 1 ? GKV_DPP_I(u, 0x112, 0xF) : q == 2 ? GKV_DPP_I(u, 0x114, 0xF)
                : q == 3 ? GKV_DPP_I(u, 0x118, 0xF) : q == 4 ? GKV_DPP_I(u, 0x142, 0xA) : GKV_DPP_I(u, 0x143, 0xC);
    v = fmaxf(v, __int_as_float(w));             // (lanes without a source get 0)
  }
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Inclusive scan over the 256 threads of a block; `tmp` holds 4 ints of LDS.
__device__ __forceinline__ int block_inclusive_scan(int v, int* tmp) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  v = wave_inclusive_sum(v);
  __syncthreads();
  if (lane == 63) tmp[wv] = v;
  __syncthreads();
  int add = 0;
  for (int i = 0; i < wv; ++i) add += tmp[i];
  return v + add;
}

// Monotone map float -> uint32 (larger float, larger key); -0 is folded onto +0 first.
__device__ __forceinline__ uint32_t sortable_key(float f) {
  f = f + 0.0f;
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// ---- global score (Section 4) and top-(b-w) ---------------------------------------------------
// One kernel for gkv_global_update (UPDATE), gkv_select_topk (SELECT) and the two in one launch.
// A thread keeps its entries n = tid + 256 i, i < IPT, in registers.  They are requested before the
// state record has arrived (every index is below the capacity), so a workgroup makes one trip to
// memory, not three.
//
// UPDATE: Sn = S / max S, combined with alpha * F_hist, written to F_out (and selected on).
//
// SELECT: the k-th largest key bit pair by bit pair from the top.  With p the bits found so far, the
// entries at or above p + 1, p + 2, p + 3 (in the pair's place) are counted with ballots, one word per
// wavefront and count passes through LDS, and the largest of them with at least k entries becomes p;
// as soon as exactly k entries are at or above p these are the kept ones, which scores that are
// not tied reach after half the pairs.  Otherwise p ends as the k-th largest key, and of the entries
// equal to it the first k - (number above it) by index are kept.  Kept entries are numbered by ballots
// and one scan over the (i, wavefront) counts: ascending indices, always k of them, whatever the bits.
// Bound: latency (launch, one memory trip, about ten barriers).  Against a radix select by 8-bit
// digits in LDS (four passes of atomics, scans and six barriers), update and selection in one launch: 4 units
// of 624 candidates 8.5 -> 7.0 us, 256 of 1056 12.7 -> 9.5; the update alone, which read S twice, 11.2 -> 6.3
// at 1792 units of 1136; the selection alone there 16.7 to 18.6 -> 16.4 to 19.0 by the scores (by then the
// counting is the bound), 896 units of 624 9.1 -> 8.4.  Maximum, scan and look-ups through registers, four counts to a word of
// LDS (in a graph): selection of 4 units of 640 rows 5.5 -> 5.05 us, 64 of 1152 7.1 -> 6.6, 1792 of 1152 13.0 -> 12.6; update 2.6 -> 2.1, 3.0 -> 2.6, 5.5 ->
// 5.0.  (The counts as scalars: 12.6 -> 14.2 at 1792 units.)
template <int IPT, bool UPDATE, bool SELECT>
__global__ __launch_bounds__(256) void score_topk_kernel(GkvDims dm, const float* __restrict__ S,
                                                         const float* __restrict__ F_hist,
                                                         const int32_t* __restrict__ d_state, int step,
                                                         float* __restrict__ F_out, int32_t* __restrict__ keep_idx) {
  step = resolve_step(dm, step);
  __shared__ __attribute__((aligned(16))) float red[4];
  __shared__ i32x4 cnt[2][4];
  __shared__ int scan_s[64];
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv), tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* Su = S + (size_t)unit * dm.cap;
  float f[IPT], h[UPDATE ? IPT : 1];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int n = tid + 256 * i;
    f[i] = n < dm.cap ? Su[n] : 0.f;
    if constexpr (UPDATE) h[i] = n < dm.cap ? F_hist[(size_t)unit * dm.cap + n] : 0.f;
  }
  const SeqState st = load_state(d_state, lb);
  const int l = compression_length(st, step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const int c = l - dm.w;

  if constexpr (UPDATE) {
    int n_hist = st.n_hist;
    n_hist = n_hist < 0 ? 0 : (n_hist > c ? c : n_hist);
    float* Fu = F_out + (size_t)unit * dm.cap;
    float mx = 0.f;
#pragma unroll
    for (int i = 0; i < IPT; ++i)
      if (tid + 256 * i < c) mx = fmaxf(mx, f[i]);
    mx = wave_max_nonneg(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int n = tid + 256 * i;
      const float sn = mx > 0.f ? f[i] / mx : 0.f;
      f[i] = sn;
      if (n < n_hist) {
        const float hh = dm.alpha * h[i];
        f[i] = dm.combine == GKV_COMBINE_MAX ? fmaxf(hh, sn)
             : dm.combine == GKV_COMBINE_AVG ? hh + (1.f - dm.alpha) * sn
                                             : hh + sn;
      }
      if (n < c) Fu[n] = f[i];
    }
  }
  if constexpr (SELECT) {
    const int k = dm.b - dm.w;                   // c > k because l > b
    uint32_t key[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) key[i] = tid + 256 * i < c ? sortable_key(f[i]) : 0u;   // 0 is never counted below
    uint32_t prefix = 0;
    bool exact = false;                          // exactly k entries are at or above prefix
    for (int pass = 15; pass >= 0 && !exact; --pass) {
      int mine[3] = {0, 0, 0};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const uint32_t t = prefix | ((uint32_t)(q + 1) << (2 * pass));
#pragma unroll
        for (int i = 0; i < IPT; ++i) mine[q] += __popcll(__ballot(key[i] >= t));
      }
      i32x4 (&slot)[4] = cnt[pass & 1];          // two sets in turn: one barrier per pass
      if (lane == 0) slot[wave] = i32x4{mine[0], mine[1], mine[2], 0};
      __syncthreads();
      const i32x4 all = (slot[0] + slot[1]) + (slot[2] + slot[3]);
      uint32_t digit = 0;
      int got = 0;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const int n_ge = all[q];
        if (n_ge >= k) { digit = q + 1; got = n_ge; }          // counts fall with q
      }
      prefix |= digit << (2 * pass);
      exact = digit != 0 && got == k;
    }
    // Entries above prefix, and equal to it: counts per (i, wavefront) in index order.
    uint64_t above[IPT], equal[IPT];
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const bool in = tid + 256 * i < c;
      above[i] = __ballot(in && (exact ? key[i] >= prefix : key[i] > prefix));
      equal[i] = __ballot(in && !exact && key[i] == prefix);
      if (lane == 0) scan_s[4 * i + wave] = __popcll(above[i]) | (__popcll(equal[i]) << 16);
    }
    __syncthreads();
    const int v = wave_inclusive_sum(lane < 4 * IPT ? scan_s[lane] : 0);   // low half: above, high half: equal (at most 4096 of each)
    const int rest = k - (__builtin_amdgcn_readlane(v, 63) & 0xffff);      // how many of the equal ones are kept
    int32_t* Ku = keep_idx + (size_t)unit * k;
    const uint64_t below = (1ull << lane) - 1;
#pragma unroll
    for (int i = 0; i < IPT; ++i) {
      const int at = 4 * i + wave - 1;
      const int before = at < 0 ? 0 : __builtin_amdgcn_readlane(v, at < 0 ? 0 : at);
      const int n_above = (before & 0xffff) + __popcll(above[i] & below);
      const int n_equal = (before >> 16) + __popcll(equal[i] & below);
      const bool is_above = (above[i] >> lane) & 1, is_equal = (equal[i] >> lane) & 1;
      const int out = n_above + min(n_equal, rest);
      if ((is_above || (is_equal && n_equal < rest)) && out < k) Ku[out] = tid + 256 * i;
    }
  }
}

template <bool UPDATE, bool SELECT>
hipError_t launch_score_topk(const GkvLaunch& ln, const GkvDims& dm, const float* S, const float* F_hist,
                             const int32_t* d_state, int32_t step, float* F_out, int32_t* keep_idx) {
  const int per = (dm.cap + 255) / 256;                          // capacity <= 4096: at most 16
  auto kern = per <= 1 ? score_topk_kernel<1, UPDATE, SELECT> : per <= 2 ? score_topk_kernel<2, UPDATE, SELECT>
            : per <= 3 ? score_topk_kernel<3, UPDATE, SELECT> : per <= 5 ? score_topk_kernel<5, UPDATE, SELECT>
            : per <= 9 ? score_topk_kernel<9, UPDATE, SELECT> : score_topk_kernel<16, UPDATE, SELECT>;
  return gkv_launch(ln, kern, dim3(dm.L * dm.B * dm.Hkv), dim3(256), 0, dm, S, F_hist, d_state, (int)step, F_out, keep_idx);
}

// ---- compaction ----------------------------------------------------------------------------
// grid (units, 2 * shares): the first `shares` workgroups of a unit move K (the very first one pos and
// F_hist too), the others V (row-major); a share is a range of 16-byte columns of every row, so the
// shares of a unit have nothing to do with each other.  Not so where K changes its format (N_TILED is
// not the new one, as in a prompt's first compression): a tile's columns then land on other columns of
// its own rows, and the first share moves them all.
// K source rows are in tiled format below the old N_TILED and row-major above; destination rows
// are tiled below nt_new = b rounded down to 16 and row-major above.  Both formats keep a
// 16-row tile inside the same tile-sized block, so the stable-compaction argument still holds
// with chunks that start on tile boundaries: rows are produced in ascending chunks, every
// source piece of a chunk is loaded, then a barrier, then the stores.  Destination index <=
// source index and sources ascend, so a chunk's stores (which stay inside the chunk's tiles)
// never touch a row that a later chunk still has to read.
// State record: every workgroup reads it at its start.  With a ticket array (one counter per
// (layer, sequence), zero between launches) the workgroup that finishes last among the 2 h_kv shares
// of a (layer, sequence) knows that all of them have read the record, and rewrites it; no data
// depends on that write inside this launch, so the counter needs no fence.  Without a ticket
// array a separate launch rewrites the records.
// Dynamic LDS: int keep_s[b - w]: the kept indices, read from memory once.
// Bound: HBM at hundreds of units; instructions below, as many as a lone wavefront issues in turn.
// POW2: rows of 2^np_log pieces (bf16 and fp32 at d = 64 and 128, among others): a thread's piece is the same in every row it moves, rows
// follow by a constant, and nothing is divided at run time (us with the copy of the record, in a graph, before -> now: 4 units of b =
// 98 6.2 -> 5.7, of 512 8.7 -> 8.0, 32 of 512 10.7 -> 10.2, fp32 8 of 322 9.3 -> 8.7).
template <int PPT, int NT, bool SHARED, bool POW2>
__global__ __launch_bounds__(NT) void compact_kernel(GkvDims dm, int esz, int np_log, const int32_t* __restrict__ keep_idx,
                                                     const float* __restrict__ F, void* K, void* V,
                                                     float* __restrict__ F_hist, int32_t* pos,
                                                     int32_t* d_state, int step, int32_t* state_ticket, int shares) {
  step = resolve_step(dm, step);
  if constexpr (!SHARED) shares = 1;             // known to the compiler
  extern __shared__ int keep_s[];
  __shared__ int red_i[NT / 64];
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv), tid = threadIdx.x;
  const bool isK = (int)blockIdx.y < shares;
  const int share = isK ? blockIdx.y : blockIdx.y - shares;
  const bool isPos = blockIdx.y == 0;
  const int k = dm.b - dm.w, b = dm.b;
  const int32_t* Ku = keep_idx + (size_t)unit * k;
  // the first kept indices of a thread, requested before the state record is waited for: as many as there are
  // (all four for a short unit too, copies of its last: 4 units of b = 200 6.55 -> 6.65 us, 896 of b = 98 20.3 -> 20.7)
  constexpr int EARLY = 4;
  int early[EARLY];
#pragma unroll
  for (int i = 0; i < EARLY; ++i) {
    early[i] = 0;
    if (i == 0 || NT * i < k) early[i] = Ku[min(tid + NT * i, k - 1)];
  }
  const SeqState st = load_state(d_state, lb);
  const int l = compression_length(st, step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const int c = l - dm.w;
  const int nt_old = st.n_tiled, nt_new = b & ~15;

  // first destination row whose source differs from it; a K format change rewrites everything
  int first = k;
#pragma unroll
  for (int i = 0; i < EARLY; ++i) {
    const int n = tid + NT * i;
    if (n < k) {
      keep_s[n] = early[i];
      if (early[i] != n && first == k) first = n;
    }
  }
  for (int n = tid + NT * EARLY; n < k; n += NT) {
    const int src = Ku[n];
    keep_s[n] = src;
    if (src != n && first == k) first = n;       // ascending per thread: the first hit is its minimum
  }
  for (int o = 32; o > 0; o >>= 1) first = min(first, __shfl_xor(first, o));
  if ((tid & 63) == 0) red_i[tid >> 6] = first;
  __syncthreads();
  first = red_i[0];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) first = min(first, red_i[i]);
  if (isK && nt_old != nt_new) first = 0;
  first &= ~15;                                  // chunks start on tile boundaries

  if (isPos) {
    float* Hu = F_hist + (size_t)unit * dm.cap;
    const float* Fu = F + (size_t)unit * dm.cap;
    for (int n = tid; n < k; n += NT) {
      int src = keep_s[n];
      src = src < 0 ? 0 : (src >= c ? c - 1 : src);
      Hu[n] = Fu[src];
    }
  }

  const int NP = POW2 ? 1 << np_log : dm.d * esz / 16;   // 16-byte pieces per row
  const bool whole = !SHARED || (isK && nt_old != nt_new);
  const int PS = whole ? NP : NP / shares, p0 = whole ? 0 : share * PS;   // this share's
  const int ps_log = POW2 ? __builtin_ctz(PS) : 0;
  const int end = whole && share > 0 ? 0 : b;
  constexpr int PR = NT > 256 ? 2 : 1;           // positions per thread and chunk
  int R = POW2 ? (NT * PPT) >> ps_log : (NT * PPT) / PS;   // rows per chunk: whole tiles, at most PR per thread
  R = (R > PR * NT ? PR * NT : R) & ~15;
  u32x4* base = (u32x4*)((char*)(isK ? K : V) + (size_t)unit * dm.cap * dm.d * esz);
  int32_t* pu = pos + (size_t)unit * dm.cap;

  // Every load of a round is issued before the first wait: the addresses are computed without
  // branches (pieces beyond the chunk or the budget read row 0, always in bounds, and are not
  // stored), so the PPT 16-byte loads of a thread are in flight together.
  auto source = [&](int row) {
    int src = keep_s[row < k ? row : 0];
    src = row < k ? src : c + (row - k);
    return src < 0 ? 0 : (src >= l ? l - 1 : src);
  };
  const int old_tiled = isK ? nt_old : 0, new_tiled = isK ? nt_new : 0;
  auto pow2_offset = [&](int row, int piece, int n_tiled) {
    const int in = row & 15;
    return row < n_tiled ? (row << np_log) + (piece << 4) + in - (in << np_log) : (row << np_log) + piece;
  };
  using Index = std::conditional_t<POW2, uint32_t, int>;
  for (int r0 = first; r0 < end; r0 += R) {
    u32x4 buf[PPT];
    int dst[PPT];
#pragma unroll
    for (int i = 0; i < PPT; ++i) {
      const int x = tid + NT * i;
      const int rr = POW2 ? (tid >> ps_log) + i * (NT >> ps_log) : x / PS;
      const int piece = p0 + (POW2 ? tid & (PS - 1) : x % PS);
      const int row = r0 + rr;
      const bool valid = rr < R && row < b;
      const int src = valid ? source(row) : 0;
      Index so;
      int d_o;
      if constexpr (POW2) {
        so = pow2_offset(src, piece, old_tiled);
        d_o = pow2_offset(row, piece, new_tiled);
      } else {
        so = (isK && src < nt_old) ? ((src >> 4) * 16 * NP + piece * 16 + (src & 15)) : (src * NP + piece);
        d_o = (isK && row < nt_new) ? ((row >> 4) * 16 * NP + piece * 16 + (row & 15)) : (row * NP + piece);
      }
      dst[i] = valid ? d_o : -1;
      buf[i] = base[so];
    }
    int pos_val[PR];
#pragma unroll
    for (int i = 0; i < PR; ++i) {
      const int rr = tid + NT * i;
      pos_val[i] = pu[isPos && rr < R && r0 + rr < b ? source(r0 + rr) : 0];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PPT; ++i)
      if (dst[i] >= 0) base[(Index)dst[i]] = buf[i];
#pragma unroll
    for (int i = 0; i < PR; ++i) {
      const int rr = tid + NT * i;
      if (isPos && rr < R && r0 + rr < b) pu[r0 + rr] = pos_val[i];
    }
  }
  // (every wavefront of this workgroup passed the barrier above after reading the record)
  if (state_ticket != nullptr && tid == 0) {
    const int done = atomicAdd(&state_ticket[lb], 1);
    if (done == 2 * shares * dm.Hkv - 1) {
      state_ticket[lb] = 0;
      *(int4*)(d_state + 4 * (size_t)lb) = make_int4(dm.b, step + 1, dm.b - dm.w, dm.b & ~15);
    }
  }
}

// ---- sequence-wise max-pooling of a score over the candidates --------------------------------
// Dynamic LDS: float f[cap]
__global__ __launch_bounds__(256) void pool_scores_kernel(GkvDims dm, const float* __restrict__ F,
                                                          const int32_t* __restrict__ d_state, int step,
                                                          int kernel, float* __restrict__ F_out) {
  step = resolve_step(dm, step);
  extern __shared__ float fbuf[];
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv), tid = threadIdx.x;
  const int l = compression_length(load_state(d_state, lb), step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const int c = l - dm.w, half = kernel / 2;
  const float* Fu = F + (size_t)unit * dm.cap;
  for (int n = tid; n < c; n += 256) fbuf[n] = Fu[n];
  __syncthreads();
  float* Fo = F_out + (size_t)unit * dm.cap;
  for (int n = tid; n < c; n += 256) {
    const int lo = max(0, n - half), hi = min(c - 1, n + half);
    float m = fbuf[lo];
    for (int x = lo + 1; x <= hi; ++x) m = fmaxf(m, fbuf[x]);
    Fo[n] = m;
  }
}

// ---- eviction log: original positions of the candidates that are about to be dropped -------
// A compression from l rows drops l - b of them: s in steady state, up to capacity - b when a
// prompt longer than the budget is compressed, hence capacity - b log entries per unit.
// Dynamic LDS: uint32 kept[cap]
__global__ __launch_bounds__(256) void evicted_positions_kernel(GkvDims dm, const int32_t* __restrict__ keep_idx,
                                                                const int32_t* __restrict__ pos,
                                                                const int32_t* __restrict__ d_state, int step,
                                                                int32_t* __restrict__ evicted) {
  step = resolve_step(dm, step);
  extern __shared__ uint32_t kept[];
  __shared__ int tmp[4];
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv), tid = threadIdx.x;
  const int n_log = dm.cap - dm.b;
  int32_t* Eu = evicted + (size_t)unit * n_log;
  const int l = compression_length(load_state(d_state, lb), step, dm.b, dm.w, dm.cap);
  if (l == 0) {
    for (int i = tid; i < n_log; i += 256) Eu[i] = -1;
    return;
  }
  const int c = l - dm.w, k = dm.b - dm.w;
  for (int n = tid; n < c; n += 256) kept[n] = 0u;
  __syncthreads();
  const int32_t* Ku = keep_idx + (size_t)unit * k;
  for (int r = tid; r < k; r += 256) {
    const int n = Ku[r];
    if (n >= 0 && n < c) kept[n] = 1u;
  }
  __syncthreads();
  const int per = (c + 255) / 256;
  const int lo = tid * per, hi = min(c, lo + per);
  int n_out = 0;
  for (int n = lo; n < hi; ++n) n_out += (kept[n] == 0u);
  int out = block_inclusive_scan(n_out, tmp) - n_out;
  const int32_t* pu = pos + (size_t)unit * dm.cap;
  for (int n = lo; n < hi; ++n)
    if (kept[n] == 0u && out < n_log) Eu[out++] = pu[n];
  // pad what is left (exactly c - k = l - b rows are dropped when keep_idx holds k distinct candidates)
  const int total = c - k;
  for (int i = total + tid; i < n_log; i += 256) Eu[i] = -1;
}

__global__ void finalize_state_kernel(GkvDims dm, int32_t* d_state, int step) {
  step = resolve_step(dm, step);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= dm.L * dm.B) return;
  const SeqState st = load_state(d_state, i);
  const int l = compression_length(st, step, dm.b, dm.w, dm.cap);
  if (l > 0) *(int4*)(d_state + 4 * (size_t)i) = make_int4(dm.b, step + 1, dm.b - dm.w, dm.b & ~15);
}

__global__ void add_int_kernel(int32_t* p, int32_t delta) { *p += delta; }

__global__ void fill_zero_kernel(int32_t* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

}  // namespace

hipError_t gkv_launch_global_update(const GkvLaunch& ln, const GkvDims& dm, const float* S,
                                    const float* F_hist, const int32_t* d_state, int32_t step, float* F_out) {
  return launch_score_topk<true, false>(ln, dm, S, F_hist, d_state, step, F_out, nullptr);
}

hipError_t gkv_launch_select_topk(const GkvLaunch& ln, const GkvDims& dm, const float* F,
                                  const int32_t* d_state, int32_t step, int32_t* keep_idx) {
  return launch_score_topk<false, true>(ln, dm, F, nullptr, d_state, step, nullptr, keep_idx);
}

hipError_t gkv_launch_update_and_select(const GkvLaunch& ln, const GkvDims& dm, const float* S, const float* F_hist,
                                        const int32_t* d_state, int32_t step, float* F_out, int32_t* keep_idx) {
  return launch_score_topk<true, true>(ln, dm, S, F_hist, d_state, step, F_out, keep_idx);
}

hipError_t gkv_launch_compact(const GkvLaunch& ln, const GkvDims& dm, int esz, const int32_t* keep_idx,
                              const float* F, void* K, void* V, float* F_hist, int32_t* pos,
                              int32_t* d_state, int32_t step, int32_t* state_ticket) {
  const int units = dm.L * dm.B * dm.Hkv;
  const size_t shmem = sizeof(int) * (size_t)(dm.b - dm.w);
  const int ppt = ln.ctx ? ln.ctx->compact_ppt : 8;
  // A workgroup moves its rows in rounds of 32 KiB whose loads wait for the stores before them, about
  // 2.5 us each; with few units the chip is empty meanwhile, so the rows' columns are shared out (at
  // least 64 bytes of a row each) and a share of more than 64 KiB gets 1024 threads, four times the round; up to 16 units
  // one of more than 32 KiB too if it would be more than two rounds of 256 rows (with the record's copy in a graph:
  // bf16 8 units of b = 630 10.8 -> 9.7, 4 of 1000 12.9 -> 9.9; in two rounds the wider workgroup starts later than it saves: fp32,
  // d = 128 4 of b = 322 9.3 -> 9.7, 8 of 400 9.7 -> 9.85, 16 of 322 9.6 -> 9.95, even at b = 512, 10.45 -> 10.2 at 8 units; 64 bf16 of 512
  // 10.6 -> 11.0).
  // us per launch, whole -> shared (bf16, d = 128): 4 units of b = 512 13.8 -> 7.2, of b = 2048 43.1 -> 10.8;
  // 32 of 2048 47.1 -> 14.6; 64 of 1024 26.1 -> 14.2; 128 of 2048 61.4 -> 51.2.  From 256 units on both
  // cost more than they bring (256 of 2048 120.3 -> 120.9 in halves, 126 with 1024 threads).
  const int row_bytes = dm.d * esz, pieces = row_bytes / 16;
  const int64_t unit_bytes = (int64_t)dm.b * row_bytes;
  int shares = units <= 16 || (units <= 32 && unit_bytes >= 256 * 1024) ? 4 : units <= 128 ? 2 : 1;
  while (shares > 1 && (pieces % shares != 0 || pieces / shares < 4)) shares >>= 1;
  const bool wide = ppt == 8 && units <= 128 && unit_bytes / shares > (units <= 16 && dm.b > 2 * 256 ? 32 : 64) * 1024;
  // One share is an instantiation of its own: with the column arithmetic at run time 672 units of b = 287, d = 64
  // take 25.3 us, without 25.0; 604 of b = 323 21.6 / 21.4.
  // Without divisions up to 512 units, whose two workgroups a unit, four a CU, all run at once.  us between two events, cold
  // caches, with the divisions -> without: bf16, d = 128 4 units of b = 100 7.8 -> 7.1, 32 of 505 12.9 -> 12.3, 96 of 1024 33.2 -> 31.2, 256 of 256
  // 25.0 -> 24.0, of 700 51.5 -> 50.7, 336 of 256 32.4 -> 31.6, 512 of 256 39.7 -> 38.6, fp32 384 of 400 103.9 -> 103.6, but 160 of 505 31.0 -> 31.7, 256 of
  // 1024 65.9 -> 67.0, 336 of 700 69.4 -> 70.1.  Above, memory is the bound and it goes either way: 911 of 533 121.7 -> 124.1, 1792 of 2048 799.0 ->
  // 804.8, fp32 600 of 400 136.6 -> 138.1, but 9216 of 90 224.1 -> 220.8, bf16, d = 64 640 of 500 46.8 -> 44.1.
  const bool pow2 = (pieces & (pieces - 1)) == 0 && units <= 512;
  const int np_log = pow2 ? __builtin_ctz(pieces) : 0;
#define GKV_COMPACT(PPT_, NT_) (shares > 1 ? (pow2 ? compact_kernel<PPT_, NT_, true, true> : compact_kernel<PPT_, NT_, true, false>) \
                                           : (pow2 ? compact_kernel<PPT_, NT_, false, true> : compact_kernel<PPT_, NT_, false, false>))
  auto kern = ppt == 16 ? GKV_COMPACT(16, 256) : ppt == 4 ? GKV_COMPACT(4, 256) : wide ? GKV_COMPACT(8, 1024) : GKV_COMPACT(8, 256);
#undef GKV_COMPACT
  const int threads = wide ? 1024 : 256;
  hipError_t e = gkv_launch(ln, kern, dim3(units, 2 * shares), dim3(threads), shmem, dm, esz, np_log, keep_idx, F, K, V,
                            F_hist, pos, d_state, (int)step, state_ticket, shares);
  if (e != hipSuccess || state_ticket != nullptr) return e;
  const int nlb = dm.L * dm.B;
  GkvLaunch plain{ln.ctx, -1, ln.stream};
  return gkv_launch(plain, finalize_state_kernel, dim3((nlb + 255) / 256), dim3(256), 0, dm, d_state, (int)step);
}

hipError_t gkv_launch_pool_scores(const GkvLaunch& ln, const GkvDims& dm, const float* F, const int32_t* d_state,
                                  int32_t step, int32_t kernel, float* F_out) {
  const int units = dm.L * dm.B * dm.Hkv;
  return gkv_launch(ln, pool_scores_kernel, dim3(units), dim3(256), sizeof(float) * dm.cap, dm, F, d_state, (int)step,
                    (int)kernel, F_out);
}

hipError_t gkv_launch_evicted_positions(const GkvLaunch& ln, const GkvDims& dm, const int32_t* keep_idx,
                                        const int32_t* pos, const int32_t* d_state, int32_t step, int32_t* evicted) {
  const int units = dm.L * dm.B * dm.Hkv;
  return gkv_launch(ln, evicted_positions_kernel, dim3(units), dim3(256), sizeof(uint32_t) * dm.cap, dm, keep_idx, pos,
                    d_state, (int)step, evicted);
}

hipError_t gkv_launch_fill_zero(hipStream_t stream, int32_t* p, size_t n) {
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

hipError_t gkv_launch_add_int(hipStream_t stream, int32_t* p, int32_t delta) {
  hipLaunchKernelGGL(add_int_kernel, dim3(1), dim3(1), 0, stream, p, delta);
  return hipGetLastError();
}
