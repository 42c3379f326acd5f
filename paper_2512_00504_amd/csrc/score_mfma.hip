// Local score of the observation window on the matrix cores: bf16 or fp32, head_dim 64 or 128,
// group size g <= 16, any window.
//
// One workgroup of NW wavefronts per (unit, key share).  The window queries of the group's heads
// are staged in LDS in blocks of 16 rows, each 1 KiB piece laid out as the matrix cores' operand
// (lane-contiguous: no bank conflicts).  A wavefront takes KT 16-key tiles of K at a time (one
// contiguous 1 KiB load per 16-byte chunk column, thanks to the tiled K layout) and computes
// logits^T[key, row] against every block of rows.
//   row statistics (max, sum of exponentials) of Eq. 1 over the keys each window row saw: under
//           the causal reading these are what the decode kernel computed when the row's query was
//           decoded, and it records them next to the window ring; they are taken from there, or,
//           when the last w decode calls were not this window's, computed by a first pass over K;
//   scores: a row's probability is 2^(z*scale*log2e - max)/sum = 2^y with the normaliser folded
//           into the exponent, y = z*scale*log2e - (max + log2 sum).  The max over the heads of a
//           group is taken on y, so there is one exponential per (window row, key) instead of one
//           per (head, window row, key); then the sum over the lanes that hold the window rows
//           (Eq. 2).  Only S leaves the chip; the [g, w, l] matrix never exists in memory.
//
// Precision of y.  scale*log2e is carried as hi + lo, and so is the offset c = max + log2 sum
// (formed in fp64 once per row): y = fma(z, hi, -c_hi) + fma(z, lo, -c_lo).  The first term is the
// small difference of two numbers of a few tens and is rounded as a small number; neither the
// scale's nor the offset's own rounding enters.  c is lowered by 3 (and the sum scaled back by 2^-3 at
// the end): probabilities between 1 and 1/64, which decide the error of S, then have |y| below 4,
// where its rounding is smallest.  Error of S against 64 bits (2-norm): 2.1e-7 at 28 layers, b = 1024,
// as with an exponential and a reciprocal per head (3.7e-7 with c lowered by 32).
//
// Blocks of rows: a window of more than 8 rows takes 16 lanes per head and 16 window rows (block =
// one head); up to 8 rows, two heads share a block.  Rows beyond the window or the group have a
// huge offset and add nothing.
#include "gkv_internal.h"

#include <type_traits>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 ld16(const void* p) { return *(const u32x4*)p; }
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

#define GKV_DPP_F(v, ctrl) __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, false))

template <typename T, int D>
struct Geo {
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr int ROW_BYTES = D * (int)sizeof(T);
  static constexpr int TILE_BYTES = 16 * ROW_BYTES;
  static constexpr int NL = ROW_BYTES / 64;      // 1 KiB operand pieces per 16 rows
  static constexpr int RP = ROW_BYTES / 16;      // 16-byte chunks per row
};

template <typename T, int D> using Tile = u32x4[Geo<T, D>::NL];

// A operand of tile t: lane (row r, kb) gets chunk 4c+kb of key 16t+r; tiled tiles are
// lane-contiguous, row-major tiles (rows appended since the last compaction) are not.
template <typename T, int D, bool ONCE = false>
__device__ __forceinline__ void load_k_tile(Tile<T, D>& kA, const char* Kh, int t, int n_tiled, int lane, int r, int kb) {
  const bool tiled = 16 * t < n_tiled;
  const char* p = Kh + (size_t)t * Geo<T, D>::TILE_BYTES + (tiled ? lane * 16 : r * Geo<T, D>::ROW_BYTES + kb * 16);
  const int step_off = tiled ? 1024 : 64;
#pragma unroll
  for (int c = 0; c < Geo<T, D>::NL; ++c)
    kA[c] = ONCE ? __builtin_nontemporal_load((const u32x4*)(p + c * step_off)) : ld16(p + c * step_off);
}

// logits[row, key] of 16 staged rows and 16 keys: lane (key = lane % 16, kb) gets rows 4 kb + e
template <typename T, int NL>
__device__ __forceinline__ f32x4 logits(const u32x4 (&q)[NL], const u32x4 (&kA)[NL]) {
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NL; ++c) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(q[c][i]), __uint_as_float(kA[c][i]), acc, 0, 0, 0);
    } else {
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(q[c]), as_bf16x8(kA[c]), acc, 0, 0, 0);
    }
  }
  return acc;
}

// One logit into a lane's running maximum m (log2 units) and sum of a row; rescaled only when some lane's
// maximum moved.  EXACT: right for every logit; without it (what is tried first, a fifth less work) logits of
// -inf and maxima of huge size may leave a wrong sum, and stats_in_doubt tells.
template <bool EXACT>
__device__ __forceinline__ void add_to_stats(float z, float s_hi, float s_lo, float& m, float& sum) {
  const float tm = rounded_product(z, s_hi);
  if (__any(tm > m)) {
    const float mnew = fmaxf(m, tm);
    sum *= __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
  }
  sum += __builtin_amdgcn_exp2f(EXACT ? log2_weight(z, s_hi, s_lo, m) : fmaf(z, s_lo, fmaf(z, s_hi, -m)));
}
__device__ __forceinline__ bool stats_in_doubt(float m, float sum) {
  return sum != sum || (fabsf(m) >= GKV_HUGE_LOG2 && m != GKV_NO_MAX);
}

// Offset of a window row with maximum m (log2 units) and sum s, as hi + lo; a row that is not there has a
// huge negative one.  Rows with a huge maximum keep it as it is in hi, for log2_score<true>.
__device__ __forceinline__ float2 row_offset(bool valid, float m, float s) {
  if (!valid) return make_float2(-INFINITY, 0.f);
  const double l = log2((double)s);
  if (fabsf(m) >= GKV_HUGE_LOG2) return make_float2(-m, (float)(3.0 - l));
  const double off = 3.0 - ((double)m + l);
  const float hi = (float)off;
  return make_float2(hi, (float)(off - (double)hi));
}
// Whether an offset may be that of a row with a huge maximum.
__device__ __forceinline__ bool huge_offset(float hi) { return fabsf(hi) >= GKV_HUGE_LOG2 && hi != -INFINITY; }

// y of a logit.  HUGE_ROWS: some row of the workgroup has a huge maximum, and all of them round the
// product as such a row's maximum and sum were formed (1e-6 less exact for the others).
template <bool HUGE_ROWS>
__device__ __forceinline__ float log2_score(float z, float s_hi, float s_lo, float c_hi, float c_lo) {
  if constexpr (HUGE_ROWS) return (rounded_product(z, s_hi) + c_hi) + c_lo;
  return fmaf(z, s_hi, c_hi) + fmaf(z, s_lo, c_lo);
}

// How a launch is cut (host): heads per block, blocks per 16 window rows, 16-row window blocks in
// all and per staging pass, key shares per unit, bytes of the LDS regions.
struct ScorePlan {
  int32_t pair_heads;      // 1: window of at most 8 rows, two heads per block
  int32_t n_blk, nt, nt_pass, ksplit;
  int32_t use_sbuf;        // S is collected in LDS over several passes
  GkvDivisor by_ksplit;
};

// Dynamic LDS: q pieces [nt_pass*n_blk][NL][1 KiB]; float row_hi[rows], row_lo[rows]; float sbuf[cap] if
// use_sbuf; and, when the row statistics are computed here, float2 red_ms[NW][rows].
// HAVE_STATS: a.stats holds (max, sum) of every window row, recorded by the decode kernel.
template <typename T, int D, int NW, int KT, bool HAVE_STATS>
__global__ __launch_bounds__(NW * 64) void score_mfma_kernel(GkvDims dm, ScoreArgs a, ScorePlan pl) {
  using G = Geo<T, D>;
  constexpr int NL = G::NL;
  a.step = resolve_step(dm, a.step);
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kb = lane >> 4;
  const int unit = quotient(blockIdx.x, pl.by_ksplit), share = (int)blockIdx.x - unit * pl.ksplit;
  const int lb = quotient(unit, dm.by_hkv), j = unit - lb * dm.Hkv;
  const int cap = dm.cap, w = dm.w, g = dm.g;
  const bool pair = pl.pair_heads;

  const int rows_pass = pl.nt_pass * pl.n_blk * 16;
  char* qs = smem_raw;
  float* row_hi = (float*)(qs + (size_t)rows_pass * G::ROW_BYTES);
  float* row_lo = row_hi + rows_pass;
  float* sbuf = row_lo + rows_pass;
  float2* red_ms = (float2*)(sbuf + (pl.use_sbuf ? cap : 0));

  // The window queries of a pass go straight to LDS, piece by piece (wavefront `wave` fetches pieces wave, wave + NW, ...): a
  // lane's window row is the same in all blocks of sixteen rows, their heads follow each other in memory.  Rows beyond the
  // window or the group repeat a valid one; their offset drops them.  Nothing here waits for the state record.  (With
  // each 16-byte piece's row worked out for itself, behind the record, and the first statistics and key tiles behind the queries, us
  // in a graph, before -> now: fp32, D = 128, g = 7 4 units of 612 rows 13.0 -> 9.5, 32 of 544 17.2 -> 14.1, 256 47.3 -> 43.7; D = 64, g = 4 2 of 80
  // 5.3 -> 4.95; bf16, g = 16 64 of 576 17.7 -> 11.7, 896 of 576 68.5 -> 55.4; with own statistics 32 of 544 147 -> 137.)
  const int t_first = a.step - w + 1;
  int slot0 = t_first % w;
  slot0 = slot0 < 0 ? slot0 + w : slot0;                 // slot of window row 0; row k sits in slot0 + k, wrapped
  auto ring_row = [&](int h, int k) {
    int slot = slot0 + k;
    slot = slot >= w ? slot - w : slot;
    return ((size_t)slot * dm.L * dm.B + lb) * dm.Hq + j * g + h;
  };
  auto fetch_queries = [&](int nt0, int nts) {
    for (int nt = 0; nt < nts; ++nt) {
      const int k = min(pair ? (r & 7) : 16 * (nt0 + nt) + r, w - 1);
      const char* row = (const char*)a.qwin + ring_row(0, k) * G::ROW_BYTES + kb * 16;
      for (int x = wave; x < pl.n_blk * NL; x += NW) {
        const int i = x / NL, c = x % NL;
        const int h = min(pair ? 2 * i + (r >> 3) : i, g - 1);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(row + h * G::ROW_BYTES + c * 64),
                                         (__attribute__((address_space(3))) void*)(qs + (size_t)(nt * pl.n_blk * NL + x) * 1024), 16, 0, 0);
      }
    }
  };
  fetch_queries(0, min(pl.nt_pass, pl.nt));
  // head and window row (k-th oldest) of staged row x of the pass that starts at nt0
  auto head_of = [&](int x) { return pair ? 2 * (x >> 4) + ((x >> 3) & 1) : (x >> 4) % pl.n_blk; };
  auto k_of = [&](int x, int nt0) { return pair ? (x & 7) : 16 * (nt0 + (x >> 4) / pl.n_blk) + (x & 15); };
  auto stats_of = [&](int x, int nt0) { return a.stats[ring_row(min(head_of(x), g - 1), min(k_of(x, nt0), w - 1))]; };
  float2 first_stats = make_float2(0.f, 1.f);
  if constexpr (HAVE_STATS) first_stats = stats_of(min(tid, rows_pass - 1), 0);

  const SeqState seq = load_state(a.d_state, lb);
  const int l = compression_length(seq, a.step, dm.b, w, cap);
  const int cc = l - w;                     // number of candidates

  const char* Kh = (const char*)a.K + (size_t)unit * cap * G::ROW_BYTES;
  const float s_hi = dm.scale_l2_hi, s_lo = dm.scale_l2_lo;
  float* So = a.S + (size_t)unit * cap;

  // this workgroup's groups of KT candidate tiles
  const int groups = l == 0 ? 0 : (((cc + 15) >> 4) + KT - 1) / KT;
  const int per_share = (groups + pl.ksplit - 1) / pl.ksplit;
  const int g0 = share * per_share, g1 = min(groups, g0 + per_share);
  if (g0 >= g1) {                           // (where there is a compression, cc > 0 and share 0 has work)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    return;
  }

  const int n_pass = (pl.nt + pl.nt_pass - 1) / pl.nt_pass;
  for (int pass = 0; pass < n_pass; ++pass) {
    const int nt0 = pass * pl.nt_pass, nts = min(pl.nt_pass, pl.nt - nt0);
    const int rows = nts * pl.n_blk * 16;
    if (pass) {
      __syncthreads();                      // the previous pass has been read
      fetch_queries(nt0, nts);
    }
    u32x4 kA[KT][NL], kN[KT][NL];
    auto load_group = [&](u32x4 (&k)[KT][NL], int p) {
#pragma unroll
      for (int tt = 0; tt < KT; ++tt) load_k_tile<T, D>(k[tt], Kh, p * KT + tt, seq.n_tiled, lane, r, kb);
    };
    if (HAVE_STATS && g0 + wave < g1) load_group(kA, g0 + wave);
    auto store_offset = [&](int x, float m, float s) {
      const float2 c = row_offset(head_of(x) < g && k_of(x, nt0) < w, m, s);
      row_hi[x] = c.x;
      row_lo[x] = c.y;
    };
    if constexpr (HAVE_STATS) {
      for (int x = tid; x < rows; x += NW * 64) {
        const float2 ms = pass == 0 && x == tid ? first_stats : stats_of(x, nt0);
        store_offset(x, ms.x, ms.y);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // the queries are in LDS
    __syncthreads();

    auto load_q = [&](u32x4 (&q)[NL], int blk) {
#pragma unroll
      for (int c = 0; c < NL; ++c) q[c] = *(const u32x4*)(qs + (size_t)blk * G::TILE_BYTES + c * 1024 + lane * 16);
    };

    if constexpr (!HAVE_STATS) {
      // ---- first pass over K: row max and row sum over the keys visible to each window row -----
      // NB blocks at a time keep their running (max, sum) in registers; only the last tiles (those
      // reaching into the window) need the causal mask.
      constexpr int NB = 4;
      const int n_tiles = (l + 15) >> 4, n_full = (cc + 1) >> 4;   // the first n_full: every row sees all of their keys
      const int n_blocks = nts * pl.n_blk;
      for (int b0 = 0; b0 < n_blocks; b0 += NB) {
        float rm[NB][4], rs[NB][4];                            // this lane's keys of rows 4 kb + e
        int last_vis[NB][4];                                   // row k sees keys [0, cc + k]
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            rm[i][e] = GKV_NO_MAX; rs[i][e] = 0.f;
            last_vis[i][e] = cc + k_of(16 * min(b0 + i, n_blocks - 1) + 4 * kb + e, nt0);
          }
        auto stats_tile = [&](const u32x4 (&kA)[NL], int t, auto exact) {
          constexpr bool EXACT = decltype(exact)::value;
          const int key = 16 * t + r;
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            u32x4 q[NL];
            load_q(q, min(b0 + i, n_blocks - 1));
            f32x4 z = logits<T, NL>(q, kA);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              // a key the row did not see has the logit -inf: it never becomes the maximum and adds 0
              if (EXACT && key > last_vis[i][e]) z[e] = -INFINITY;
              add_to_stats<EXACT>(z[e], s_hi, s_lo, rm[i][e], rs[i][e]);
            }
          }
        };
        auto exact_tiles = [&](int t0) {
          for (int t = t0; t < n_tiles; t += NW) {
            u32x4 kA[NL];
            load_k_tile<T, D>(kA, Kh, t, seq.n_tiled, lane, r, kb);
            stats_tile(kA, t, std::true_type{});
          }
        };
        int t = wave;
        for (; t < n_full; t += NW) {
          u32x4 kA[NL];
          load_k_tile<T, D>(kA, Kh, t, seq.n_tiled, lane, r, kb);
          stats_tile(kA, t, std::false_type{});
        }
        bool again = false;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) again |= stats_in_doubt(rm[i][e], rs[i][e]);
        if (__any(again)) {
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) { rm[i][e] = GKV_NO_MAX; rs[i][e] = 0.f; }
          t = wave;
        }
        exact_tiles(t);
        // the 16 lanes of a row, then (below) the wavefronts
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float m = rm[i][e];
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
            float sum = rs[i][e] * __builtin_amdgcn_exp2f(rm[i][e] - m);
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) sum += __shfl_xor(sum, o);
            if (r == 0 && b0 + i < n_blocks) red_ms[wave * rows_pass + 16 * (b0 + i) + 4 * kb + e] = make_float2(m, sum);
          }
      }
      __syncthreads();
      for (int x = tid; x < rows; x += NW * 64) {
        float M = red_ms[x].x;
#pragma unroll
        for (int wv = 1; wv < NW; ++wv) M = fmaxf(M, red_ms[wv * rows_pass + x].x);
        float Z = 0.f;
#pragma unroll
        for (int wv = 0; wv < NW; ++wv) {
          const float2 ms = red_ms[wv * rows_pass + x];
          Z += ms.y * __builtin_amdgcn_exp2f(ms.x - M);
        }
        store_offset(x, M, Z);
      }
      __syncthreads();
    }

    // ---- scores of this share's candidates ------------------------------------------------------
    const float mean = 0x1p-3f / (float)w;
    // S of tile t from this lane's sum over its window rows
    auto finish = [&](float tot, int t) {
      float sv = tot + __shfl_xor(tot, 16);
      if (!pair) sv += __shfl_xor(sv, 32);
      const int key = 16 * t + r;
      if (kb == 0 && key < cc) {
        sv *= mean;
        if (pass) sv += sbuf[key];                             // this lane's own value of the pass before
        if (pl.use_sbuf) sbuf[key] = sv;
        if (pass == n_pass - 1) So[key] = sv;
      }
    };
    bool huge = false;
    for (int x = lane; x < rows; x += 64) huge |= huge_offset(row_hi[x]);
    if (__any(huge)) {
      // seldom: a tile at a time, by the wavefront that has it in the other passes too
      for (int t = (g0 + wave) * KT; t < g1 * KT; t = t % KT == KT - 1 ? t + (NW - 1) * KT + 1 : t + 1) {
        u32x4 kT[NL];
        load_k_tile<T, D>(kT, Kh, t, seq.n_tiled, lane, r, kb);
        float tot = 0.f;
#pragma unroll 1
        for (int nt = 0; nt < nts; ++nt) {
          f32x4 ymax = {-1e30f, -1e30f, -1e30f, -1e30f};
#pragma unroll 1
          for (int blk = nt * pl.n_blk; blk < (nt + 1) * pl.n_blk; ++blk) {
            u32x4 q[NL];
            load_q(q, blk);
            const f32x4 z = logits<T, NL>(q, kT);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int x = blk * 16 + 4 * kb + e;
              ymax[e] = fmaxf(ymax[e], log2_score<true>(z[e], s_hi, s_lo, row_hi[x], row_lo[x]));
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) tot += __builtin_amdgcn_exp2f(pair ? fmaxf(ymax[e], __shfl_xor(ymax[e], 32)) : ymax[e]);
        }
        finish(tot, t);
      }
      continue;
    }
    if (!HAVE_STATS && g0 + wave < g1) load_group(kA, g0 + wave);
    for (int p = g0 + wave; p < g1; p += NW) {
      // the wavefront's next tiles are requested before these are worked on (clamped at the end:
      // the same number of requests in flight on every path keeps the wait for this group short)
      load_group(kN, min(p + NW, g1 - 1));
      float tot[KT];
#pragma unroll
      for (int tt = 0; tt < KT; ++tt) tot[tt] = 0.f;
      for (int nt = 0; nt < nts; ++nt) {
        f32x4 ymax[KT];
#pragma unroll
        for (int tt = 0; tt < KT; ++tt) ymax[tt] = f32x4{-1e30f, -1e30f, -1e30f, -1e30f};
        for (int blk = nt * pl.n_blk; blk < (nt + 1) * pl.n_blk; ++blk) {
          u32x4 q[NL];
          load_q(q, blk);
          const f32x4 c_hi = *(const f32x4*)(row_hi + blk * 16 + 4 * kb);
          const f32x4 c_lo = *(const f32x4*)(row_lo + blk * 16 + 4 * kb);
#pragma unroll
          for (int tt = 0; tt < KT; ++tt) {
            // candidates are visible to every window row; keys >= cc are discarded below
            const f32x4 z = logits<T, NL>(q, kA[tt]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              ymax[tt][e] = fmaxf(ymax[tt][e], log2_score<false>(z[e], s_hi, s_lo, c_hi[e], c_lo[e]));
          }
        }
#pragma unroll
        for (int tt = 0; tt < KT; ++tt) {
          if (pair) {                                            // rows 8 .. 15 are the block's other head
#pragma unroll
            for (int e = 0; e < 4; ++e) ymax[tt][e] = fmaxf(ymax[tt][e], __shfl_xor(ymax[tt][e], 32));
          }
          tot[tt] += (__builtin_amdgcn_exp2f(ymax[tt][0]) + __builtin_amdgcn_exp2f(ymax[tt][1])) +
                     (__builtin_amdgcn_exp2f(ymax[tt][2]) + __builtin_amdgcn_exp2f(ymax[tt][3]));
        }
      }
#pragma unroll
      for (int tt = 0; tt < KT; ++tt) finish(tot[tt], p * KT + tt);
#pragma unroll
      for (int tt = 0; tt < KT; ++tt)
#pragma unroll
        for (int c = 0; c < NL; ++c) kA[tt][c] = kN[tt][c];
    }
  }
}

// The common case: bf16 and so few blocks of window rows (NT sixteens of NB) that a wavefront can hold all
// of their operands in registers; OWN computes the rows' statistics first.  The kernel above reads 1 KiB of
// LDS per MFMA at one key tile per wavefront, which makes the CU's 128 B a cycle its bound; here LDS
// only hands the queries round once.  K^T Q instead of Q^T K: a lane keeps one row's offset per
// block (two registers, not eight), and the 16 window rows end up across the lanes.
// Bound: HBM at several hundred units (28 layers, batch 16, b = 1024: 516 MB of K in 98 to 114 us, with two tiles in
// turn instead of three 115 to 124 and then 97 with one block's arithmetic left of seven), arithmetic and the start
// of a workgroup (state, queries, first tile: three dependent trips to memory) below.  Per launch
// against a kernel that kept the queries in LDS and took an exponential per head and logit: 256 units
// of 1088 rows, g = 5, w = 32 25.8 -> 20.0 us; 4608 such units 347 -> 310 us; 448 units of 640 rows,
// g = 7, w = 16 20.8 -> 17.8 us; 4 units 11.1 -> 5.8 us.  Against the plain kernel: bf16 D = 64, 128 units
// 2780 -> 7.4 us; fp32 D = 128, 32 units 3495 -> 14.1 us (kernel above, bound by fp32 MFMAs).
// Dynamic LDS: q pieces [NT*NB][NL][1 KiB]; float2 row_c[16*NT*NB]; OWN: float2 red_ms[NW][16*NT*NB].
template <int D, int NW, int NB, int NT, bool ONCE, bool OWN>
__global__ __launch_bounds__(NW * 64, 2) void score_regs_kernel(GkvDims dm, ScoreArgs a, int pair, int ksplit, GkvDivisor by_ksplit) {
  using T = uint16_t;
  using G = Geo<T, D>;
  constexpr int NL = G::NL;
  a.step = resolve_step(dm, a.step);
  extern __shared__ __attribute__((aligned(16))) char qs[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, kb = lane >> 4;
  const int unit = quotient(blockIdx.x, by_ksplit), share = (int)blockIdx.x - unit * ksplit;
  const int lb = quotient(unit, dm.by_hkv), j = unit - lb * dm.Hkv;
  const int cap = dm.cap, w = dm.w, g = dm.g;
  float2* row_c = (float2*)(qs + (size_t)NT * NB * G::TILE_BYTES);

  // Requests that do not depend on the state record go out first: the queries, straight to LDS
  // (wavefront `wave` fetches pieces wave, wave + NW, ...; rows beyond the window or the group repeat
  // a valid one, their offset drops them), and the statistics, one row per thread.
  auto row_src = [&](int nt, int i, int row, int& h, int& k) {
    h = pair ? 2 * i + (row >> 3) : i;
    k = pair ? (row & 7) : 16 * nt + row;
    const bool valid = h < g && k < w;
    h = min(h, g - 1); k = min(k, w - 1);
    return valid;
  };
  const int t_first = a.step - w + 1;
  int slot0 = t_first % w;
  slot0 = slot0 < 0 ? slot0 + w : slot0;                 // slot of window row 0; row k sits in slot0 + k, wrapped
  auto ring_row = [&](int h, int k) {
    int slot = slot0 + k;
    slot = slot >= w ? slot - w : slot;
    return ((size_t)slot * dm.L * dm.B + lb) * dm.Hq + j * g + h;
  };
  for (int x = wave; x < NT * NB * NL; x += NW) {
    const int blk = x / NL, c = x % NL;
    int h, k;
    row_src(blk / NB, blk % NB, r, h, k);
    const char* src = (const char*)a.qwin + ring_row(h, k) * G::ROW_BYTES + (4 * c + kb) * 16;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(qs + x * 1024), 16, 0, 0);
  }
  static_assert(NT * NB * 16 <= NW * 64, "a row per thread");
  float2 ms = make_float2(0.f, 1.f);
  bool row_valid = false;
  if (tid < NT * NB * 16) {
    int h, k;
    row_valid = row_src((tid >> 4) / NB, (tid >> 4) % NB, tid & 15, h, k);
    if constexpr (!OWN) ms = a.stats[ring_row(h, k)];
  }

  const SeqState seq = load_state(a.d_state, lb);
  const int l = compression_length(seq, a.step, dm.b, w, cap);
  const int cc = l - w;                     // number of candidates
  const int tiles = l == 0 ? 0 : (cc + 15) >> 4;
  const int per_share = (tiles + ksplit - 1) / ksplit;
  const int g0 = share * per_share, g1 = min(tiles, g0 + per_share);
  const char* Kh = (const char*)a.K + (size_t)unit * cap * G::ROW_BYTES;
  // Two tiles on their way while a third is worked on where K comes from memory and the registers allow it: 1792
  // units of 1152 rows, g = 7 124 -> 114 us, g = 8 117 -> 103, g = 4 100 -> 97; K within the memory-side cache 30.3 -> 29.7
  // (896 units), 64 units 6.7 -> 7.0; ten blocks of 128 bytes 72 -> 79.  A fourth: 115, 114, 99.
  // The tiles are an array (as two objects 672 units of 309 rows, g = 8 take 19.0 us instead of 18.2, three cost 1 per cent), but two
  // objects where the rows' own statistics come first: with the array that pass took 8 to 34 registers more, and 38
  // spilled took 18432 units, g = 5, w = 32 from 2480 to 4530 us.
  constexpr int DEPTH = ONCE && NT * NB <= 8 ? 3 : 2;
  Tile<T, D> kA, kN, ring[DEPTH];
  const int n_full = OWN ? (cc + 1) >> 4 : 0;            // tiles whose keys every window row sees
  if constexpr (OWN) {
    if (wave < n_full) load_k_tile<T, D>(kA, Kh, wave, seq.n_tiled, lane, r, kb);
  } else {
    if (g0 + wave < g1) load_k_tile<T, D, ONCE>(ring[0], Kh, g0 + wave, seq.n_tiled, lane, r, kb);
    if (tid < NT * NB * 16) row_c[tid] = row_offset(row_valid, ms.x, ms.y);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the queries are in LDS
  __syncthreads();
  if (g0 >= g1) return;
  const float s_hi = dm.scale_l2_hi, s_lo = dm.scale_l2_lo;
  u32x4 q[NT * NB][NL];
  auto load_q = [&](u32x4 (&x)[NL], int b) {
#pragma unroll
    for (int c = 0; c < NL; ++c) x[c] = *(const u32x4*)(qs + (b * NL + c) * 1024 + lane * 16);
  };
  // ten blocks of 16 x 256 bytes and the first pass of OWN need more registers than there are: it takes two of them from LDS each time
  constexpr int HELD = OWN && NL == 4 && NT * NB > 8 ? 8 : NT * NB;
#pragma unroll
  for (int b = 0; b < HELD; ++b) load_q(q[b], b);

  if constexpr (OWN) {
    // ---- the rows' own statistics: a first pass over all keys, a row's (max, sum) in four lanes --------
    float rm[NT * NB], rs[NT * NB];
    auto reset = [&]() {
#pragma unroll
      for (int b = 0; b < NT * NB; ++b) { rm[b] = GKV_NO_MAX; rs[b] = 0.f; }
    };
    auto stats_tile = [&](const Tile<T, D>& kT, int t, auto exact) {
      constexpr bool EXACT = decltype(exact)::value;
#pragma unroll
      for (int b = 0; b < NT * NB; ++b) {
        if (b >= HELD) {
          asm volatile("" ::: "memory");                 // read here, not once before the loop
          load_q(q[b], b);
        }
        f32x4 z = logits<T, NL>(kT, q[b]);
        if constexpr (EXACT) {
          // a key the row did not see has the logit -inf: it never becomes the maximum and adds 0
          const int seen = cc + (pair ? (r & 7) : 16 * (b / NB) + r);
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (16 * t + 4 * kb + e > seen) z[e] = -INFINITY;
        }
        const float tm = rounded_product(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])), s_hi);
        if (__any(tm > rm[b])) {
          const float mnew = fmaxf(rm[b], tm);
          rs[b] *= __builtin_amdgcn_exp2f(rm[b] - mnew);
          rm[b] = mnew;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          rs[b] += __builtin_amdgcn_exp2f(EXACT ? log2_weight(z[e], s_hi, s_lo, rm[b])
                                                : fmaf(z[e], s_lo, fmaf(z[e], s_hi, -rm[b])));
      }
    };
    const int n_tiles = (l + 15) >> 4;
    auto exact_tiles = [&](int t0) {
      for (int t = t0; t < n_tiles; t += NW) {
        Tile<T, D> kT;
        load_k_tile<T, D>(kT, Kh, t, seq.n_tiled, lane, r, kb);
        stats_tile(kT, t, std::true_type{});
      }
    };
    reset();
    for (int t = wave; t < n_full; t += 2 * NW) {
      load_k_tile<T, D>(kN, Kh, min(t + NW, n_full - 1), seq.n_tiled, lane, r, kb);
      stats_tile(kA, t, std::false_type{});
      if (t + NW >= n_full) break;
      load_k_tile<T, D>(kA, Kh, min(t + 2 * NW, n_full - 1), seq.n_tiled, lane, r, kb);
      stats_tile(kN, t + NW, std::false_type{});
    }
    bool again = false;
#pragma unroll
    for (int b = 0; b < NT * NB; ++b) again |= stats_in_doubt(rm[b], rs[b]);
    if (__any(again)) reset();
    exact_tiles(__any(again) ? wave : n_full + (wave + NW - n_full % NW) % NW);
    if (g0 + wave < g1) load_k_tile<T, D>(kA, Kh, g0 + wave, seq.n_tiled, lane, r, kb);
    float2* red_ms = row_c + NT * NB * 16;               // [NW][rows]
#pragma unroll
    for (int b = 0; b < NT * NB; ++b) {
      float m = fmaxf(rm[b], __shfl_xor(rm[b], 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      float sum = rs[b] * __builtin_amdgcn_exp2f(rm[b] - m);
      sum += __shfl_xor(sum, 16);
      sum += __shfl_xor(sum, 32);
      if (kb == 0) red_ms[wave * (NT * NB * 16) + 16 * b + r] = make_float2(m, sum);
    }
    __syncthreads();
    if (tid < NT * NB * 16) {
      float M = GKV_NO_MAX, Z = 0.f;
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) M = fmaxf(M, red_ms[wv * (NT * NB * 16) + tid].x);
#pragma unroll
      for (int wv = 0; wv < NW; ++wv) {
        const float2 part = red_ms[wv * (NT * NB * 16) + tid];
        Z += part.y * __builtin_amdgcn_exp2f(part.x - M);
      }
      row_c[tid] = row_offset(row_valid, M, Z);
    }
#pragma unroll
    for (int b = HELD; b < NT * NB; ++b) load_q(q[b], b);
    __syncthreads();
  }
  const float mean = 0x1p-3f / (float)w;
  float* So = a.S + (size_t)unit * cap;
  // S of tile t from tot[e], the sum over the sixteens of window rows of row r's probability of key 4 kb + e
  auto finish = [&](const f32x4& tot, int t) {
    // Sum of tot[e] over the 16 lanes of a quarter (over 8 of them with two heads in a block: both
    // halves hold the same then): two exchange-and-add steps leave value e = r % 4 of a quad in each
    // lane, rotations by 4 and 8 add the quads.
    const bool odd = r & 1, upper = r & 2;
    float p01 = odd ? tot[1] : tot[0], x01 = odd ? tot[0] : tot[1];
    float p23 = odd ? tot[3] : tot[2], x23 = odd ? tot[2] : tot[3];
    p01 += GKV_DPP_F(x01, 0xB1);                           // quad_perm [1,0,3,2]
    p23 += GKV_DPP_F(x23, 0xB1);
    float sv = upper ? p23 : p01, xs = upper ? p01 : p23;
    sv += GKV_DPP_F(xs, 0x4E);                             // quad_perm [2,3,0,1]
    sv += GKV_DPP_F(sv, 0x124);                            // row_ror:4
    if (!pair) sv += GKV_DPP_F(sv, 0x128);                 // row_ror:8
    const int key = 16 * t + 4 * kb + r;
    if (r < 4 && key < cc) So[key] = sv * mean;
  };
  float c_hi[NT * NB], c_lo[NT * NB];
#pragma unroll
  for (int b = 0; b < NT * NB; ++b) {
    const float2 c = row_c[16 * b + r];
    c_hi[b] = c.x; c_lo[b] = c.y;
  }
  auto tile = [&](const Tile<T, D>& kT, int t) {
    f32x4 tot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      f32x4 ymax = {-1e30f, -1e30f, -1e30f, -1e30f};
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int b = nt * NB + i;
        const f32x4 z = logits<T, NL>(kT, q[b]);           // lane (row r, kb): keys 4 kb + e
#pragma unroll
        for (int e = 0; e < 4; ++e)
          ymax[e] = fmaxf(ymax[e], log2_score<false>(z[e], s_hi, s_lo, c_hi[b], c_lo[b]));
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float y = ymax[e];
        if (pair) y = fmaxf(y, GKV_DPP_F(y, 0x128));       // row_ror:8: the block's other head
        tot[e] += __builtin_amdgcn_exp2f(y);
      }
    }
    finish(tot, t);
  };
  // the tiles in turn: the next ones are always requested before one is worked on, and stay where they land
  // (copied over at the end of each round instead: 121 -> 117 us at 1792 units of b = 1024)
  auto request = [&](Tile<T, D>& kT, int t) { load_k_tile<T, D, ONCE>(kT, Kh, min(t, g1 - 1), seq.n_tiled, lane, r, kb); };
  if constexpr (OWN) {
    for (int t = g0 + wave; t < g1; t += 2 * NW) {
      request(kN, t + NW);
      tile(kA, t);
      if (t + NW >= g1) break;
      request(kA, t + 2 * NW);
      tile(kN, t + NW);
    }
  } else {
#pragma unroll
    for (int p = 1; p < DEPTH - 1; ++p) request(ring[p], g0 + wave + p * NW);
    for (int t = g0 + wave; t < g1; t += DEPTH * NW) {
#pragma unroll
      for (int p = 0; p < DEPTH; ++p) {
        if (p > 0 && t + p * NW >= g1) break;
        request(ring[(p + DEPTH - 1) % DEPTH], t + (p + DEPTH - 1) * NW);
        tile(ring[p], t + p * NW);
      }
    }
  }
  bool huge = false;
#pragma unroll
  for (int x = 0; x < NT * NB * 16; x += 64) huge |= huge_offset(row_c[min(x + lane, NT * NB * 16 - 1)].x);
  if (__any(huge)) {
    // seldom: block by block from LDS, a tile at a time, over what the loop above stored
    for (int t = g0 + wave; t < g1; t += NW) {
      Tile<T, D> kT;
      load_k_tile<T, D>(kT, Kh, t, seq.n_tiled, lane, r, kb);
      f32x4 tot = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int nt = 0; nt < NT; ++nt) {
        f32x4 ymax = {-1e30f, -1e30f, -1e30f, -1e30f};
#pragma unroll 1
        for (int b = nt * NB; b < (nt + 1) * NB; ++b) {
          u32x4 qb[NL];
          load_q(qb, b);
          const float2 c = row_c[16 * b + r];
          const f32x4 z = logits<T, NL>(kT, qb);
#pragma unroll
          for (int e = 0; e < 4; ++e) ymax[e] = fmaxf(ymax[e], log2_score<true>(z[e], s_hi, s_lo, c.x, c.y));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
          tot[e] += __builtin_amdgcn_exp2f(pair ? fmaxf(ymax[e], GKV_DPP_F(ymax[e], 0x128)) : ymax[e]);
      }
      finish(tot, t);
    }
  }
}

// Own statistics: every workgroup goes through all of its unit's keys first, so units are shared out only
// while there are fewer than compute units, and 8 wavefronts share that pass.  us per launch, the kernel
// above (4 wavefronts, a sweep over K per four blocks) -> this one: 4 units of 640 rows, g = 7, w = 16 40 -> 13; of
// 2176 rows, g = 8 91 -> 32; 256 of 1088, g = 5, w = 32 127 -> 38; 896 of 640, g = 7, w = 16 122 -> 73; 18432 of 1088,
// g = 5, w = 32 4670 -> 2480.  Bound: the arithmetic of two passes (the second alone, with recorded statistics:
// 38 us at 896 units).
template <int D, int NB, int NT>
hipError_t launch_regs_own(const GkvLaunch& ln, const GkvDims& dm, const ScoreArgs& a, int len_max, bool pair) {
  constexpr int NW = 8, ROWS = NT * NB * 16;
  const int units = dm.L * dm.B * dm.Hkv;
  const int tiles = (len_max + 15) / 16, most = (tiles + NW - 1) / NW;
  int ksplit = 256 / units;
  ksplit = ksplit < 1 ? 1 : (ksplit > most ? (most < 1 ? 1 : most) : ksplit);
  return gkv_launch(ln, score_regs_kernel<D, NW, NB, NT, false, true>, dim3(units * ksplit), dim3(NW * 64),
                    (size_t)ROWS * (Geo<uint16_t, D>::ROW_BYTES + 8 + 8 * NW), dm, a, (int)pair, ksplit, gkv_divisor(ksplit));
}

template <int D, int NB, int NT>
hipError_t launch_regs(const GkvLaunch& ln, const GkvDims& dm, const ScoreArgs& a, int len_max, bool pair) {
  if (!a.stats) return launch_regs_own<D, NB, NT>(ln, dm, a, len_max, pair);
  constexpr int NW = 4;
  const int units = dm.L * dm.B * dm.Hkv;
  // Two workgroups of 4 wavefronts fit a CU at these register counts: fewer than 512 units are cut into
  // key shares, down to one tile per wavefront (4 units of 640 rows: 11.0 us whole, 5.8 us in shares; 256 of
  // 1088 21.6 / 20.0).
  const int tiles = (len_max + 15) / 16, most = (tiles + NW - 1) / NW;
  int ksplit = 512 / units;
  ksplit = ksplit < 1 ? 1 : (ksplit > most ? (most < 1 ? 1 : most) : ksplit);
  // K beyond the 256 MiB memory-side cache is read with non-temporal loads: right after a decode step
  // 80 -> 67 us at 280 MB of K (1792 units), 134 -> 113 us at 504 MB, 305 -> 285 us at 1.2 GB; at 70 and
  // 140 MB there is no difference then, and a second reader of the same K finds it cached.
  const bool once = (size_t)units * len_max * Geo<uint16_t, D>::ROW_BYTES > (size_t)256 << 20;
  auto kern = once ? score_regs_kernel<D, NW, NB, NT, true, false> : score_regs_kernel<D, NW, NB, NT, false, false>;
  return gkv_launch(ln, kern, dim3(units * ksplit), dim3(NW * 64),
                    (size_t)NT * NB * (Geo<uint16_t, D>::TILE_BYTES + 128), dm, a, (int)pair, ksplit, gkv_divisor(ksplit));
}

// false: no such instantiation
template <int D>
bool try_launch_regs(const GkvLaunch& ln, const GkvDims& dm, const ScoreArgs& a, int len_max, hipError_t* e) {
  const bool pair = dm.w <= 8;
  const int nb = pair ? (dm.g + 1) / 2 : dm.g, nt = pair ? 1 : (dm.w + 15) / 16;
#define GKV_CASE(NB_, NT_) if (nb == NB_ && nt == NT_) { *e = launch_regs<D, NB_, NT_>(ln, dm, a, len_max, pair); return true; }
  GKV_CASE(1, 1) GKV_CASE(2, 1) GKV_CASE(3, 1) GKV_CASE(4, 1) GKV_CASE(5, 1) GKV_CASE(6, 1) GKV_CASE(7, 1) GKV_CASE(8, 1)
  GKV_CASE(1, 2) GKV_CASE(2, 2) GKV_CASE(3, 2) GKV_CASE(4, 2) GKV_CASE(5, 2)
#undef GKV_CASE
  return false;
}

template <typename T, int D, int NW, int KT>
hipError_t launch(const GkvLaunch& ln, const GkvDims& dm, const ScoreArgs& a, int len_max) {
  using G = Geo<T, D>;
  const int units = dm.L * dm.B * dm.Hkv;
  ScorePlan pl;
  pl.pair_heads = dm.w <= 8;
  pl.n_blk = pl.pair_heads ? (dm.g + 1) / 2 : dm.g;
  pl.nt = pl.pair_heads ? 1 : (dm.w + 15) / 16;
  const int block_bytes = pl.n_blk * G::TILE_BYTES;
  pl.nt_pass = 72 * 1024 / block_bytes;
  pl.nt_pass = pl.nt_pass < 1 ? 1 : (pl.nt_pass > pl.nt ? pl.nt : pl.nt_pass);
  pl.use_sbuf = pl.nt_pass < pl.nt;
  const int groups = ((len_max + 15) / 16 + KT - 1) / KT;
  const int k = 512 / units, most = (groups + NW - 1) / NW;
  pl.ksplit = k < 1 ? 1 : (k > most ? (most < 1 ? 1 : most) : k);
  pl.by_ksplit = gkv_divisor(pl.ksplit);
  const size_t rows = (size_t)pl.nt_pass * pl.n_blk * 16;
  const size_t shmem = rows * G::ROW_BYTES + rows * 8 + (pl.use_sbuf ? 4 * (size_t)dm.cap : 0) +
                       (a.stats ? 0 : NW * rows * 8);
  auto kern = a.stats ? score_mfma_kernel<T, D, NW, KT, true> : score_mfma_kernel<T, D, NW, KT, false>;
  if (shmem > GKV_LDS_LIMIT) {                             // beyond the default per-workgroup limit: opt in (a CU holds 160 KiB)
    const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem);
    if (e != hipSuccess) return e;
  }
  return gkv_launch(ln, kern, dim3(units * pl.ksplit), dim3(NW * 64), shmem, dm, a, pl);
}

}  // namespace

hipError_t gkv_launch_score_mfma(const GkvLaunch& ln, const GkvDims& dm, int dtype, const ScoreArgs& a, int len_max) {
  if (dtype == GKV_F32)
    return dm.d == 64 ? launch<float, 64, 4, 2>(ln, dm, a, len_max) : launch<float, 128, 4, 1>(ln, dm, a, len_max);
  hipError_t e;
  if (dm.d == 64 ? try_launch_regs<64>(ln, dm, a, len_max, &e) : try_launch_regs<128>(ln, dm, a, len_max, &e)) return e;
  return dm.d == 64 ? launch<uint16_t, 64, 4, 2>(ln, dm, a, len_max) : launch<uint16_t, 128, 4, 2>(ln, dm, a, len_max);
}
