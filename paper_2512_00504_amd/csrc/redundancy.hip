// Redundancy score of the cached keys and its combination with the global score
// (paper, appendix "Integrating the Global Score with Other Methods"):
//   Kn = K / (||K|| + eps);  C = Kn Kn^T;  entries below tau, the diagonal and the columns of
//   the n_recent newest rows are zeroed;  col_j = sum_k C'_kj;  R = softmax_j(col);
//   R' = R / max_j R = exp(col_j - max_j col)   (the softmax denominator cancels);
//   F_sel = lambda * F - (1 - lambda) * R'  over the candidates.
// A workgroup per unit, or several that share its columns in launches of few units.  The l x l x d contraction runs on
// the matrix cores: in 32 bits for bf16, d = 128, in 64 bits for fp32 at d = 64 or 128 and bf16 at d = 64 (groups of at
// most 16 heads, K 16-byte aligned); a plain vector-ALU kernel covers the rest.
#include "gkv_internal.h"
#include <atomic>
#include <type_traits>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct RedArgs {
  const void* K; const int32_t* d_state; int32_t step; const float* F;
  float lambda, tau, eps; int32_t n_recent; float* R_norm; float* F_sel;
};

// Precision.  A column sum adds up to l cosines and reaches the hundreds, R' = exp(col - max col)
// is compared at 1e-5 relative, and the threshold turns each cosine into a yes/no.  The
// reciprocal norms are formed in fp64.  A column's own norm is a common factor of its whole sum,
// so it is applied once, in fp64, to the finished sum and folded into the threshold (C >= tau
// <=> dot * inv_k >= tau / inv_j); a per-entry fp32 rounding of it would be a systematic error of
// col_j * 1e-7.  What is left per entry in the matrix-core kernel is dot * inv_k in fp32 (dot:
// fp32 accumulation of exact bf16 products; inv_k: the fp64 value rounded once): its error is a
// few 1e-8 of the cosine, random from entry to entry, far inside the 1e-6 band in which a
// threshold decision may legitimately differ from fp64, and it averages out in the sums.  Sums
// run in fp32 over a lane's four entries of a tile pair and in fp64 from there on; exp(col - max)
// is fp64.  The plain kernel does everything in fp64.
// Exchanges between lanes go through registers (through LDS one takes 60 ns): sums over the lanes l and l ^ 16, l and
// l ^ 32, in both, and the maximum of a wavefront.  With these, and a row's square root and quotient (forty instructions in
// 64 bits) in one lane instead of four, us a call in a graph: fp32, d = 128 8 units of 348 rows 18.6 -> 17.3, d = 64 20 of 348 17.1 ->
// 16.2, bf16, d = 64 32 of 400 27.4 -> 25.8; bf16, d = 128 4 of 640 20.1 -> 19.5, 896 of 640 the same to 2%.
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ double add_halves(double v) {
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(u[0], u[0], false, false));
  const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(u[1], u[1], false, false));
  return __builtin_bit_cast(double, (u32x2{lo[0], hi[0]})) + __builtin_bit_cast(double, (u32x2{lo[1], hi[1]}));
}
__device__ __forceinline__ double add_quarters(double v) {
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(u[0], u[0], false, false));
  const u32x2 hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(u[1], u[1], false, false));
  return add_halves(__builtin_bit_cast(double, (u32x2{lo[0], hi[0]})) + __builtin_bit_cast(double, (u32x2{lo[1], hi[1]})));
}
__device__ __forceinline__ double wave_max_f64(double v) {
#define GKV_STEP(ctrl, rows) { \
    const u32x2 u = __builtin_bit_cast(u32x2, v); \
    const u32x2 o = u32x2{(uint32_t)__builtin_amdgcn_update_dpp((int)u[0], (int)u[0], ctrl, rows, 0xF, false), \
                          (uint32_t)__builtin_amdgcn_update_dpp((int)u[1], (int)u[1], ctrl, rows, 0xF, false)}; \
    v = fmax(v, __builtin_bit_cast(double, o)); }
  GKV_STEP(0x111, 0xF) GKV_STEP(0x112, 0xF) GKV_STEP(0x114, 0xF) GKV_STEP(0x118, 0xF)   // row_shr; lanes without a source keep their own
  GKV_STEP(0x142, 0xA) GKV_STEP(0x143, 0xC)
#undef GKV_STEP
  const u32x2 u = __builtin_bit_cast(u32x2, v);
  return __builtin_bit_cast(double, (u32x2{(uint32_t)__builtin_amdgcn_readlane((int)u[0], 63), (uint32_t)__builtin_amdgcn_readlane((int)u[1], 63)}));
}

template <int NW>
__device__ __forceinline__ double block_max_f64(double v, double* red) {
  v = wave_max_f64(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double m = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) m = fmax(m, red[i]);
  return m;
}

// Shared tail: R' from the column sums in LDS, then the combination.  cs[j] valid for j < l; `red`
// holds a double per wavefront.
template <int NW>
__device__ __forceinline__ void finish_unit(const GkvDims& dm, const RedArgs& a, int unit, int l,
                                            const double* cs, double* red) {
  const int tid = threadIdx.x;
  double mx = -1e300;
  for (int j = tid; j < l; j += NW * 64) mx = fmax(mx, cs[j]);
  mx = block_max_f64<NW>(mx, red);
  float* Ru = a.R_norm + (size_t)unit * dm.cap;
  float* Fs = a.F_sel + (size_t)unit * dm.cap;
  const float* Fu = a.F + (size_t)unit * dm.cap;
  const int c = l - dm.w;
  for (int j = tid; j < l; j += NW * 64) {
    const float rn = (float)exp(cs[j] - mx);
    Ru[j] = rn;
    if (j < c) Fs[j] = a.lambda * Fu[j] - (1.f - a.lambda) * rn;
  }
}

// Column sums [j0, j1) of a unit whose columns several workgroups share, on their way to redundancy_finish_kernel in the
// places of the results: low words in R', high words in F_sel.  The window's columns have no place in F_sel: this
// serves n_recent >= w, where their sums are 0.
__device__ __forceinline__ void store_sums(const GkvDims& dm, const RedArgs& a, int unit, int j0, int j1, const double* cs,
                                           int tid, int threads) {
  for (int j = j0 + tid; j < j1; j += threads) {
    a.R_norm[(size_t)unit * dm.cap + j] = __int_as_float(__double2loint(cs[j]));
    a.F_sel[(size_t)unit * dm.cap + j] = __int_as_float(__double2hiint(cs[j]));
  }
}

// ---- any dtype / shape ------------------------------------------------------------------------
// Dynamic LDS: double cs[cap]; double red[4]; double inv[cap]
template <typename T>
__global__ __launch_bounds__(256) void redundancy_generic_kernel(GkvDims dm, RedArgs a) {
  a.step = resolve_step(dm, a.step);
  extern __shared__ double smem[];
  constexpr int EPC = Elem<T>::EPC;
  const int tid = threadIdx.x, unit = blockIdx.x, lb = quotient(unit, dm.by_hkv), d = dm.d;
  double* cs = (double*)smem;
  double* red = cs + dm.cap;
  double* inv = red + 4;
  const SeqState st = load_state(a.d_state, lb);
  const int l = compression_length(st, a.step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const T* Kh = (const T*)a.K + (size_t)unit * dm.cap * d;
  for (int n = tid; n < l; n += 256) {
    double ss = 0.0;
    for (int ch = 0; ch < d; ++ch) {
      const double x = (double)Elem<T>::ld(Kh + k_elem_offset<EPC>(n, ch, d, st.n_tiled));
      ss = fma(x, x, ss);
    }
    inv[n] = 1.0 / (sqrt(ss) + (double)a.eps);
  }
  __syncthreads();
  const int first_recent = l - a.n_recent;
  for (int j = tid; j < l; j += 256) {
    double col = 0.0;
    if (j < first_recent) {
      for (int k = 0; k < l; ++k) {
        if (k == j) continue;
        double dot = 0.0;
        for (int ch = 0; ch < d; ++ch)
          dot = fma((double)Elem<T>::ld(Kh + k_elem_offset<EPC>(k, ch, d, st.n_tiled)),
                    (double)Elem<T>::ld(Kh + k_elem_offset<EPC>(j, ch, d, st.n_tiled)), dot);
        const double cv = dot * inv[k] * inv[j];
        if (cv >= (double)a.tau) col += cv;
      }
    }
    cs[j] = col;
  }
  __syncthreads();
  finish_unit<4>(dm, a, unit, l, cs, red);
}

// ---- bf16, d = 128, matrix cores ----------------------------------------------------------------
constexpr int ROW_BYTES = 256;
constexpr int TILE_BYTES = 16 * ROW_BYTES;

__device__ __forceinline__ void load_k_tile(u32x4 (&kA)[4], const char* Kh, int T, int n_tiled,
                                            int lane, int r, int kb) {
  const bool tiled = 16 * T < n_tiled;
  const char* p = Kh + (size_t)T * TILE_BYTES + (tiled ? lane * 16 : r * ROW_BYTES + kb * 16);
  const int step_off = tiled ? 1024 : 64;
#pragma unroll
  for (int c = 0; c < 4; ++c) kA[c] = *(const u32x4*)(p + c * step_off);
}

// MFMA 32x32x16: the A operand of a 32-key tile (lane = key + 32 * half, 8 channels) is also a valid B
// operand, so C[k, j] = sum_c mfma(A_T[c], A_J[c]) lands as lane (j = lane % 32, half): element i holds row
// k = 32 T + 8 (i / 4) + 4 half + i % 4.  The column tiles are shared out over eight wavefronts, each of
// which holds up to three in registers per pass; in each pass the workgroup walks all row tiles T together.
//
// What bounds it is how vector instructions and matrix products share a SIMD.  Measured with two
// wavefronts per SIMD: a 16x16x32 product takes 16 cycles and hides two vector instructions, with four it
// takes 27; a 32x32x16 product takes 32 and hides six, with eight 45.  An entry needs a product with the
// row's norm, a comparison and a sum, 16 of them per lane and 8 products: so the large tiles, and the
// comparison as a clamp (below).  The entries of one column tile are worked on between the products of the
// next one, and those of the last between the first products of the next row tile.
//
// Row tiles reach the wavefronts through LDS: every wavefront needs every row tile in every pass,
// and if each fetched them itself a unit's keys (l * 256 bytes) would be read 8 * passes times; the
// units resident on one XCD together exceed its L2, so those re-reads would come from memory and
// bound the kernel.  Instead the workgroup moves through the row tiles in groups of four: each
// wavefront fetches 16 rows of the next group while all work on the current group, stores them
// into the other half of a two-group ring, and one barrier per group hands the ring over.  Eight wavefronts
// instead of two workgroups of four halve the passes, and the keys that the units resident on an XCD
// send through its L2.
//
// A column's own reciprocal norm is wanted until its sum is finished, so the sums take the norms' place.
//
// Up to 128 units several workgroups share a unit's columns from a capacity of 448 rows on (14 column tiles for eight
// wavefronts; above 64 units, where there are two or three shares, from 704 on): a share costs the norms and the start again,
// and the sums a finishing launch.  us per call, a workgroup per unit -> shared: 4 units of 332
// rows 13.4 -> 15.1, of 400 16.1 -> 16.2, of 480 17.6 -> 16.6, of 640 24.6 -> 19.5, of 1128 67 -> 29; 64 of 332 13.8 -> 15.7, of 480 18.0 ->
// 17.1, of 640 25.2 -> 21.6, of 1128 68 -> 40; 110 of 544 22.7 -> 24.5, of 640 25.4 -> 27.5, of 704 30.0 -> 29.9, of 1128 69 -> 58;
// 128 of 640 25.5 -> 26.0, of 768 32.7 -> 31.5, of 1128 70 -> 57.
//
// Per launch in a graph, against 16x16 tiles, comparisons and selections, and two workgroups of four wavefronts per
// compute unit: 896 units of 640 rows 145 -> 122 us, of 332 92 -> 61, of 700 214 -> 141; 1792 of 1152 760 -> 637; 4 of 640
// 55 -> 26 (a workgroup each).  With every compute unit at it the clock falls (a product with random operands then takes 42 to 52
// of the nominal cycles, not 32), and units start together: all fetch their keys, then all multiply.
//
// Dynamic LDS: double cs[cap]; double red[8]; float inv_f[cap]; then the ring, 2 groups x 4 tiles x 8 KiB
constexpr int RED_NW = 8, RED_TILE = 32 * ROW_BYTES, RED_RING_BYTES = 2 * 4 * RED_TILE;
constexpr size_t RED_LDS_ROW = sizeof(double) + sizeof(float), RED_LDS_FIXED = sizeof(double) * RED_NW + RED_RING_BYTES;
// Everything that is compared and added up is scaled by a power of two, so that clamp(x) to [0, 1] of a difference of
// two scaled numbers is 1 or 0 (the next number above a threshold is at least 1 above it): as a modifier of the
// subtraction the clamp costs nothing, where a comparison and a selection are two instructions.  2^80 does for norms
// (eps included) of 2^-30 to 2^44: a cosine is scaled by 2^49 at least, |tau| from 2^-25 on has the spacing, and below that
// what can be counted in part is within 2^-49 of the threshold.  A unit with others has a scale of its own with the same
// properties (unit_scale): 4 units of 640 rows 21 -> 23 us, 896 122 -> 127.  Where its norms span too much for one, or a key
// is infinite or NaN, it is served by comparisons: 40 and 376 us.
constexpr double RED_SCALE = 0x1p80, RED_INV_MIN = 0x1p-44, RED_INV_MAX = 0x1p30;

// A power of two S for reciprocal norms from `least` to `most`, or 0: norms times S stay below 2^100, reciprocals times S
// below 2^126, and dots (of norms from 2^-38 to 2^60) are normal numbers of fp32.
__device__ __forceinline__ double unit_scale(double least, double most) {
  if (!(least >= 0x1p-60 && most <= 0x1p38 && most <= least * 0x1p50)) return 0.0;
  return ldexp(1.0, min(100 + ilogb(least), 125 - ilogb(most)));
}
typedef float f32x16 __attribute__((ext_vector_type(16)));

__global__ __launch_bounds__(RED_NW * 64, 2) void redundancy_mfma_kernel(GkvDims dm, RedArgs a) {
  a.step = resolve_step(dm, a.step);
  extern __shared__ double smem[];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, kb = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv);
  double* cs = (double*)smem;
  double* inv = cs;                                      // until the column's sum is finished
  double* red = cs + dm.cap;
  float* inv_f = (float*)(red + RED_NW);                      // the norms, scaled, in fp32
  char* ring = (char*)(inv_f + dm.cap);                  // (no other shared variable before these: 16-byte pieces want the alignment)
  int& s_odd = *(int*)red;
  double* s_scale = red + 1;                             // the scale and its reciprocal: not in registers through the passes
  if (tid == 0) { s_odd = 0; s_scale[0] = RED_SCALE; s_scale[1] = 1.0 / RED_SCALE; }
  const SeqState st = load_state(a.d_state, lb);
  const int l = compression_length(st, a.step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const char* Kh = (const char*)a.K + (size_t)unit * dm.cap * ROW_BYTES;
  const int n_tiles = (l + 31) >> 5;                     // of 32 keys; the capacity holds whole ones
  __syncthreads();

  // Every pass shares barriers, so all wavefronts make as many; their column tiles differ by one at most, and
  // wavefronts w and w + 4, which share a SIMD, get the odd ones from both ends.
  const int r32 = lane & 31, half = lane >> 5;
  // In a launch of few units gridDim.y workgroups share a unit's columns, and each forms the norms of all.
  const int shares = gridDim.y, share = blockIdx.y;
  const int order = wave < 4 ? 2 * wave : 2 * (wave - 4) + 1;
  struct Own { int lo, n, passes; };
  auto own_of = [&](int part, int parts) {
    const int lo = n_tiles * part / parts;
    return Own{lo, n_tiles * (part + 1) / parts - lo, ((n_tiles + parts - 1) / parts + 2) / 3};
  };
  u32x4 colA[3][8];
  auto load_columns = [&](int J0, int J1) {
#pragma unroll
    for (int cc = 0; cc < 3; ++cc) {
      if (cc > 0 && J0 + cc >= J1) break;                // (without any column one tile is computed and dropped)
      const int n = 32 * min(J0 + cc, n_tiles - 1) + r32;
      const bool tiled = n < st.n_tiled;
      const char* p = Kh + (size_t)(n >> 4) * TILE_BYTES + (tiled ? half * 256 + (n & 15) * 16 : (n & 15) * ROW_BYTES + half * 16);
      const int step_off = tiled ? 512 : 32;
#pragma unroll
      for (int c = 0; c < 8; ++c) colA[cc][c] = *(const u32x4*)(p + c * step_off);
    }
  };
  // The wavefront's 16 rows of a group, on their way to the ring (clamped past the end: fetched, stored, never
  // used), where a tile's 16-byte pieces lie in operand order.
  u32x4 nxt[4];
  auto request = [&](int G) { load_k_tile(nxt, Kh, min(RED_NW * G + wave, 2 * n_tiles - 1), st.n_tiled, lane, r, kb); };

  // Row norms in fp64, each wavefront those of its own columns, which it needs anyway: the last passes' first, so
  // that those of the first are there when it starts.
  {
    bool odd = false;
    const Own own = own_of(order, RED_NW);
    for (int p = own.passes - 1; p >= 0; --p) {
      const int J0 = own.lo + own.n * p / own.passes, J1 = own.lo + own.n * (p + 1) / own.passes;
      load_columns(J0, J1);
      if (p == 0) request(0);
#pragma unroll
      for (int cc = 0; cc < 3; ++cc) {
        if (J0 + cc >= J1) break;
        double q[4] = {0.0, 0.0, 0.0, 0.0};              // in four chains
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const double lo = (double)__uint_as_float(colA[cc][c][i] << 16), hi = (double)__uint_as_float(colA[cc][c][i] & 0xffff0000u);
            q[i] = fma(lo, lo, q[i]);
            q[i] = fma(hi, hi, q[i]);
          }
        double ss = (q[0] + q[1]) + (q[2] + q[3]);
        ss = add_halves(ss);
        const int n = 32 * (J0 + cc) + r32;
        const double x = n < l ? 1.0 / (sqrt(ss) + (double)a.eps) : 0.0;
        odd |= n < l && !(x >= RED_INV_MIN && x <= RED_INV_MAX);
        if (half == 0) { inv[n] = x; inv_f[n] = (float)(x * RED_SCALE); }
      }
    }
    if (__any(odd) && lane == 0) s_odd = 1;
  }

  const int first_recent = l - a.n_recent;
  const double tau = (double)a.tau;
  const int S_lo = n_tiles * share / shares, S_hi = n_tiles * (share + 1) / shares;   // this workgroup's column tiles
  // the sums of this workgroup's columns are in cs
  auto finish = [&]() {
    __syncthreads();
    if (shares == 1) finish_unit<RED_NW>(dm, a, unit, l, cs, red);
    else store_sums(dm, a, unit, 32 * S_lo, min(32 * S_hi, l - dm.w), cs, tid, RED_NW * 64);
  };
  __syncthreads();
  if (s_odd) {
    // seldom: the unit's own scale, from the least and the largest of its reciprocals (a NaN is neither and stays)
    double least = __builtin_inf(), most = 0.0;
    bool nan = false;
    for (int n = lane; n < l; n += 64) {
      const double x = inv[n];
      least = fmin(least, x); most = fmax(most, x); nan |= x != x;
    }
    for (int o = 32; o > 0; o >>= 1) { least = fmin(least, __shfl_xor(least, o)); most = fmax(most, __shfl_xor(most, o)); }
    const double scale = __any(nan) ? 0.0 : unit_scale(least, most);
    for (int n = tid; n < 32 * n_tiles; n += RED_NW * 64) inv_f[n] = (float)(scale > 0.0 ? inv[n] * scale : inv[n]);
    if (tid == 0) { s_scale[0] = scale; s_scale[1] = 1.0 / scale; }
    __syncthreads();
  }
  if (s_odd && s_scale[0] == 0.0) {
    // sixteen by sixteen keys at a time, by comparisons
    for (int J = 2 * S_lo + wave; J < 2 * S_hi; J += RED_NW) {
      u32x4 kj[4];
      load_k_tile(kj, Kh, J, st.n_tiled, lane, r, kb);
      const int j = 16 * J + r;
      const double inv_j = inv[j];
      const float thr = inv_j > 0.0 ? (float)(tau / inv_j) : 3e38f;
      double col = 0.0;
      for (int T = 0; T < 2 * n_tiles; ++T) {
        u32x4 kt[4];
        load_k_tile(kt, Kh, T, st.n_tiled, lane, r, kb);
        const f32x4 invk = *(const f32x4*)(inv_f + 16 * T + 4 * kb);
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c)
          z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kt[c]), __builtin_bit_cast(bf16x8, kj[c]), z, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float t = z[e] * invk[e];
          const int k = 16 * T + 4 * kb + e;
          if (t >= thr && k != j && k < l) col += (double)t;
        }
      }
      col += __shfl_xor(col, 16);
      col += __shfl_xor(col, 32);
      if (kb == 0 && j < l) cs[j] = j < first_recent ? col * inv_j : 0.0;
    }
    finish();
    return;
  }

  auto ring_store = [&](int G) {
    char* p = ring + (G & 1) * 4 * RED_TILE + (wave >> 1) * RED_TILE + (kb >> 1) * 1024 + ((kb & 1) * 32 + (wave & 1) * 16 + r) * 16;
    const bool stale = 16 * (RED_NW * G + wave) + r >= l;     // stale rows must not reach the products
#pragma unroll
    for (int c = 0; c < 4; ++c) *(u32x4*)(p + c * 2048) = stale ? u32x4{0u, 0u, 0u, 0u} : nxt[c];
  };
  auto ring_piece = [&](int T, int c) {
    return *(const u32x4*)(ring + (T & 7) * RED_TILE + c * 1024 + lane * 16);
  };

  // one pass: the row tiles against NC column tiles from J0 on
  auto pass = [&](int J0, int J_end, auto nc) {
    constexpr int NC = decltype(nc)::value;
    float thr[NC];
    double col[NC];
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      // C = dot * inv_k * inv_j >= tau  <=>  dot * inv_k >= tau / inv_j: one product per entry, the
      // column's factor applied once to the sum (columns >= l and duplicates never pass and are dropped
      // below; a duplicate's norm may have given way to its sum already: its own column must not look)
      const double inv_j = J0 + cc < J_end ? inv[32 * (J0 + cc) + r32] : 0.0;
      thr[cc] = inv_j > 0.0 ? (float)(tau * s_scale[0] / inv_j) : 3e38f;
      // the number before the threshold: "above it" stands for "at the threshold or above"
      const int bits = __float_as_int(thr[cc]);
      thr[cc] = thr[cc] == 0.f ? -1e-45f : __int_as_float(bits < 0 ? bits + 1 : bits - 1);
      col[cc] = 0.0;
    }
    // an eighth of the entries of one row tile and column tile cc
    f32x16 acc[2];
    f32x4 invk[4];                                         // of the row tile whose entries are being worked on
    float part = 0.f;
    auto eighth = [&](const f32x16& z, int c, int cc) {
      if (!(c & 1)) part = 0.f;                            // four entries of this lane, then fp64
#pragma unroll
      for (int i = 2 * c; i < 2 * c + 2; ++i) {
        const float t = rounded_product(z[i], invk[i >> 2][i & 3]);
        part = fmaf(__builtin_amdgcn_fmed3f(t - thr[cc], 0.f, 1.f), t, part);
      }
      asm volatile("" : "+v"(part));                     // here, not behind a later branch
      if (c & 1) {
        col[cc] += (double)part;
        asm volatile("" : "+v"(col[cc]));
      }
    };
    // Where the row tile is the column tile the entries with k == j are left out, by a branch of the whole
    // wavefront: a second version of the loop that tests every entry makes every workgroup fetch it (39 -> 33 us
    // at 4 units of 640 rows).
    auto drop_diagonal = [&](f32x16& z) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i >> 2) + 4 * half + (i & 3) == r32) z[i] = 0.f;
    };
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) invk[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    u32x4 row[8];
    // One row tile against the NC column tiles; u: T's parity.  The pieces of the next row tile, and the norms of
    // this one, take their predecessors' place behind the last use.
    auto row_tile = [&](int T, auto u_) {
      constexpr int u = decltype(u_)::value;
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) {
        const int at = (u * NC + cc) & 1, done = cc > 0 ? cc - 1 : NC - 1;
        if (cc == NC - 1 && u == 1 && (T & 2)) __syncthreads();   // the next group is in the ring
        if ((cc > 0 ? T : T - 1) == J0 + done) drop_diagonal(acc[at ^ 1]);
        f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, row[c]), __builtin_bit_cast(bf16x8, colA[cc][c]), z, 0, 0, 0);
          if (cc == NC - 1) row[c] = ring_piece(T + 1, c);
          eighth(acc[at ^ 1], c, done);
          if (cc == 0 && (c & 1)) invk[c >> 1] = *(const f32x4*)(inv_f + 32 * T + 8 * (c >> 1) + 4 * half);
          __builtin_amdgcn_sched_barrier(0);             // in this order: vector instructions between the products
        }
        acc[at] = z;
      }
    };

    // Group G + 1 goes into the ring while group G is worked on: into the half that held group G - 1,
    // whose last tile every wavefront had in registers at the barrier of that group.
    ring_store(0);
    request(1);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 8; ++c) row[c] = ring_piece(0, c);
    for (int T = 0; T < n_tiles; T += 2) {
      row_tile(T, std::integral_constant<int, 0>{});
      if (!(T & 2)) {
        ring_store((T >> 2) + 1);
        request((T >> 2) + 2);
      }
      if (T + 1 < n_tiles) row_tile(T + 1, std::integral_constant<int, 1>{});
    }
    f32x16 z = n_tiles & 1 ? acc[(NC - 1) & 1] : acc[(2 * NC - 1) & 1];
    if (n_tiles - 1 == J0 + NC - 1) drop_diagonal(z);
#pragma unroll
    for (int c = 0; c < 8; ++c) eighth(z, c, NC - 1);
    __syncthreads();                                       // what the last group asked the ring for has been read
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) {
      const double v = col[cc] + __shfl_xor(col[cc], 32);
      const int j = 32 * (J0 + cc) + r32;
      if (half == 0 && J0 + cc < J_end && j < l) cs[j] = j < first_recent ? v * (inv[j] * s_scale[1]) : 0.0;
    }
  };
  const Own own = own_of(RED_NW * share + order, RED_NW * shares);
  for (int p = 0; p < own.passes; ++p) {
    const int J0 = own.lo + own.n * p / own.passes, J1 = own.lo + own.n * (p + 1) / own.passes;
    if (p > 0 || shares > 1) {
      load_columns(J0, J1);
      request(0);
    }
    if (J1 - J0 == 3) pass(J0, J1, std::integral_constant<int, 3>{});
    else if (J1 - J0 == 2) pass(J0, J1, std::integral_constant<int, 2>{});
    else pass(J0, J1, std::integral_constant<int, 1>{});   // (or none: computed and dropped)
  }
  finish();
}

// ---- fp32 at d = 64 or 128 and bf16 at d = 64: the matrix cores in 64 bits --------------------------
// These shapes compute cosines and sums in fp64, here with MFMAs 16x16x4 of doubles: 2048 flops in 64
// cycles per SIMD; a unit is one workgroup of NW wavefronts, 16, or 8 at 512-byte rows, whose three
// tiles need the registers.  A wavefront takes column tiles wave, wave + NW, ... and walks all row tiles
// for each; a 16-byte piece holds EPC channels of its key and feeds EPC MFMAs, the i-th with channel i
// of every lane's piece.  The result lane (j = lane%16, kb) holds rows 4 i + kb in element i (not
// 4 kb + i as the 32-bit results do).
// Bound: fp64 matrix rate.  Against the plain kernel (a thread per column, scalar loads), per launch:
// l = 332, fp32 d = 128, 16 units 13.6 ms -> 145 us; fp32 d = 64, 32 units 6.6 ms -> 77 us; bf16 d = 64, 32
// units 6.0 ms -> 82 us; l = 152, 4 units 1.35 ms -> 23 us.
template <typename T, int D, int NW>
__global__ __launch_bounds__(NW * 64) void redundancy_f64_kernel(GkvDims dm, RedArgs a) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  constexpr int ROW_B = D * (int)sizeof(T), NL = ROW_B / 64, EPC = Elem<T>::EPC;
  a.step = resolve_step(dm, a.step);
  extern __shared__ double smem[];
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, kb = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv);
  double* cs = smem;
  double* inv = cs + dm.cap;
  double* red = inv + dm.cap;
  const SeqState st = load_state(a.d_state, lb);
  const int l = compression_length(st, a.step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const char* Kh = (const char*)a.K + (size_t)unit * dm.cap * ROW_B;
  const int n_tiles = (l + 15) >> 4;
  auto load_tile = [&](u32x4 (&k)[NL], int t) {
    const bool tiled = 16 * t < st.n_tiled;
    const char* p = Kh + (size_t)t * 16 * ROW_B + (tiled ? lane * 16 : r * ROW_B + kb * 16);
    const int step_off = tiled ? 1024 : 64;
#pragma unroll
    for (int c = 0; c < NL; ++c) k[c] = *(const u32x4*)(p + c * step_off);
  };
  auto elem = [](const u32x4& v, int i) {
    if constexpr (sizeof(T) == 4) return (double)__uint_as_float(v[i]);
    else return (double)__uint_as_float((i & 1) ? (v[i >> 1] & 0xffff0000u) : (v[i >> 1] << 16));
  };

  // row norms: a tile per wavefront, the 4 lanes of a row each sum their pieces
  for (int t = wave; t < n_tiles; t += NW) {
    u32x4 k[NL];
    load_tile(k, t);
    double ss = 0.0;
#pragma unroll
    for (int c = 0; c < NL; ++c)
#pragma unroll
      for (int i = 0; i < EPC; ++i) { const double x = elem(k[c], i); ss = fma(x, x, ss); }
    ss = add_quarters(ss);
    if (kb == 0) inv[16 * t + r] = ss;
  }
  __syncthreads();
  for (int n = tid; n < 16 * n_tiles; n += NW * 64) inv[n] = n < l ? 1.0 / (sqrt(inv[n]) + (double)a.eps) : 0.0;   // a row a thread, not four
  __syncthreads();

  const int first_recent = l - a.n_recent;
  const double tau = (double)a.tau;
  for (int J = wave; J < n_tiles; J += NW) {
    u32x4 kj[NL], cur[NL], nxt[NL];
    load_tile(kj, J);
    load_tile(cur, 0);
    const int j = 16 * J + r;
    const double inv_j = inv[j];
    double col = 0.0;
    for (int t = 0; t < n_tiles; ++t) {
      load_tile(nxt, min(t + 1, n_tiles - 1));
      f64x4 dot = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < NL; ++c)
#pragma unroll
        for (int i = 0; i < EPC; ++i)
          dot = __builtin_amdgcn_mfma_f64_16x16x4f64(elem(cur[c], i), elem(kj[c], i), dot, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 16 * t + 4 * i + kb;
        const double cv = dot[i] * inv[k] * inv_j;
        if (cv >= tau && k < l && k != j) col += cv;
      }
#pragma unroll
      for (int c = 0; c < NL; ++c) cur[c] = nxt[c];
    }
    col = add_quarters(col);
    if (kb == 0 && j < l) cs[j] = j < first_recent ? col : 0.0;
  }
  __syncthreads();
  finish_unit<NW>(dm, a, unit, l, cs, red);
}

// The same for few units: a workgroup takes one column tile at a time (gridDim.y of them share a unit's), its four
// wavefronts a quarter of the row tiles each, and the sums are added up in a fixed order.  Every workgroup forms the
// norms of all rows: as many reads as its own rows, a tenth of the arithmetic.  us per call with the finishing launch,
// against a workgroup per unit: fp32 d = 128 8 units of 366 rows 160 -> 19, 64 of 232 73 -> 34; bf16 d = 64 32 of 428
// 120 -> 31, 128 of 232 43 -> 30; fp32 d = 64 16 of 132 21 -> 8.7.  Not above 128 units: 256 of 160 24 -> 26, fp32 d = 128 512 of 132
// 73 -> 80.
constexpr int RED_SPLIT_UNITS = 128;
template <typename T, int D>
__global__ __launch_bounds__(256) void redundancy_f64_split_kernel(GkvDims dm, RedArgs a) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  constexpr int ROW_B = D * (int)sizeof(T), NL = ROW_B / 64, EPC = Elem<T>::EPC, NW = 4;
  a.step = resolve_step(dm, a.step);
  extern __shared__ double smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r = lane & 15, kb = lane >> 4;
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv);
  double* inv = smem;
  double* part = inv + dm.cap;                           // [NW][16]
  double* cs = part + NW * 16;                           // [16]
  const SeqState st = load_state(a.d_state, lb);
  const int l = compression_length(st, a.step, dm.b, dm.w, dm.cap);
  const int n_tiles = (l + 15) >> 4;
  if ((int)blockIdx.y >= n_tiles) return;                // (l == 0 among them)
  const char* Kh = (const char*)a.K + (size_t)unit * dm.cap * ROW_B;
  auto load_tile = [&](u32x4 (&k)[NL], int t) {
    const bool tiled = 16 * t < st.n_tiled;
    const char* p = Kh + (size_t)t * 16 * ROW_B + (tiled ? lane * 16 : r * ROW_B + kb * 16);
    const int step_off = tiled ? 1024 : 64;
#pragma unroll
    for (int c = 0; c < NL; ++c) k[c] = *(const u32x4*)(p + c * step_off);
  };
  auto elem = [](const u32x4& v, int i) {
    if constexpr (sizeof(T) == 4) return (double)__uint_as_float(v[i]);
    else return (double)__uint_as_float((i & 1) ? (v[i >> 1] & 0xffff0000u) : (v[i >> 1] << 16));
  };
  for (int t = wave; t < n_tiles; t += NW) {
    u32x4 k[NL];
    load_tile(k, t);
    double ss = 0.0;
#pragma unroll
    for (int c = 0; c < NL; ++c)
#pragma unroll
      for (int i = 0; i < EPC; ++i) { const double x = elem(k[c], i); ss = fma(x, x, ss); }
    ss = add_quarters(ss);
    if (kb == 0) inv[16 * t + r] = ss;
  }
  __syncthreads();
  for (int n = tid; n < 16 * n_tiles; n += NW * 64) inv[n] = n < l ? 1.0 / (sqrt(inv[n]) + (double)a.eps) : 0.0;
  __syncthreads();
  const double tau = (double)a.tau;
  for (int J = blockIdx.y; J < n_tiles; J += gridDim.y) {
    u32x4 kj[NL], cur[NL], nxt[NL];
    load_tile(kj, J);
    load_tile(cur, min(wave, n_tiles - 1));
    const int j = 16 * J + r;
    const double inv_j = inv[j];
    double col = 0.0;
    for (int t = wave; t < n_tiles; t += NW) {
      load_tile(nxt, min(t + NW, n_tiles - 1));
      f64x4 dot = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int c = 0; c < NL; ++c)
#pragma unroll
        for (int i = 0; i < EPC; ++i)
          dot = __builtin_amdgcn_mfma_f64_16x16x4f64(elem(cur[c], i), elem(kj[c], i), dot, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 16 * t + 4 * i + kb;
        const double cv = dot[i] * inv[k] * inv_j;
        if (cv >= tau && k < l && k != j) col += cv;
      }
#pragma unroll
      for (int c = 0; c < NL; ++c) cur[c] = nxt[c];
    }
    col = add_quarters(col);
    if (kb == 0) part[16 * wave + r] = col;
    __syncthreads();
    if (tid < 16) {
      const double v = (part[tid] + part[16 + tid]) + (part[32 + tid] + part[48 + tid]);
      cs[tid] = 16 * J + tid < l - a.n_recent ? v : 0.0;
      store_sums(dm, a, unit, 16 * J, min(16 * J + 16, l - dm.w), cs - 16 * J, tid, 16);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void redundancy_finish_kernel(GkvDims dm, RedArgs a) {
  a.step = resolve_step(dm, a.step);
  extern __shared__ double smem[];
  const int unit = blockIdx.x, lb = quotient(unit, dm.by_hkv);
  double* cs = smem;
  const int l = compression_length(load_state(a.d_state, lb), a.step, dm.b, dm.w, dm.cap);
  if (l == 0) return;
  const float* lo = a.R_norm + (size_t)unit * dm.cap;
  const float* hi = a.F_sel + (size_t)unit * dm.cap;
  for (int j = threadIdx.x; j < l; j += 256)
    cs[j] = j < l - dm.w ? __hiloint2double(__float_as_int(hi[j]), __float_as_int(lo[j])) : 0.0;
  __syncthreads();
  finish_unit<4>(dm, a, unit, l, cs, cs + dm.cap);
}

// The ring passes the default per-workgroup limit of LDS (a compute unit holds 160 KiB): opt in, once a device, for the
// largest capacity.  Each call costs the host 0.3 us otherwise.
hipError_t red_opt_in() {
  static std::atomic<uint64_t> done{0};
  int dev = -1;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t set = hipFuncSetAttribute((const void*)redundancy_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)(RED_LDS_ROW * 4096 + RED_LDS_FIXED));
  if (set == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return set;
}

}  // namespace

hipError_t gkv_launch_redundancy(const GkvLaunch& ln, const GkvDims& dm, int dtype, bool mfma, bool f64_mfma, const void* K,
                                 const int32_t* d_state, int32_t step, const float* F, float lambda, float tau,
                                 float eps, int32_t n_recent, float* R_norm, float* F_sel) {
  RedArgs a{K, d_state, step, F, lambda, tau, eps, n_recent, R_norm, F_sel};
  const int units = dm.L * dm.B * dm.Hkv;
  // a unit's columns are shared out where there are few units; the sums need the results' places (store_sums)
  auto apart = [&](const float* x, const float* y) { return x < y ? y - x >= (int64_t)units * dm.cap : x - y >= (int64_t)units * dm.cap; };
  const bool few = units <= RED_SPLIT_UNITS && n_recent >= dm.w && apart(R_norm, F_sel) && apart(R_norm, F) && apart(F_sel, F);
  auto finish = [&]() {
    GkvLaunch more = ln;
    more.continued = true;
    return gkv_launch(more, redundancy_finish_kernel, dim3(units), dim3(256), sizeof(double) * ((size_t)dm.cap + 4), dm, a);
  };
  if (mfma) {
    const size_t with_ring = RED_LDS_ROW * (size_t)dm.cap + RED_LDS_FIXED;
    auto kern = redundancy_mfma_kernel;
    const hipError_t opted = red_opt_in();
    if (opted != hipSuccess) return opted;
    // as many workgroups as there are compute units, each wavefront with a column tile at least
    const int most = ((dm.cap + 31) / 32 + RED_NW - 1) / RED_NW;
    const bool share = few && dm.cap >= (units <= 64 ? 448 : 704);
    const int shares = !share ? 1 : 256 / units < most ? 256 / units : most;
    const hipError_t e = gkv_launch(ln, kern, dim3(units, shares), dim3(RED_NW * 64), with_ring, dm, a);
    return e == hipSuccess && shares > 1 ? finish() : e;
  }
  if (f64_mfma) {
    const bool wide = dtype == GKV_F32 && dm.d == 128;
    if (few) {
      const int tiles = (dm.cap + 15) / 16, shares = tiles < 1024 / units ? tiles : (1024 + units - 1) / units;
      auto split = wide ? redundancy_f64_split_kernel<float, 128>
                        : dtype == GKV_F32 ? redundancy_f64_split_kernel<float, 64> : redundancy_f64_split_kernel<uint16_t, 64>;
      const hipError_t e = gkv_launch(ln, split, dim3(units, shares), dim3(256), sizeof(double) * ((size_t)dm.cap + 80), dm, a);
      if (e != hipSuccess) return e;
      return finish();
    }
    auto kern = wide ? redundancy_f64_kernel<float, 128, 8>
                     : dtype == GKV_F32 ? redundancy_f64_kernel<float, 64, 16> : redundancy_f64_kernel<uint16_t, 64, 16>;
    return gkv_launch(ln, kern, dim3(units), dim3(wide ? 512 : 1024), sizeof(double) * (2 * (size_t)dm.cap + 16), dm, a);
  }
  const size_t shmem = sizeof(double) * (2 * (size_t)dm.cap + 4);
  if (dtype == GKV_F32)
    return gkv_launch(ln, redundancy_generic_kernel<float>, dim3(units), dim3(256), shmem, dm, a);
  return gkv_launch(ln, redundancy_generic_kernel<uint16_t>, dim3(units), dim3(256), shmem, dm, a);
}
