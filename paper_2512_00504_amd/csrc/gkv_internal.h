// Internal declarations shared by the C-ABI layer and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gkv.h"
#include "gkv_bench.h"

// x / d = (2 x mul) >> (32 + shift) for 0 <= x < 2^31, with mul = 2^(31 + shift) / d rounded up and
// 2^shift >= d the smallest (mul d exceeds 2^(31 + shift) by less than d <= 2^shift).
struct GkvDivisor { uint32_t mul; uint32_t shift; };
static inline GkvDivisor gkv_divisor(int32_t d) {
  uint32_t shift = 0;
  while ((int64_t)1 << shift < d) ++shift;
  return GkvDivisor{(uint32_t)((((uint64_t)1 << (31 + shift)) + d - 1) / d), shift};
}

// Dimensions every kernel needs, passed by value.
struct GkvDims {
  int32_t L, B, Hq, Hkv, d, g;
  int32_t b, w, s, cap;
  int32_t combine;
  float alpha;
  float scale;   // softmax scale of Eq. 1
  // scale * log2(e) as an unevaluated sum hi + lo: the matrix-core kernels form the exponent of
  // 2 as fma(z, lo, fma(z, hi, -m)), two roundings of a small number and no systematic error
  // from a rounded scale, and the decode and window-score kernels form it the same way
  float scale_l2_hi, scale_l2_lo;
  // Device-side step counter (null: none).  When set, the `step` argument of a call is relative
  // and the kernels use *step_base + step, so recorded launches (HIP graphs) can be replayed.
  const int32_t* step_base;
  GkvDivisor by_hkv;
};

struct GkvProfile;   // event pools, defined in gkv_api.hip

// Decode calls that the library cuts by its own choice use one of this many sets of tickets and partial
// results in the workspace, by the stream they are enqueued on: calls on one stream follow each other,
// calls on different ones may overlap.  A recorded call runs later than what is enqueued on its stream
// now, so each capture counts as a stream of its own.
constexpr int GKV_SPLIT_SETS = 8;
constexpr int GKV_TICKETS = 8;   // tickets per unit and set: one for each wavefront that has outputs (g * d / 256, at most 8)
struct GkvStreamKey { const void* stream; unsigned long long capture; };

struct gkv_ctx {
  gkv_config cfg;
  GkvDims dims;
  int32_t esz;            // bytes per element
  int32_t attend_splits;  // 0 = automatic
  int32_t ws_splits;      // "attend_splits" the workspace was sized for by gkv_workspace_bytes (1 = no partials)
  int32_t ws_auto_splits; // the same for the library's own choice
  const void* split_ws;   // workspace whose tickets gkv_workspace_init of this context zeroed
  int32_t n_split_keys;   // streams that have a set so far; they keep it for the context's life, recorded calls being replayed at any time
  GkvStreamKey split_key[GKV_SPLIT_SETS];
  int32_t attend_tile;    // keys per wavefront iteration of the matrix-core attend kernel: 16 or 32
  int32_t force_generic;
  int32_t attend_waves;   // 0 = automatic
  int32_t fuse_global;    // gkv_evict: as fuse_select (the global score is not a launch of its own)
  int32_t fuse_select;    // gkv_evict: global score at the head of the top-k kernel (default)
  int32_t compact_ppt;    // 16-byte pieces per thread and chunk round of the compaction kernel: 4, 8 or 16
  int32_t reuse_stats;    // window score may reuse the softmax statistics the decode kernel recorded
  bool mfma_shape;        // d == 64 or 128, g <= 16: the matrix-core decode and window-score kernels cover it
  bool mfma_redundancy;   // bf16, d == 128, g <= 16: the matrix-core redundancy kernel does
  GkvProfile* prof;
  // Host record of which ring slots hold softmax statistics written by the matrix-core decode
  // kernel: stats_step[slot] = decode step whose statistics the slot holds (-1 = none), valid for
  // exactly these buffers.
  int32_t* stats_step;    // [w]
  const void* stats_ws; const void* stats_K; const void* stats_qwin;
  GkvStreamKey stats_key;   // stream of the last decode call
  bool stats_mixed;         // the context has decoded another K cache on another stream
};

// Workspace layout (bytes from the base):
//   [0, 4*GKV_TICKETS*units*sets)   split tickets (int32, self-resetting); sets = GKV_SPLIT_SETS and one for
//                                   "attend_splits", or the latter alone where the library never cuts
//   [.., + 4*L*B)                   compaction tickets
//   [.., + 8*w*L*B*h_q)             softmax statistics ring: per (slot, layer, sequence, query head)
//                                   the running max (log2 units) and the sum of the decode step
//                                   whose q sits in that slot of the window ring
//   [.., + 4*units*splits*g*(d+2) per set)  split-K partials (float)
struct GkvWorkspace {
  int32_t* split_ticket;  // of the call's set, as partials
  int32_t* state_ticket;  // [L*B]: compaction workgroups of a (layer, sequence) that have finished; zero between launches
  float2* stats;
  float* partials;
};

static inline size_t gkv_align256(size_t x) { return (x + 255) & ~size_t(255); }

constexpr size_t GKV_LDS_LIMIT = 65536;
size_t gkv_max_lds_bytes(const gkv_config* cfg);
GkvWorkspace gkv_carve_workspace(const gkv_ctx* ctx, void* base, int split_set = 0);

// Launch record for profiling: the wrappers launch through gkv_launch() below.
struct GkvLaunch {
  gkv_ctx* ctx;
  int kernel_id;
  hipStream_t stream;
  bool continued = false;   // a further launch of the same call: its time counts, the call does not count again
};

// ---- launch wrappers implemented in the kernel files -------------------------------------
struct AttendArgs {
  const void* q; const void* k_new; const void* v_new;
  void* K; void* V; int32_t* pos; int32_t step; void* qwin; const int32_t* d_state; void* out;
  GkvWorkspace ws; int32_t splits; int32_t tile_keys;
  int32_t copy_q;   // 0 when q already is the ring slot of this step
  int32_t write_stats;   // record (max, sum) of every query head's softmax in ws.stats
  int32_t waves;         // wavefronts per workgroup of the matrix-core kernel: 4, 8 or 16
  int32_t split_iters;   // slices per piece (a unit of n slices is cut into ceil(n / split_iters)); 0 = all splits
};
hipError_t gkv_launch_attend_generic(const GkvLaunch& ln, const GkvDims& dm, int dtype, const AttendArgs& a);
hipError_t gkv_launch_attend_mfma(const GkvLaunch& ln, const GkvDims& dm, int dtype, const AttendArgs& a);
// LDS of a workgroup of that kernel (bytes)
size_t gkv_attend_mfma_lds(int esz, int d, int g, int waves);

struct ScoreArgs {
  const void* qwin; const void* K; const int32_t* d_state; int32_t step; float* S;
  const float2* stats;   // softmax statistics of the window's decode steps, or null: compute them
};
hipError_t gkv_launch_score_generic(const GkvLaunch& ln, const GkvDims& dm, int dtype, const ScoreArgs& a);
hipError_t gkv_launch_score_mfma(const GkvLaunch& ln, const GkvDims& dm, int dtype, const ScoreArgs& a, int len_max);

hipError_t gkv_launch_global_update(const GkvLaunch& ln, const GkvDims& dm, const float* S,
                                    const float* F_hist, const int32_t* d_state, int32_t step, float* F_out);
hipError_t gkv_launch_select_topk(const GkvLaunch& ln, const GkvDims& dm, const float* F,
                                  const int32_t* d_state, int32_t step, int32_t* keep_idx);
hipError_t gkv_launch_update_and_select(const GkvLaunch& ln, const GkvDims& dm, const float* S, const float* F_hist,
                                        const int32_t* d_state, int32_t step, float* F_out, int32_t* keep_idx);
hipError_t gkv_launch_compact(const GkvLaunch& ln, const GkvDims& dm, int esz, const int32_t* keep_idx,
                              const float* F, void* K, void* V, float* F_hist, int32_t* pos,
                              int32_t* d_state, int32_t step, int32_t* state_ticket);
hipError_t gkv_launch_redundancy(const GkvLaunch& ln, const GkvDims& dm, int dtype, bool mfma, bool f64_mfma, const void* K,
                                 const int32_t* d_state, int32_t step, const float* F, float lambda, float tau,
                                 float eps, int32_t n_recent, float* R_norm, float* F_sel);
hipError_t gkv_launch_pool_scores(const GkvLaunch& ln, const GkvDims& dm, const float* F, const int32_t* d_state,
                                  int32_t step, int32_t kernel, float* F_out);
hipError_t gkv_launch_evicted_positions(const GkvLaunch& ln, const GkvDims& dm, const int32_t* keep_idx,
                                        const int32_t* pos, const int32_t* d_state, int32_t step, int32_t* evicted);
hipError_t gkv_launch_fill_zero(hipStream_t stream, int32_t* p, size_t n);
hipError_t gkv_launch_add_int(hipStream_t stream, int32_t* p, int32_t delta);

// Event bracketing for profiling (gkv_api.hip).  Returns the events to pass to
// hipExtLaunchKernelGGL, or nulls when profiling is off.
void gkv_profile_events(const GkvLaunch& ln, hipEvent_t* start, hipEvent_t* stop);

// ---- device helpers ------------------------------------------------------------------------
#ifdef __HIPCC__
#include <hip/hip_ext.h>

template <typename... Args, typename F = void (*)(Args...)>
static inline hipError_t gkv_launch(const GkvLaunch& ln, F kernel, dim3 grid, dim3 block,
                                    size_t shmem, Args... args) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  gkv_profile_events(ln, &e0, &e1);
  if (e0) {
    hipExtLaunchKernelGGL(kernel, grid, block, shmem, ln.stream, e0, e1, 0, args...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, shmem, ln.stream, args...);
  }
  return hipGetLastError();
}

// x / d for 0 <= x < 2^31.  An integer division is some twenty instructions, at the start of kernels whose first
// requests wait for it.
__device__ __forceinline__ int quotient(int x, GkvDivisor d) { return (int)(__umulhi(2u * (uint32_t)x, d.mul) >> d.shift); }

// The per-(layer, sequence) record of d_state, read with one 16-byte load.
struct SeqState {
  int32_t len, len_step, n_hist, n_tiled;
};
__device__ __forceinline__ SeqState state_record(const int4& v) {
  // the tiled prefix is whole tiles and never reaches past the stored length
  int nt = v.w & ~15;
  const int lim = (v.x > 0 ? v.x : 0) & ~15;
  nt = nt < 0 ? 0 : (nt > lim ? lim : nt);
  return SeqState{v.x, v.y, v.z, nt};
}
__device__ __forceinline__ SeqState load_state(const int32_t* d_state, int lb) {
  return state_record(*(const int4*)(d_state + 4 * (size_t)lb));
}
// Length before decode step `t` (every step since len_step appended one row), kept inside [0, cap].
__device__ __forceinline__ int length_before_step(const SeqState& s, int t, int cap) {
  const int l = s.len + (t - s.len_step);
  return l < 0 ? 0 : (l > cap ? cap : l);
}

// The decode step a kernel works on: its argument, plus the device-side step base if there is one.
__device__ __forceinline__ int resolve_step(const GkvDims& dm, int step) {
  return dm.step_base ? step + *dm.step_base : step;
}

// Whether the compression after decode step `step` applies to this (layer, sequence): its cache
// must exceed the budget, and the observation window must consist of generated tokens, i.e. at
// least w steps were decoded since the cache was loaded or last compacted (a prompt brings keys
// and values but no window queries).  Returns the length l the compression sees, or 0 for "skip".
__device__ __forceinline__ int compression_length(const SeqState& s, int step, int b, int w, int cap) {
  const int l = length_before_step(s, step + 1, cap);
  return (l > b && step + 1 - s.len_step >= w) ? l : 0;
}

// Element offset of (row n, channel c) in one KV head's K block whose first n_tiled rows are in
// tiled format; EPC = elements per 16 bytes.
template <int EPC>
__device__ __forceinline__ int k_elem_offset(int n, int c, int d, int n_tiled) {
  if (n >= n_tiled) return n * d + c;
  return (n >> 4) * 16 * d + (c / EPC) * (16 * EPC) + (n & 15) * EPC + (c % EPC);
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {   // round to nearest even
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);   // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int EPC = 4;
  __device__ static __forceinline__ float ld(const float* p) { return *p; }
  __device__ static __forceinline__ void st(float* p, float v) { *p = v; }
};
template <> struct Elem<uint16_t> {     // bf16 bit patterns
  static constexpr int EPC = 8;
  __device__ static __forceinline__ float ld(const uint16_t* p) { return bf16_bits_to_float(*p); }
  __device__ static __forceinline__ void st(uint16_t* p, float v) { *p = float_to_bf16_bits(v); }
};

// Running maximum (log2 units) before the first key.
constexpr float GKV_NO_MAX = -3.402823466e38f;
// From this magnitude of a running maximum on, products with the scale are rounded one by one.
constexpr float GKV_HUGE_LOG2 = 0x1p22f;
__device__ __forceinline__ float rounded_product(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}
// z * (hi + lo) - m, the exponent of 2 of a logit's weight under the running maximum m = round(max z * hi),
// with two roundings of a small number.  For the largest logit that is what rounding m left over, up to
// |m| * 2^-24, which must not reach the exponential once m is in the millions: there the product is rounded
// as m was (as the plain kernels round theirs), which gives the largest logit exactly 0.  A logit of -inf
// gives -inf (weight 0) whatever the sign of lo, one of +inf or NaN gives NaN, as exp(z - max) does.
__device__ __forceinline__ float log2_weight(float z, float hi, float lo, float m) {
  if (fabsf(m) >= GKV_HUGE_LOG2) return rounded_product(z, hi) - m;
  return fmaf(fmaxf(z, -3.402823466e38f), lo, fmaf(z, hi, -m));
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
#endif  // __HIPCC__
