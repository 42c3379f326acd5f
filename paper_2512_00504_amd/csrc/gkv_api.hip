// C-ABI layer: argument validation, workspace carving, kernel selection, profiling events.
#include <math.h>
#include <string.h>

#include <initializer_list>
#include <mutex>
#include <new>
#include <vector>

#include "gkv_internal.h"

// ---- profiling ----------------------------------------------------------------------------------
struct GkvProfile {
  bool on = false;
  struct Rec { hipEvent_t e0, e1; bool continued; };
  std::vector<Rec> recs[GKV_K_COUNT];
  double done_ms[GKV_K_COUNT] = {};
  int64_t done_n[GKV_K_COUNT] = {};
};

void gkv_profile_events(const GkvLaunch& ln, hipEvent_t* start, hipEvent_t* stop) {
  *start = nullptr; *stop = nullptr;
  GkvProfile* p = ln.ctx ? ln.ctx->prof : nullptr;
  if (!p || !p->on || ln.kernel_id < 0 || ln.kernel_id >= GKV_K_COUNT) return;
  GkvProfile::Rec rec;
  rec.continued = ln.continued;
  if (hipEventCreate(&rec.e0) != hipSuccess) return;
  if (hipEventCreate(&rec.e1) != hipSuccess) { (void)hipEventDestroy(rec.e0); return; }
  p->recs[ln.kernel_id].push_back(rec);
  *start = rec.e0; *stop = rec.e1;
}

static void profile_drain(GkvProfile* p, int k) {
  for (auto& rec : p->recs[k]) {
    float ms = 0.f;
    if (hipEventSynchronize(rec.e1) == hipSuccess && hipEventElapsedTime(&ms, rec.e0, rec.e1) == hipSuccess) {
      p->done_ms[k] += ms;
      p->done_n[k] += !rec.continued;
    }
    (void)hipEventDestroy(rec.e0);
    (void)hipEventDestroy(rec.e1);
  }
  p->recs[k].clear();
}

// ---- context ------------------------------------------------------------------------------------
static gkv_status validate_config(const gkv_config* c) {
  if (!c) return GKV_ERR_INVALID_ARG;
  if (c->dtype != GKV_F32 && c->dtype != GKV_BF16) return GKV_ERR_INVALID_ARG;
  if (c->combine < GKV_COMBINE_MAX || c->combine > GKV_COMBINE_SUM) return GKV_ERR_INVALID_ARG;
  if (c->n_layers < 1 || c->batch < 1 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->head_dim < 1)
    return GKV_ERR_INVALID_ARG;
  if (c->n_q_heads % c->n_kv_heads != 0) return GKV_ERR_INVALID_ARG;
  if (c->budget < 2 || c->window < 1 || c->interval < 1) return GKV_ERR_INVALID_ARG;
  if (c->window > c->interval || c->window >= c->budget) return GKV_ERR_INVALID_ARG;
  if (!(c->alpha >= 0.f && c->alpha <= 1.f)) return GKV_ERR_INVALID_ARG;
  if (!(c->softmax_scale >= 0.f) || isinf(c->softmax_scale)) return GKV_ERR_INVALID_ARG;
  const int esz = c->dtype == GKV_F32 ? 4 : 2;
  const int epc = 16 / esz;
  if (c->head_dim % epc != 0 || c->head_dim * esz > 1024) return GKV_ERR_SHAPE;
  if (c->capacity < c->budget + c->interval || c->capacity % 32 != 0 || c->capacity > 4096)
    return GKV_ERR_SHAPE;
  const int64_t units = (int64_t)c->n_layers * c->batch * c->n_kv_heads;
  if (units > (1 << 24)) return GKV_ERR_SHAPE;
  if (gkv_max_lds_bytes(c) > GKV_LDS_LIMIT) return GKV_ERR_SHAPE;
  return GKV_OK;
}

// Largest LDS footprint (dynamic + static, bytes) of any kernel that can be selected for this
// configuration; the plain vector-ALU kernels are included because "force_generic" may select them
// for any shape.  A workgroup gets 64 KiB without opting in to more.
size_t gkv_max_lds_bytes(const gkv_config* c) {
  const size_t cap = (size_t)c->capacity, d = (size_t)c->head_dim;
  const size_t g = (size_t)(c->n_q_heads / c->n_kv_heads);
  size_t need = 16 * (cap + 1 + d);                                 // attend_generic: 4 wavefronts x float[cap + 1 + d]
  auto upd = [&](size_t x) { if (x > need) need = x; };
  upd(4 * (3 * cap + d));                                           // score_generic: at least one wavefront's float[3 cap + d]
  upd(16 * cap + 32);                                               // redundancy: double cs[cap], red[4], inv[cap]
  if ((d == 64 || d == 128) && g <= 16) upd(16 * cap + 128);        // its 64-bit matrix-core form: a double per wavefront
  // (the matrix-core redundancy kernel takes 12 cap + 64 KiB, with its ring of row tiles, and asks for the
  // larger per-workgroup allowance itself: 110 KiB at 3936 rows, the most that pass at d = 128, of the 160 KiB a
  // compute unit holds)
  upd(4 * cap + 64);                                                // pooled score / eviction log
  if ((d == 64 || d == 128) && g <= 16)                             // attend_mfma: partial outputs + staged rows
    upd(gkv_attend_mfma_lds(c->dtype == GKV_F32 ? 4 : 2, (int)d, (int)g, 4) + 16);
  return need;
}

extern "C" gkv_status gkv_create(const gkv_config* cfg, gkv_ctx** out_ctx) {
  if (!out_ctx) return GKV_ERR_INVALID_ARG;
  *out_ctx = nullptr;
  gkv_status st = validate_config(cfg);
  if (st != GKV_OK) return st;
  gkv_ctx* c = new (std::nothrow) gkv_ctx();
  if (!c) return GKV_ERR_INVALID_ARG;
  c->cfg = *cfg;
  GkvDims& d = c->dims;
  d.L = cfg->n_layers; d.B = cfg->batch; d.Hq = cfg->n_q_heads; d.Hkv = cfg->n_kv_heads;
  d.d = cfg->head_dim; d.g = cfg->n_q_heads / cfg->n_kv_heads;
  d.b = cfg->budget; d.w = cfg->window; d.s = cfg->interval; d.cap = cfg->capacity;
  d.combine = cfg->combine; d.alpha = cfg->alpha;
  d.scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : (float)(1.0 / sqrt((double)cfg->head_dim));
  {
    const double sl2 = (double)d.scale * 1.4426950408889634074;
    d.scale_l2_hi = (float)sl2;
    d.scale_l2_lo = (float)(sl2 - (double)d.scale_l2_hi);
  }
  d.step_base = nullptr;
  d.by_hkv = gkv_divisor(d.Hkv);
  c->esz = cfg->dtype == GKV_F32 ? 4 : 2;
  c->attend_splits = 0;
  c->ws_splits = 1;
  c->ws_auto_splits = 1;
  c->split_ws = nullptr;
  c->n_split_keys = 0;
  c->attend_tile = 16;
  c->force_generic = 0;
  c->reuse_stats = 1;
  c->compact_ppt = 8;
  c->fuse_global = 0;
  c->fuse_select = 1;
  c->attend_waves = 0;
  c->stats_step = new (std::nothrow) int32_t[cfg->window];
  if (!c->stats_step) { delete c; return GKV_ERR_INVALID_ARG; }
  for (int i = 0; i < cfg->window; ++i) c->stats_step[i] = -1;
  c->stats_ws = c->stats_K = c->stats_qwin = nullptr;
  c->stats_key = GkvStreamKey{nullptr, 0};
  c->stats_mixed = false;
  c->mfma_redundancy = cfg->dtype == GKV_BF16 && d.d == 128 && d.g <= 16;
  c->mfma_shape = (d.d == 64 || d.d == 128) && d.g <= 16;
  c->prof = new (std::nothrow) GkvProfile();
  *out_ctx = c;
  return GKV_OK;
}

extern "C" void gkv_destroy(gkv_ctx* ctx) {
  if (!ctx) return;
  if (ctx->prof) {
    for (int k = 0; k < GKV_K_COUNT; ++k) profile_drain(ctx->prof, k);
    delete ctx->prof;
  }
  delete[] ctx->stats_step;
  delete ctx;
}

extern "C" const char* gkv_status_string(gkv_status st) {
  switch (st) {
    case GKV_OK: return "ok";
    case GKV_ERR_INVALID_ARG: return "invalid argument";
    case GKV_ERR_SHAPE: return "unsupported shape";
    case GKV_ERR_WORKSPACE: return "workspace missing";
    case GKV_ERR_HIP: return "HIP runtime error";
    case GKV_ERR_UNSUPPORTED: return "unsupported";
    case GKV_ERR_OVERFLOW: return "cache capacity exceeded";
    case GKV_ERR_SCRATCH: return "configuration exceeds the static scratch array";
  }
  return "unknown status";
}

static int max_splits(const gkv_ctx* ctx) {
  // a split workgroup of 4 wavefronts covers 128 keys per round
  int m = ctx->dims.cap / 128;
  return m < 1 ? 1 : (m > 64 ? 64 : m);
}

// Workgroups per unit asked for with "attend_splits" (1: not asked for).
static int explicit_splits(const gkv_ctx* ctx) {
  if (!ctx->mfma_shape || ctx->force_generic || ctx->attend_splits <= 1) return 1;
  const int m = max_splits(ctx);
  return ctx->attend_splits > m ? m : ctx->attend_splits;
}

// How the matrix-core decode kernel cuts a launch: wavefronts per workgroup, workgroups per unit at
// most, and the slices per piece (0: every unit is cut into all of its pieces; n slices make
// ceil(n / iters) of them, so the last may be shorter).  Depends on the configuration alone, so the same
// call gives the same bits whatever bound of the length the caller passes.
//
// A workgroup on a CU of its own takes a microsecond per round of slices, one for each wavefront; cutting a unit shortens
// that and costs the merge, 1.7 us and more with every piece, and from 256 workgroups on some CUs have two.  So up to 128 units are cut.
//
// Where every CU gets a workgroup and each piece 20 slices of a unit of ordinary length b + s/2, pieces have
// 8 wavefronts, and a unit of more than eight slices for each of them is cut into all of them.  us per launch with cold caches, 4 wavefronts and
// two slices in flight -> this: bf16, D = 128 128 units x 720 rows 11.4 -> 11.1, x 2113 24.1 -> 23.3, 100 x 800 10.9 -> 10.5, 64 x
// 1300 11.2 -> 10.9, x 2113 14.6 -> 14.4; D = 64 128 x 1300 12.2 -> 10.55, 64 x 3900 15.5 -> 13.4; fp32, D = 64 128 x 800 13.1 -> 12.2, 64 x
// 1300 11.8 -> 11.1, but 128 x 600 10.55 / 11.0 (18 slices a piece), and bf16 32 x 2113 (19) 10.0 / 10.2.  Ragged to 3900 rows: 128 units 28.5 ->
// 29.0, 64 17.7 -> 17.1; to 1500 100 14.1 -> 12.9.  (Pieces of 128 slices there, so that shorter units stay whole: 27.8 and 16.6, but then fewer
// wavefronts round their probabilities by a maximum of their own, and the error against 64 bits grows, see WHOLE in attend_mfma.hip.)
//
// Otherwise pieces of 4 wavefronts with equal rounds, at most 7 of them (units of more than 168 slices: as many as leave a piece 24
// slices, 6 rounds), for a unit of ordinary length; longer ones get more pieces of that size while there are workgroups left.  us per launch in a
// graph, pieces x wavefronts (rounds), bf16, D = 128 (before their probabilities entered in two parts, which adds 1 to 2%):
//   4 units x 577 rows: uncut 6.4 with 8, 6.8 with 4; 3x4(4) 5.9, 4x4(3) 5.6, 5x4(2) 5.5, 10x4(1) 6.2, 5x8(1) 5.9
//   32 x 577: uncut 7.0; 3x4 6.4, 4x4 6.2, 5x4(2) 6.0, 10x4 7.9;  32 x 1100: 11.8; 5x4 7.5, 6x4(3) 7.0, 8x4 7.8, 9x4(2) 8.7
//   4 x 2113: 13.3; 5x4 7.35, 7x4(5) 6.9, 9x4 7.15, 16x4 7.8;  4 x 3900: 27.4; 7x4(9) 9.5, 11x4(6) 8.1, 16x4 8.3;  64 x 577: 8.7; 4x4(3) 7.2, 5x4 7.7
// ragged: 84 to 464 uncut 8.1, 3x4 6.3; 16 to 307 5.9, 5x4 4.9.  fp32: D = 128 32 x 528 uncut 15.3, 5x4(2) 8.2, 8x4 8.6, 9x4(1) 9.8, 48 x 300 10.7,
// 5x4(1) 6.5, 100 x 300 11.4, 2x4 10.1; D = 64 8 x 350 7.1, 6x4(1) 4.85.  bf16, D = 64: 16 x 528 5.65, 5x4(1) 5.15.
//
// Short units stay whole: up to 17 slices (4 x 300 4.85, 5x4(1) 4.9; 2 x 200 4.5, 5.0); where there are only two pieces up to 39 (cold, uncut with 8 / cut:
// 128 x 545 9.15 / 9.8, x 640 10.1 / 10.6, x 800 11.6 / 11.8, x 1000 13.5 both, but ragged to 800 11.4 / 9.7; bf16, D = 64 x 1056, of 32 rows
// a slice, 9.3 / 9.5, x 1500 11.75 / 11.6), 29 in fp32 (128 x 400 8.9 / 9.5, x 500 10.0 both, x 650 11.6 / 11.1).  Prompts
// much longer than that are cut: from 64 slices of capacity where there are two pieces (fp32: 48), else from twice as many.
// Uncut, 8 wavefronts serve up to 256 units that give each two slices (4 units x 260 5.1 -> 4.6, x 200 4.6 -> 4.9; 128 x 260 6.4 -> 6.1) and
// more than 512 units of 64 slices (896 x 2113 159.5 -> 157, ragged to 3900 174 -> 170); in between 4 do (512 x 1100 45.2 against 45.7, 270 x
// 2000 55.3 / 59.5).  fp32 at D = 128 has 16 KiB slices and stays at 4 (256 x 577 25.6 / 26.9).  With "attend_splits" pieces of 48 slices and more
// have 8 (2 x 64 units of 2000 fp32 rows, D = 64 18.8 -> 17.8).
struct AttendPlan { int waves, splits, iters; };

static AttendPlan attend_plan(const gkv_ctx* ctx, int asked) {
  const GkvDims& d = ctx->dims;
  auto fits = [&](int waves) { return gkv_attend_mfma_lds(ctx->esz, d.d, d.g, waves) <= 65000; };
  const int64_t units = (int64_t)d.L * d.B * d.Hkv;
  const int row_bytes = d.d * ctx->esz;
  const bool wide = row_bytes > 256;                                  // 16 KiB slices
  const int keys = row_bytes == 128 ? 32 : 16;                        // per slice
  const int typical = (d.b + d.s / 2 + keys - 1) / keys, full = d.cap / keys;   // slices of a unit
  const bool long_slices = ctx->attend_tile == 32 && ctx->cfg.dtype == GKV_BF16 && d.d == 128;   // 4 wavefronts only
  const bool may_have_8 = !wide && fits(8) && !long_slices;
  AttendPlan p{4, 1, 0};
  if (asked > 0) {
    p.splits = explicit_splits(ctx);
  } else if (units <= 128) {
    const int most = (int)(256 / units) < 16 ? (int)(256 / units) : 16;
    const int aim = typical > 24 * 7 ? (typical + 23) / 24 : 7, n = aim < most ? aim : most;
    const bool bf16 = ctx->cfg.dtype == GKV_BF16;
    const int enough = n == 2 ? (wide ? 12 : bf16 ? 40 : 30) : wide ? 9 : keys == 32 ? 10 : 18;
    const int prompt = n == 2 && !wide ? (bf16 ? 64 : 48) : 2 * enough;
    if (n == most && typical >= enough && typical >= 20 * n && may_have_8) {
      p = AttendPlan{8, most, 8};
    } else if (typical >= enough || full >= prompt) {
      // units of ordinary length stay whole where that is the better, and prompts much longer are cut
      p.iters = typical >= enough ? 4 * ((typical + 4 * n - 1) / (4 * n)) : typical > 8 ? (typical + 3) / 4 * 4 : 8;
      p.splits = (full + p.iters - 1) / p.iters < most ? (full + p.iters - 1) / p.iters : most;
    }
    if (p.splits < 2) p = AttendPlan{4, 1, 0};
  }
  const int slices = (int)((int64_t)d.cap * 2 * row_bytes / 8192);    // in units of 8 KiB, at full capacity
  const bool more = p.splits == 1 ? (units <= 256 && slices >= (keys == 32 ? 12 : 16)) || (units > 512 && slices >= 64)
                                  : asked > 0 && slices / p.splits >= 48;
  if (more && may_have_8) p.waves = 8;
  if (ctx->attend_waves > 0) p.waves = fits(ctx->attend_waves) ? ctx->attend_waves : 4;
  return p;
}

static size_t ws_stats_bytes(const gkv_ctx* ctx) {
  return (size_t)ctx->dims.w * ctx->dims.L * ctx->dims.B * ctx->dims.Hq * sizeof(float2);
}

// Split-K partials for `splits` workgroups per unit (none when a unit is not split).
static size_t ws_partials_bytes(const gkv_ctx* ctx, int splits) {
  if (!ctx->mfma_shape || splits <= 1) return 0;
  const size_t units = (size_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hkv;
  return units * splits * ctx->dims.g * (ctx->dims.d + 2) * sizeof(float);
}

// Sets for the library's own cuts (attend_plan cuts up to 128 units); the set of "attend_splits" follows them.
static int auto_sets(const gkv_ctx* ctx) {
  return ctx->mfma_shape && (int64_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hkv <= 128 ? GKV_SPLIT_SETS : 0;
}
static size_t ws_ticket_bytes(const gkv_ctx* ctx) {
  const size_t units = (size_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hkv;
  return gkv_align256(units * (auto_sets(ctx) + 1) * GKV_TICKETS * 4);
}

GkvWorkspace gkv_carve_workspace(const gkv_ctx* ctx, void* base, int split_set) {
  GkvWorkspace w;
  char* p = (char*)base;
  const size_t units = (size_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hkv;
  w.split_ticket = (int32_t*)p + split_set * units * GKV_TICKETS; p += ws_ticket_bytes(ctx);
  w.state_ticket = (int32_t*)p; p += gkv_align256((size_t)ctx->dims.L * ctx->dims.B * 4);
  w.stats = (float2*)p; p += gkv_align256(ws_stats_bytes(ctx));
  w.partials = (float*)(p + split_set * ws_partials_bytes(ctx, ctx->ws_auto_splits));
  return w;
}

extern "C" gkv_status gkv_workspace_bytes(gkv_ctx* ctx, size_t* out_bytes) {
  if (!ctx || !out_bytes) return GKV_ERR_INVALID_ARG;
  // the workspace is sized for the split counts in force now: the decode call refuses a larger one
  // that was asked for, and does without one of its own choice
  ctx->ws_splits = explicit_splits(ctx);
  ctx->ws_auto_splits = ctx->mfma_shape && !ctx->force_generic ? attend_plan(ctx, 0).splits : 1;
  const size_t automatic = auto_sets(ctx) * ws_partials_bytes(ctx, ctx->ws_auto_splits);
  *out_bytes = ws_ticket_bytes(ctx) + gkv_align256((size_t)ctx->dims.L * ctx->dims.B * 4) +
               gkv_align256(ws_stats_bytes(ctx)) +
               gkv_align256(automatic + ws_partials_bytes(ctx, ctx->ws_splits)) + 256;
  return GKV_OK;
}

extern "C" gkv_status gkv_workspace_init(gkv_ctx* ctx, void* workspace, void* stream) {
  if (!ctx) return GKV_ERR_INVALID_ARG;
  if (!workspace) return GKV_ERR_WORKSPACE;
  const size_t n = (ws_ticket_bytes(ctx) + gkv_align256((size_t)ctx->dims.L * ctx->dims.B * 4)) / 4;   // both ticket arrays
  if (gkv_launch_fill_zero((hipStream_t)stream, (int32_t*)workspace, n) != hipSuccess) return GKV_ERR_HIP;
  ctx->split_ws = workspace;
  return GKV_OK;
}

extern "C" gkv_status gkv_cache_bytes(const gkv_config* cfg, int32_t rows, int32_t score_elem_bytes,
                                      size_t* kv_bytes, size_t* score_bytes) {
  if (!cfg || rows < 0 || score_elem_bytes < 1) return GKV_ERR_INVALID_ARG;
  if (cfg->dtype != GKV_F32 && cfg->dtype != GKV_BF16) return GKV_ERR_INVALID_ARG;
  const size_t esz = cfg->dtype == GKV_F32 ? 4 : 2;
  const size_t heads = (size_t)cfg->n_layers * cfg->batch * cfg->n_kv_heads;
  if (kv_bytes) *kv_bytes = heads * (size_t)rows * cfg->head_dim * esz * 2;            // K and V
  if (score_bytes) {
    const int64_t n = (int64_t)cfg->budget - cfg->window;
    *score_bytes = heads * (size_t)(n > 0 ? n : 0) * (size_t)score_elem_bytes;
  }
  return GKV_OK;
}

extern "C" int64_t gkv_k_offset(const gkv_config* cfg, int32_t row, int32_t channel, int32_t n_tiled) {
  if (!cfg || row < 0 || channel < 0 || channel >= cfg->head_dim || n_tiled < 0) return -1;
  const int epc = cfg->dtype == GKV_F32 ? 4 : 8;
  const int64_t d = cfg->head_dim;
  if (row >= (n_tiled & ~15)) return (int64_t)row * d + channel;
  return (int64_t)(row / 16) * 16 * d + (int64_t)(channel / epc) * (16 * epc) + (row % 16) * epc + channel % epc;
}

extern "C" gkv_status gkv_set_param(gkv_ctx* ctx, const char* name, int32_t value) {
  if (!ctx || !name) return GKV_ERR_INVALID_ARG;
  if (!strcmp(name, "attend_splits")) {
    if (value < 0 || value > 64) return GKV_ERR_INVALID_ARG;
    ctx->attend_splits = value;
    return GKV_OK;
  }
  if (!strcmp(name, "attend_tile")) {
    if (value != 16 && value != 32) return GKV_ERR_INVALID_ARG;
    ctx->attend_tile = value;
    return GKV_OK;
  }
  if (!strcmp(name, "force_generic")) { ctx->force_generic = value != 0; return GKV_OK; }
  if (!strcmp(name, "compact_ppt")) {
    if (value != 4 && value != 8 && value != 16) return GKV_ERR_INVALID_ARG;
    ctx->compact_ppt = value;
    return GKV_OK;
  }
  if (!strcmp(name, "attend_waves")) {
    if (value != 0 && value != 4 && value != 8 && value != 16) return GKV_ERR_INVALID_ARG;
    if (value * ctx->dims.g * 132 * 4 + value * 128 + (32 + 16 * ctx->dims.g) * 16 > 65000) return GKV_ERR_SHAPE;
    ctx->attend_waves = value;
    return GKV_OK;
  }
  if (!strcmp(name, "evict_fuse_global")) { ctx->fuse_global = value != 0; return GKV_OK; }
  if (!strcmp(name, "evict_fuse_select")) { ctx->fuse_select = value != 0; return GKV_OK; }
  if (!strcmp(name, "score_reuse_stats")) { ctx->reuse_stats = value != 0; return GKV_OK; }
  return GKV_ERR_INVALID_ARG;
}

// ---- device-side step counter ----------------------------------------------------------------------
extern "C" gkv_status gkv_set_step_base(gkv_ctx* ctx, const int32_t* d_step_base) {
  if (!ctx) return GKV_ERR_INVALID_ARG;
  ctx->dims.step_base = d_step_base;
  for (int i = 0; i < ctx->dims.w; ++i) ctx->stats_step[i] = -1;    // recorded steps were counted from another origin
  return GKV_OK;
}

extern "C" gkv_status gkv_advance_step_base(gkv_ctx* ctx, int32_t delta, void* stream) {
  if (!ctx || !ctx->dims.step_base) return GKV_ERR_INVALID_ARG;
  return gkv_launch_add_int((hipStream_t)stream, const_cast<int32_t*>(ctx->dims.step_base), delta) == hipSuccess
             ? GKV_OK : GKV_ERR_HIP;
}

// ---- the five calls -----------------------------------------------------------------------------
static bool use_mfma_redundancy(const gkv_ctx* ctx) { return ctx->mfma_redundancy && !ctx->force_generic; }
// The matrix-core decode and window-score kernels move 16-byte pieces; callers are asked for 16-byte
// aligned base pointers, and others fall back to the plain kernels.
static bool use_mfma(const gkv_ctx* ctx, std::initializer_list<const void*> ptrs) {
  if (!ctx->mfma_shape || ctx->force_generic) return false;
  uintptr_t bits = 0;
  for (const void* p : ptrs) bits |= (uintptr_t)p;
  return (bits & 15) == 0;
}
static gkv_status check_len(const gkv_ctx* ctx, int32_t len_max_host, bool appending) {
  if (len_max_host < 0) return GKV_ERR_INVALID_ARG;
  if (len_max_host > ctx->dims.cap || (appending && len_max_host >= ctx->dims.cap)) return GKV_ERR_OVERFLOW;
  return GKV_OK;
}
static inline gkv_status hip_status(hipError_t e) { return e == hipSuccess ? GKV_OK : GKV_ERR_HIP; }

// What distinguishes calls that follow each other on the GPU from calls that may overlap.  false: unknown
// (the per-thread default stream is another stream in every thread).
static bool stream_key(hipStream_t stream, GkvStreamKey* key) {
  if (stream == hipStreamPerThread) return false;
  *key = GkvStreamKey{stream, 0};
  if (stream == nullptr) return true;                    // the legacy stream cannot be captured
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(stream, &status, &id) != hipSuccess) { (void)hipGetLastError(); return false; }
  if (status == hipStreamCaptureStatusInvalidated) return false;
  if (status == hipStreamCaptureStatusActive) key->capture = id + 1;
  return true;
}

// Host bookkeeping of the statistics ring: which decode step each slot's statistics belong to,
// and for which buffers.  Calls on one K cache are ordered by the caller (each appends to it), so "enqueued"
// is as good as "written".  Calls on another cache and another stream need not be: what they write to
// the statistics ring may land at any time, and from then on nothing is taken from it.
static void note_stats(gkv_ctx* ctx, int32_t step, bool written, const void* ws, const void* K, const void* qwin,
                       hipStream_t stream) {
  const int w = ctx->dims.w;
  GkvStreamKey key;
  const bool known = stream_key(stream, &key);
  const bool same_stream = known && key.stream == ctx->stats_key.stream && key.capture == ctx->stats_key.capture;
  ctx->stats_key = known ? key : GkvStreamKey{hipStreamPerThread, 0};   // never equal to a known one
  if (ctx->stats_K && K != ctx->stats_K && !same_stream) ctx->stats_mixed = true;
  if (ws != ctx->stats_ws || K != ctx->stats_K || qwin != ctx->stats_qwin) {
    for (int i = 0; i < w; ++i) ctx->stats_step[i] = -1;
    ctx->stats_ws = ws; ctx->stats_K = K; ctx->stats_qwin = qwin;
  }
  ctx->stats_step[step % w] = written ? step : -1;
}
static bool stats_cover_window(const gkv_ctx* ctx, int32_t step, const void* ws, const void* K, const void* qwin) {
  const int w = ctx->dims.w;
  if (!ctx->reuse_stats || ctx->stats_mixed || !ws || ws != ctx->stats_ws || K != ctx->stats_K || qwin != ctx->stats_qwin) return false;
  if (step + 1 < w) return false;
  for (int k = 0; k < w; ++k) {
    const int t = step - w + 1 + k;
    if (ctx->stats_step[t % w] != t) return false;
  }
  return true;
}

// The set of the stream a cut decode call goes to, or -1: no set left, or not this context's workspace.
static int split_set(gkv_ctx* ctx, const void* workspace, hipStream_t stream) {
  GkvStreamKey key;
  if (workspace != ctx->split_ws || !stream_key(stream, &key)) return -1;
  for (int i = 0; i < ctx->n_split_keys; ++i)
    if (ctx->split_key[i].stream == key.stream && ctx->split_key[i].capture == key.capture) return i;
  if (ctx->n_split_keys == GKV_SPLIT_SETS) return -1;
  ctx->split_key[ctx->n_split_keys] = key;
  return ctx->n_split_keys++;
}

extern "C" gkv_status gkv_attend_decode(gkv_ctx* ctx, const void* q, const void* k_new, const void* v_new,
                                        void* K, void* V, int32_t* pos, int32_t step, void* qwin,
                                        const int32_t* d_state, int32_t len_max_host, void* out,
                                        void* workspace, void* stream) {
  if (!ctx || !q || !K || !V || !pos || !qwin || !d_state || !out || step < 0) return GKV_ERR_INVALID_ARG;
  if ((k_new == nullptr) != (v_new == nullptr)) return GKV_ERR_INVALID_ARG;
  if (!workspace) return GKV_ERR_WORKSPACE;
  gkv_status st = check_len(ctx, len_max_host, k_new != nullptr);
  if (st != GKV_OK) return st;
  AttendArgs a{q, k_new, v_new, K, V, pos, step, qwin, d_state, out, gkv_carve_workspace(ctx, workspace), 1,
               ctx->attend_tile, 1, 0, 4, 0};
  {
    const size_t slot_bytes = (size_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hq * ctx->dims.d * ctx->esz;
    a.copy_q = (const char*)q != (const char*)qwin + (size_t)(step % ctx->dims.w) * slot_bytes;
  }
  GkvLaunch ln{ctx, GKV_K_ATTEND, (hipStream_t)stream};
  if (use_mfma(ctx, {q, k_new, v_new, K, V, qwin, out})) {
    AttendPlan plan = attend_plan(ctx, ctx->attend_splits);
    int set = auto_sets(ctx);                                       // "attend_splits"
    if (ctx->attend_splits > 0) {
      if (plan.splits > ctx->ws_splits) return GKV_ERR_WORKSPACE;   // partials would not fit the workspace as sized
    } else if (plan.splits > 1) {
      set = plan.splits > ctx->ws_auto_splits ? -1 : split_set(ctx, workspace, (hipStream_t)stream);
      if (set < 0) { plan = attend_plan(ctx, 1); set = 0; }         // not cut
    }
    a.ws = gkv_carve_workspace(ctx, workspace, set);
    a.waves = plan.waves; a.splits = plan.splits; a.split_iters = plan.iters;
    // An appending step leaves (max, sum) of every query head's softmax in the ring slot
    // of this step; the window score can then skip its own pass over the keys for them.
    a.write_stats = k_new != nullptr;
    note_stats(ctx, step, a.write_stats != 0, workspace, K, qwin, (hipStream_t)stream);
    return hip_status(gkv_launch_attend_mfma(ln, ctx->dims, ctx->cfg.dtype, a));
  }
  note_stats(ctx, step, false, workspace, K, qwin, (hipStream_t)stream);
  return hip_status(gkv_launch_attend_generic(ln, ctx->dims, ctx->cfg.dtype, a));
}

extern "C" gkv_status gkv_score_window(gkv_ctx* ctx, const void* qwin, const void* K, const int32_t* d_state,
                                       int32_t step, int32_t len_max_host, float* S,
                                       void* workspace, void* stream) {
  if (!ctx || !qwin || !K || !d_state || !S || step < 0) return GKV_ERR_INVALID_ARG;
  gkv_status st = check_len(ctx, len_max_host, false);
  if (st != GKV_OK) return st;
  ScoreArgs a{qwin, K, d_state, step, S, nullptr};
  GkvLaunch ln{ctx, GKV_K_SCORE, (hipStream_t)stream};
  if (use_mfma(ctx, {qwin, K})) {
    // Under the causal reading of Eq. 1 a window row's softmax runs over exactly the keys its
    // query attended to when it was decoded: if the last w decode calls on these buffers were the
    // window's steps, their recorded (max, sum) are the row statistics and one pass suffices.
    if (stats_cover_window(ctx, step, workspace, K, qwin)) a.stats = gkv_carve_workspace(ctx, workspace).stats;
    return hip_status(gkv_launch_score_mfma(ln, ctx->dims, ctx->cfg.dtype, a, len_max_host));
  }
  return hip_status(gkv_launch_score_generic(ln, ctx->dims, ctx->cfg.dtype, a));
}

extern "C" gkv_status gkv_global_update(gkv_ctx* ctx, const float* S, const float* F_hist,
                                        const int32_t* d_state, int32_t step, int32_t len_max_host,
                                        float* F_out, void* stream) {
  if (!ctx || !S || !F_hist || !d_state || !F_out || step < 0) return GKV_ERR_INVALID_ARG;
  gkv_status st = check_len(ctx, len_max_host, false);
  if (st != GKV_OK) return st;
  GkvLaunch ln{ctx, GKV_K_GLOBAL, (hipStream_t)stream};
  return hip_status(gkv_launch_global_update(ln, ctx->dims, S, F_hist, d_state, step, F_out));
}

extern "C" gkv_status gkv_select_topk(gkv_ctx* ctx, const float* F, const int32_t* d_state, int32_t step,
                                      int32_t len_max_host, int32_t* keep_idx, void* workspace, void* stream) {
  (void)workspace;
  if (!ctx || !F || !d_state || !keep_idx || step < 0) return GKV_ERR_INVALID_ARG;
  gkv_status st = check_len(ctx, len_max_host, false);
  if (st != GKV_OK) return st;
  GkvLaunch ln{ctx, GKV_K_TOPK, (hipStream_t)stream};
  return hip_status(gkv_launch_select_topk(ln, ctx->dims, F, d_state, step, keep_idx));
}

extern "C" gkv_status gkv_compact(gkv_ctx* ctx, const int32_t* keep_idx, const float* F, void* K, void* V,
                                  float* F_hist, int32_t* pos, int32_t* d_state, int32_t step,
                                  void* workspace, void* stream) {
  if (!ctx || !keep_idx || !F || !K || !V || !F_hist || !pos || !d_state || step < 0) return GKV_ERR_INVALID_ARG;
  if (F == F_hist) return GKV_ERR_INVALID_ARG;
  GkvLaunch ln{ctx, GKV_K_COMPACT, (hipStream_t)stream};
  // with a workspace the last compaction workgroup of a (layer, sequence) rewrites its state
  // record; without one a second small launch does
  int32_t* ticket = workspace ? gkv_carve_workspace(ctx, workspace).state_ticket : nullptr;
  return hip_status(gkv_launch_compact(ln, ctx->dims, ctx->esz, keep_idx, F, K, V, F_hist, pos, d_state, step, ticket));
}

extern "C" gkv_status gkv_evict(gkv_ctx* ctx, const void* qwin, void* K, void* V, float* F_hist, int32_t* pos,
                                int32_t* d_state, int32_t step, int32_t len_max_host,
                                float* S, float* F, int32_t* keep_idx, void* workspace, void* stream) {
  if (!ctx || !qwin || !K || !V || !F_hist || !pos || !d_state || !S || !F || !keep_idx || step < 0)
    return GKV_ERR_INVALID_ARG;
  if (F == F_hist) return GKV_ERR_INVALID_ARG;
  gkv_status st = check_len(ctx, len_max_host, false);
  if (st != GKV_OK) return st;
  st = gkv_score_window(ctx, qwin, K, d_state, step, len_max_host, S, workspace, stream);
  if (st != GKV_OK) return st;
  if (ctx->fuse_select || ctx->fuse_global) {
    // the global score is formed at the head of the selection kernel (same arithmetic as
    // gkv_global_update, F written as well): one launch less per compression
    GkvLaunch ln{ctx, GKV_K_TOPK, (hipStream_t)stream};
    st = hip_status(gkv_launch_update_and_select(ln, ctx->dims, S, F_hist, d_state, step, F, keep_idx));
    if (st != GKV_OK) return st;
    return gkv_compact(ctx, keep_idx, F, K, V, F_hist, pos, d_state, step, workspace, stream);
  }
  st = gkv_global_update(ctx, S, F_hist, d_state, step, len_max_host, F, stream);
  if (st != GKV_OK) return st;
  st = gkv_select_topk(ctx, F, d_state, step, len_max_host, keep_idx, workspace, stream);
  if (st != GKV_OK) return st;
  return gkv_compact(ctx, keep_idx, F, K, V, F_hist, pos, d_state, step, workspace, stream);
}

// ---- compression for callers that cannot allocate ---------------------------------------------
// The intermediates of one compression (S, F, keep_idx) live in a fixed array in device memory
// that every GPU the library runs on holds until the process ends.  In host code the array's
// name is only a handle for hipGetSymbolAddress; the address that kernels and copies use is the
// one that call returns, looked up once per device.
static __device__ __align__(256) unsigned char scratch[GKV_STATIC_SCRATCH_BYTES];

static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[64] = {};

static gkv_status static_scratch_of_current_device(char** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return GKV_ERR_HIP;
  if (dev < 0 || dev >= 64) return GKV_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GKV_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = (char*)g_scratch_ptr[dev];
  return GKV_OK;
}

extern "C" gkv_status gkv_evict_static(gkv_ctx* ctx, const void* qwin, void* K, void* V, float* F_hist,
                                       int32_t* pos, int32_t* d_state, int32_t step, int32_t len_max_host,
                                       void* workspace, void* stream) {
  if (!ctx || !qwin || !K || !V || !F_hist || !pos || !d_state || step < 0) return GKV_ERR_INVALID_ARG;
  const size_t units = (size_t)ctx->dims.L * ctx->dims.B * ctx->dims.Hkv;
  const size_t score_bytes = gkv_align256(units * ctx->dims.cap * sizeof(float));
  const size_t keep_bytes = gkv_align256(units * (size_t)(ctx->dims.b - ctx->dims.w) * sizeof(int32_t));
  if (2 * score_bytes + keep_bytes > (size_t)GKV_STATIC_SCRATCH_BYTES) return GKV_ERR_SCRATCH;
  char* base = nullptr;
  gkv_status st = static_scratch_of_current_device(&base);
  if (st != GKV_OK) return st;
  float* S = (float*)base;
  float* F = (float*)(base + score_bytes);
  int32_t* keep_idx = (int32_t*)(base + 2 * score_bytes);
  return gkv_evict(ctx, qwin, K, V, F_hist, pos, d_state, step, len_max_host, S, F, keep_idx, workspace, stream);
}

extern "C" gkv_status gkv_redundancy_combine(gkv_ctx* ctx, const void* K, const int32_t* d_state, int32_t step,
                                             int32_t len_max_host, const float* F, float lambda, float tau,
                                             float eps, int32_t n_recent, float* R_norm, float* F_sel,
                                             void* workspace, void* stream) {
  (void)workspace;
  if (!ctx || !K || !d_state || !F || !R_norm || !F_sel || step < 0) return GKV_ERR_INVALID_ARG;
  if (!(lambda >= 0.f && lambda <= 1.f) || !(tau > -1.5f && tau < 1.5f) || !(eps >= 0.f) || n_recent < 0)
    return GKV_ERR_INVALID_ARG;
  if (F == F_sel) return GKV_ERR_INVALID_ARG;
  gkv_status st = check_len(ctx, len_max_host, false);
  if (st != GKV_OK) return st;
  GkvLaunch ln{ctx, GKV_K_REDUNDANCY, (hipStream_t)stream};
  return hip_status(gkv_launch_redundancy(ln, ctx->dims, ctx->cfg.dtype, use_mfma_redundancy(ctx),
                                          !ctx->mfma_redundancy && use_mfma(ctx, {K}), K, d_state, step, F,
                                          lambda, tau, eps, n_recent, R_norm, F_sel));
}

extern "C" gkv_status gkv_pool_scores(gkv_ctx* ctx, const float* F, const int32_t* d_state, int32_t step,
                                      int32_t kernel, float* F_out, void* stream) {
  if (!ctx || !F || !d_state || !F_out || step < 0 || kernel < 1 || F == F_out) return GKV_ERR_INVALID_ARG;
  GkvLaunch ln{ctx, -1, (hipStream_t)stream};
  return hip_status(gkv_launch_pool_scores(ln, ctx->dims, F, d_state, step, kernel, F_out));
}

extern "C" gkv_status gkv_evicted_positions(gkv_ctx* ctx, const int32_t* keep_idx, const int32_t* pos,
                                            const int32_t* d_state, int32_t step, int32_t* evicted, void* stream) {
  if (!ctx || !keep_idx || !pos || !d_state || !evicted || step < 0) return GKV_ERR_INVALID_ARG;
  GkvLaunch ln{ctx, -1, (hipStream_t)stream};
  return hip_status(gkv_launch_evicted_positions(ln, ctx->dims, keep_idx, pos, d_state, step, evicted));
}

// ---- profiling API ------------------------------------------------------------------------------
extern "C" gkv_status gkv_profile_enable(gkv_ctx* ctx, int32_t on) {
  if (!ctx || !ctx->prof) return GKV_ERR_INVALID_ARG;
  ctx->prof->on = on != 0;
  return GKV_OK;
}
extern "C" gkv_status gkv_profile_read(gkv_ctx* ctx, int32_t kernel_id, double* total_ms, int64_t* launches) {
  if (!ctx || !ctx->prof || kernel_id < 0 || kernel_id >= GKV_K_COUNT) return GKV_ERR_INVALID_ARG;
  profile_drain(ctx->prof, kernel_id);
  if (total_ms) *total_ms = ctx->prof->done_ms[kernel_id];
  if (launches) *launches = ctx->prof->done_n[kernel_id];
  return GKV_OK;
}
extern "C" gkv_status gkv_profile_reset(gkv_ctx* ctx) {
  if (!ctx || !ctx->prof) return GKV_ERR_INVALID_ARG;
  for (int k = 0; k < GKV_K_COUNT; ++k) {
    profile_drain(ctx->prof, k);
    ctx->prof->done_ms[k] = 0;
    ctx->prof->done_n[k] = 0;
  }
  return GKV_OK;
}
