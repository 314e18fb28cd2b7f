// C-ABI entry points of libckv: argument validation on the host, then kernel launches.
// Nothing here allocates or synchronises; every entry point either enqueues all of its kernels on
// the caller's stream or returns an error before the first launch.
#include <float.h>
#include <math.h>

#include <atomic>
#include <chrono>
#include <mutex>

#include "ckv_internal.h"

namespace ckv {

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

ckv_status validate(const ckv_params *p) {
  if (!p) return CKV_EINVAL;
  if (p->batch < 1 || p->n_kv_heads < 1 || p->n_q_heads < 1) return CKV_EINVAL;
  if (p->n_q_heads % p->n_kv_heads) return CKV_EINVAL;
  if (p->seq_len < 1 || p->window < 1 || p->window > p->seq_len) return CKV_EINVAL;
  if (p->n_layers < 1 || p->layer < 0 || p->layer >= p->n_layers) return CKV_EINVAL;
  if (p->dtype != CKV_F32 && p->dtype != CKV_BF16) return CKV_EINVAL;
  if (!(p->softmax_scale >= 0.0f) || isinf(p->softmax_scale)) return CKV_EINVAL;
  if (p->pool != CKV_POOL_NONE && p->pool != CKV_POOL_AVG && p->pool != CKV_POOL_MAX) return CKV_EINVAL;
  if (p->pool != CKV_POOL_NONE && (p->pool_kernel < 1 || p->pool_kernel > 63 || p->pool_kernel % 2 == 0))
    return CKV_EINVAL;
  if (p->budget_per_kv_head < p->window) return CKV_EINVAL;
  if (p->flags & ~(uint32_t)(CKV_FLAG_VALUE_NORM | CKV_FLAG_GROUP_MASS)) return CKV_EINVAL;
  if (p->head_dim < 1) return CKV_EINVAL;
  const int64_t b_tot = (int64_t)p->budget_per_kv_head * p->n_kv_heads;
  int64_t need = b_tot - (int64_t)(p->n_kv_heads - 1) * p->window;
  if (need > p->seq_len) need = p->seq_len;
  if (p->cap < need) return CKV_EINVAL;
  for (int i = 0; i < 3; ++i)
    if (p->q_stride[i] < 0 || p->k_stride[i] < 0 || p->v_stride[i] < 0) return CKV_EINVAL;
  // rows must hold head_dim contiguous elements and start 16-byte aligned for the 128-bit loads
  const int64_t per16 = p->dtype == CKV_BF16 ? 8 : 4;
  if (p->q_stride[2] < p->head_dim || p->k_stride[2] < p->head_dim || p->v_stride[2] < p->head_dim)
    return CKV_EINVAL;
  for (int i = 0; i < 3; ++i)
    if (p->q_stride[i] % per16 || p->k_stride[i] % per16 || p->v_stride[i] % per16) return CKV_EINVAL;
  if (p->head_dim != 64 && p->head_dim != 128) return CKV_EUNSUPPORTED;
  if (p->window > kMaxWindowTiles * kTile) return CKV_EUNSUPPORTED;
  if ((int64_t)p->batch * p->n_kv_heads > 65535) return CKV_EUNSUPPORTED;  // grid.y
  if (p->seq_len > (1 << 24)) return CKV_EUNSUPPORTED;
  // the staged scan addresses the 32 rows of a key tile with 32-bit offsets
  if (p->k_stride[2] * (int64_t)(p->dtype == CKV_BF16 ? 2 : 4) * kTile >= ((int64_t)1 << 31)) return CKV_EUNSUPPORTED;
  if ((int64_t)p->n_q_heads * p->seq_len >= (1 << 29)) return CKV_EUNSUPPORTED;  // scores of one batch element: < 2 GiB
  return CKV_OK;
}

// Keys per wave: the split of the key axis. One workgroup per CU runs at full speed (bf16: its four waves sweep long ranges, since
// nothing overlaps a workgroup's set-up; f32: two would fit a CU, but they halve each other's rate), so what counts is full
// rounds of that many: the least rounds x (keys + set-up), set-up being worth about 192 keys of a bf16 sweep and a tile of an f32
// one. bf16 ranges beyond 128 keys are whole four-tile pipeline rounds. The row partials stay within 1 MiB or what the plain
// even split needs, whichever is more, so that a caller's or the library's fixed scratch goes as far as it did.
// Measured against the even split alone, us: bf16, both passes and tables, 97280 keys, 24 units 324 -> 226 (264 workgroups
// became 240), 51200 keys, 40 units 328 -> 210, 5003 keys, 96 units 91.5 -> 65.8; f32 (even split for 2048 workgroups, at least 64
// keys), both passes: 1024 keys, 4/4 heads of 64 14.2 -> 10.4, 8192 keys, 32/32 heads of 64 51.7 -> 29.0, 4099 keys, 32/8 heads of
// 128 60.0 -> 42.0. (Rounds of 512 workgroups for f32: 10.4, 35.9, 41.7, and slower than the even split in 13 of 70 shapes, by up
// to 23 %: 1244 keys, 32/8 heads of 128 24.4 -> 30.1 with 320 workgroups, 21.6 with 160.)
static int64_t split_keys(const Shape &s, bool bf16, int64_t units) {
  const int64_t resident = kComputeUnits;
  const int64_t set_up = bf16 ? 192 : kTile, waves = kScoreWaves * (bf16 ? (int64_t)kComputeUnits : 2048);
  const auto workgroups = [&](int64_t kpw) { return units * ((s.T + kScoreWaves * kpw - 1) / (kScoreWaves * kpw)); };
  int64_t plain = ((int64_t)s.T * units + waves - 1) / waves;
  const int64_t quantum = bf16 && plain > 4 * kTile ? 4 * kTile : kTile;
  plain = (plain + quantum - 1) / quantum * quantum;
  if (plain < 2 * kTile) plain = 2 * kTile;
  if (plain > 4096) plain = 4096;
  const int64_t part_bytes = (int64_t)s.NQ * kTile * (int64_t)sizeof(float2);  // per workgroup
  const int64_t most = workgroups(plain) * part_bytes > (1 << 20) ? workgroups(plain) : (1 << 20) / part_bytes;
  int64_t best = plain, best_cost = INT64_MAX;
  for (int64_t kpw = bf16 ? 2 * kTile : kTile; kpw <= 4096; kpw += bf16 && kpw >= 4 * kTile ? 4 * kTile : kTile) {
    const int64_t n = workgroups(kpw);
    const int64_t cost = (n + resident - 1) / resident * (kpw + set_up);
    if (n <= most && cost <= best_cost) {
      best = kpw;
      best_cost = cost;
    }
    if (kpw >= s.T) break;
  }
  // bf16, no round less: the even split stays (shorter ranges for more of a workgroup's waves: 4096 keys, 512 units 186 -> 192 us)
  const auto rounds = [&](int64_t kpw) { return (workgroups(kpw) + resident - 1) / resident; };
  return bf16 && rounds(best) >= rounds(plain) ? plain : best;
}

void derive(const ckv_params *p, Shape *s) {
  s->Bz = p->batch;
  s->Hq = p->n_q_heads;
  s->Hkv = p->n_kv_heads;
  s->G = s->Hq / s->Hkv;
  s->d = p->head_dim;
  s->T = p->seq_len;
  s->W = p->window;
  s->P = s->T - s->W;
  s->esize = p->dtype == CKV_BF16 ? 2 : 4;
  s->WT = (s->W + kTile - 1) / kTile;
  s->n_tiles = s->G * s->WT;
  // Tiles a wave keeps in registers, whole heads only: eight for bf16 (a wave alone on its SIMD has 512
  // registers, and the matrix cores read operands from either half), four for f32 rows of 256 bytes, two for f32 rows of
  // 512 bytes where that leaves every SIMD two tile products (us, both passes and tables, one tile / two: 4099 keys, 32/8
  // heads 55.1 / 45.7, 16384 keys, 16/8 heads 64.8 / 54.5, but 700 keys 20.6 / 27.6; with up to four 59.7 for the first)
  // and pads no tile, else one head's tiles.
  const int64_t products = (int64_t)s->Bz * s->Hkv * s->n_tiles * ((s->T + kTile - 1) / kTile);
  const bool two = s->n_tiles % 2 == 0 && products >= 2 * kScoreWaves * kComputeUnits;
  const int budget_tiles = p->dtype == CKV_BF16 ? kMaxQTiles : s->d * s->esize <= 256 ? kMaxQTilesF32 : two ? 2 : 1;
  const int per_wave_max = budget_tiles >= s->WT ? (budget_tiles / s->WT) * s->WT : s->WT;
  s->n_groups = (s->n_tiles + per_wave_max - 1) / per_wave_max;
  int nq = (s->n_tiles + s->n_groups - 1) / s->n_groups;
  nq = (nq + s->WT - 1) / s->WT * s->WT;
  s->NQ = nq;
  s->n_groups = (s->n_tiles + nq - 1) / nq;
  const int64_t kpw = split_keys(*s, p->dtype == CKV_BF16, (int64_t)s->Bz * s->Hkv * s->n_groups);
  s->keys_per_wave = (int)kpw;
  s->n_chunks = (int)((s->T + kScoreWaves * kpw - 1) / (kScoreWaves * kpw));
  s->scale = p->softmax_scale > 0.0f ? p->softmax_scale : 1.0f / sqrtf((float)s->d);
}

int vnorm_blocks_per_unit(const Shape &s) {
  return (s.T + kVnormRows - 1) / kVnormRows;
}

// Four more waves per workgroup of the bf16 scan, where its own leave them registers (up to four query tiles per wave), one
// workgroup takes all query tiles of its keys, its range is whole blocks of the norms' sums, and the launch has one workgroup per CU
// at most. us, separate / beside the scan: 10006 keys, batch 4, four calls 80.6 / 71.2; 4096 keys, 32/32 heads 51.9 / 40.6;
// 20011 keys, batch 2 86.2 / 73.9; 32768, batch 16, where both reads are bound by HBM, 587 / 586. Over 200 shapes of head sizes 64 and
// 128, one to four tiles: 0.87 in the geometric mean, none slower by more than 1 %. More workgroups than CUs, where a workgroup of
// eight waves keeps a second one of four (rows of 128 bytes) off its CU and the launch's end weighs twice: 0.90 to 1.32
// of the time (us: 1024 workgroups, 2888 keys of 64 354 / 467, 4733 531 / 668; 384, 33000 keys of 64 379 / 422, 14629 of 128 467 / 518;
// 1024 of 128, 1192 keys 391 / 360; no line by size or fill parts them).
bool norms_in_scan(const ckv_params *p, const Shape &s, bool lse_given) {
  return (p->flags & CKV_FLAG_VALUE_NORM) && !lse_given && p->dtype == CKV_BF16 && s.NQ <= kMaxQTilesNorms && s.n_groups == 1 &&
         kScoreWaves * s.keys_per_wave % kVnormRows == 0 && (int64_t)s.Bz * s.Hkv * s.n_chunks <= kComputeUnits;
}

// One launch for both passes where a wave's range is no longer than its ring of key tiles, so that the keys stay in LDS between
// them, and every workgroup has a CU of its own (more of them would wait for ones that start when they end). 0.80 to 0.98 of the two
// launches' time per layer over twelve shapes of 1000 to 65536 keys (scan_short_kernel). Without value norms, whose ratio needs a
// unit's sum of them, too.
bool one_launch(const ckv_params *p, const Shape &s) {
  return p->dtype == CKV_BF16 && s.n_groups == 1 && s.keys_per_wave <= kRing * kTile && (int64_t)s.Bz * s.Hkv * s.n_chunks <= kComputeUnits;
}

// Even. The upper bits are those of a negative NaN, which no sum, position or key ends up as; the rest counts the process's launches
// from the monotonic clock's value at the first of them, in steps that touch all bits.
tag_t launch_tag() {
  static std::atomic<uint64_t> count{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count()};
  const uint64_t mixed = count.fetch_add(1, std::memory_order_relaxed) * 0x9E3779B97F4A7C15ull;
  return 0xFFF8000000000000ull | mixed >> 14 << 1;
}

void layout(const ckv_params *p, const Shape &s, Workspace *w) {
  const size_t units = (size_t)s.Bz * s.Hkv;
  size_t off = 0;
  w->part_off = off;
  w->part_bytes = units * (size_t)s.n_groups * s.NQ * kTile * s.n_chunks * sizeof(float2);
  off = align256(off + w->part_bytes);
  w->lse_off = off;
  w->lse_bytes = (size_t)s.Bz * s.Hq * s.W * sizeof(float);
  off = align256(off + w->lse_bytes);
  w->vsum_off = off;
  w->vsum_bytes = (p->flags & CKV_FLAG_VALUE_NORM) ? units * vnorm_blocks_per_unit(s) * sizeof(float) : 0;
  off = align256(off + w->vsum_bytes);
  w->select_off = off;
  w->select_bytes = select_workspace_bytes(p, s);
  // Asked of every call is what the shape alone decides, so that one buffer serves a shape with any budget (prefixes
  // of a length that is no multiple of four: nothing for the selection, which takes them with any workspace).
  w->least = align256(off + (s.P % 4 == 0 ? select_split_bytes(s) : 0));
  off = align256(off + w->select_bytes);
  w->total = off;
}

static ckv_status workspace_ok(const Workspace &w, const void *ws, size_t bytes) {
  if (!ws || ((uintptr_t)ws & 255) || bytes < w.least) return CKV_EWORKSPACE;
  return CKV_OK;
}

}  // namespace ckv

using namespace ckv;

extern "C" size_t ckv_workspace_bytes(const ckv_params *params) {
  if (validate(params) != CKV_OK) return 0;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  return w.total;
}

// How long a workgroup of the one-launch form waits for the others' row sums (units of 10 ns) before it makes some itself: they
// are there within 2 us where all run at once, and come late only where another kernel holds CUs. us per call, 5 / 10 / 30 us: beside a
// scan that holds 136 CUs 4096 keys, 32/32 heads 56 / 50 / 49, 16384, batch 2, 8/2 71 / 71 / 63; on four streams 65536, batch 2, 8/1 56 /
// 51 / 62; without either no difference.
constexpr uint32_t kExchangeWait = 1000;

// The marks lie where a call that makes the normalisers and uses them leaves its workspace alone, in the place for those: four
// bytes for each row of a unit's heads against eight for each of its workgroups. Where that is not room enough, two launches.
Exchange ckv::exchange_of(const ckv_params *p, const Shape &s, const Workspace &w, const float *lse, void *workspace) {
  Exchange e;
  if (!lse && !(p->flags & (CKV_FLAG_VALUE_NORM | CKV_FLAG_GROUP_MASS)) && one_launch(p, s) &&
      (size_t)s.Bz * s.Hkv * s.n_chunks * sizeof(tag_t) <= w.vsum_off - w.lse_off)
    e.marks = (tag_t *)((char *)workspace + w.lse_off);
  e.wait = kExchangeWait;
  return e;
}

// The calls of a layer behind validate(), derive() and layout(), which ckv_retention_layer has done once for all of them. What a step
// refuses is a function of its own: the layer asks for all of its steps' before it queues the first.
static ckv_status scores_refused(const ckv_params *params, const Shape &s, const Workspace &w, const void *q_win, const void *k,
                                 const void *v, const float *scores, const float *vnorm_ratio, const void *workspace,
                                 size_t workspace_bytes) {
  if (!q_win || !k || !scores) return CKV_EINVAL;
  if ((params->flags & CKV_FLAG_VALUE_NORM) && (!v || !vnorm_ratio)) return CKV_EINVAL;
  const ckv_status st = workspace_ok(w, workspace, workspace_bytes);
  if (st != CKV_OK) return st;
  // the group-mass output exists where one wave holds all query heads of a KV head, one tile each
  if ((params->flags & CKV_FLAG_GROUP_MASS) && !(params->dtype == CKV_BF16 && s.n_groups == 1 && s.WT == 1 && s.NQ <= 4))
    return CKV_EUNSUPPORTED;
  return CKV_OK;
}

ckv_status ckv::scores_of(const ckv_params *params, const Shape &s, const Workspace &w, const void *q_win, const void *k,
                          const void *v, const float *lse, float *scores, float *vnorm_ratio, void *workspace,
                          size_t workspace_bytes, hipStream_t stream, const Exchange &exchange) {
  const ckv_status st = scores_refused(params, s, w, q_win, k, v, scores, vnorm_ratio, workspace, workspace_bytes);
  if (st != CKV_OK) return st;
  const bool vn = params->flags & CKV_FLAG_VALUE_NORM;
  if (vn && !norms_in_scan(params, s, lse != nullptr) &&
      launch_value_norm(params, s, w, v, vnorm_ratio, (char *)workspace, stream) != hipSuccess)
    return CKV_EHIP;
  if (launch_window_scores(params, s, w, q_win, k, lse, nullptr, scores, (char *)workspace, stream, nullptr, v,
                           vn ? vnorm_ratio : nullptr, exchange) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_window_scores(const ckv_params *params, const void *q_win, const void *k,
                                        const void *v, const float *lse, float *scores,
                                        float *vnorm_ratio, void *workspace, size_t workspace_bytes,
                                        void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  return scores_of(params, s, w, q_win, k, v, lse, scores, vnorm_ratio, workspace, workspace_bytes, (hipStream_t)hip_stream,
                   exchange_of(params, s, w, lse, workspace));
}

extern "C" ckv_status ckv_window_lse(const ckv_params *params, const void *q_win, const void *k,
                                     float *lse, void *workspace, size_t workspace_bytes,
                                     void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!q_win || !k || !lse) return CKV_EINVAL;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  st = workspace_ok(w, workspace, workspace_bytes);
  if (st != CKV_OK) return st;
  if (launch_window_scores(params, s, w, q_win, k, nullptr, lse, nullptr, (char *)workspace,
                           (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

// ---------------------------------------------------------------------------------------------
// ckv_window_lse for callers that cannot allocate: the row partials of the scan's first pass live in a
// device array of the library instead of a caller's workspace. Host code never passes the array's name
// to a kernel (on the host it is only a stand-in for the symbol): the device address is looked up once
// per device, with that device current, and kept.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[CKV_STATIC_SCRATCH_BYTES];
static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mutex;
static void *g_scratch_ptr[kMaxDevices];  // device address of `scratch` on each device, once known

static hipError_t static_scratch(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!ptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

extern "C" size_t ckv_window_lse_static_bytes(const ckv_params *params) {
  if (validate(params) != CKV_OK) return 0;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  return w.part_bytes;
}

extern "C" ckv_status ckv_window_lse_static(const ckv_params *params, const void *q_win, const void *k, float *lse,
                                            void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!q_win || !k || !lse) return CKV_EINVAL;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  // only the row partials are scratch here (they sit first in the layout); LSE goes to the caller's buffer
  if (w.part_off != 0 || w.part_bytes > (size_t)CKV_STATIC_SCRATCH_BYTES) return CKV_EWORKSPACE;
  void *ptr = nullptr;
  if (static_scratch(&ptr) != hipSuccess) return CKV_EHIP;
  if (launch_window_scores(params, s, w, q_win, k, nullptr, lse, nullptr, (char *)ptr, (hipStream_t)hip_stream) !=
      hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

static ckv_status tables_refused(const ckv_params *params, const float *scores, const float *vnorm_ratio, const float *w_head,
                                 const float *t_gate, int32_t n_ent, int32_t n_ppl, const int32_t *risk_bins, const float *utility,
                                 const int32_t *budget, const float *tau) {
  if (!scores || !w_head || !utility || !budget || !tau) return CKV_EINVAL;
  if (params->flags & CKV_FLAG_GROUP_MASS) return CKV_EINVAL;  // needs per-head masses
  if ((params->flags & CKV_FLAG_VALUE_NORM) && !vnorm_ratio) return CKV_EINVAL;
  if (t_gate && (n_ent < 1 || n_ppl < 1 || !risk_bins)) return CKV_EINVAL;
  return CKV_OK;
}

static ckv_status tables_of(const ckv_params *params, const Shape &s, const float *scores, const float *vnorm_ratio,
                            const float *w_head, const float *head_share, const float *t_gate, int32_t n_ent, int32_t n_ppl,
                            const int32_t *risk_bins, float *utility, int32_t *budget, float *tau, hipStream_t stream) {
  const ckv_status st = tables_refused(params, scores, vnorm_ratio, w_head, t_gate, n_ent, n_ppl, risk_bins, utility, budget, tau);
  if (st != CKV_OK) return st;
  if (launch_apply_tables(params, s, scores, vnorm_ratio, w_head, head_share, t_gate, n_ent, n_ppl,
                          risk_bins, utility, budget, tau, stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_apply_tables(const ckv_params *params, const float *scores,
                                       const float *vnorm_ratio, const float *w_head,
                                       const float *head_share, const float *t_gate, int32_t n_ent,
                                       int32_t n_ppl, const int32_t *risk_bins, float *utility,
                                       int32_t *budget, float *tau, void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  derive(params, &s);
  return tables_of(params, s, scores, vnorm_ratio, w_head, head_share, t_gate, n_ent, n_ppl, risk_bins, utility, budget, tau,
                   (hipStream_t)hip_stream);
}

// Whether ckv_window_utility can run its fused second pass for this call (else it runs the two
// unfused steps through the scratch buffer): the pipelined bf16 kernels with at most two 32-row tiles per
// head and all query tiles of a group in one wave (at most eight), pooling kernels of at most 7 taps. Rows may start
// at any multiple of four bytes: with lengths that are no multiple of four the stores cover five lines where they
// would four (us, both passes and tables, fused / unfused: 32767 positions, batch 16: 374 / 398; 32768: 375 / 404; 20011,
// batch 2: 44.2 / 45.7; 4096, 32/32 heads 23.3 / 25.0). With the value-norm flag the ratio, which is common to
// a group's heads and non-negative, multiplies the group maximum afterwards (at the end of the same pass).
static bool utility_fast_path(const ckv_params *p, const Shape &s) {
  const int kernel = p->pool == CKV_POOL_NONE ? 1 : p->pool_kernel;
  return p->dtype == CKV_BF16 && s.n_groups == 1 && s.WT <= 2 && kernel / 2 <= kUtilMaxRadius && s.P > 0 && s.T >= 4 &&
         (int64_t)s.Hkv * s.P < (1 << 29);
}

static ckv_status utility_refused(const ckv_params *params, const Workspace &w, const void *q_win, const void *k, const void *v,
                                  const float *w_head, const float *t_gate, int32_t n_ent, int32_t n_ppl, const int32_t *risk_bins,
                                  const float *scores_scratch, const float *vnorm_ratio, const float *utility, const int32_t *budget,
                                  const float *tau, const void *workspace, size_t workspace_bytes) {
  if (!q_win || !k) return CKV_EINVAL;
  if ((params->flags & CKV_FLAG_VALUE_NORM) && !v) return CKV_EINVAL;
  const ckv_status st =
      tables_refused(params, scores_scratch, vnorm_ratio, w_head, t_gate, n_ent, n_ppl, risk_bins, utility, budget, tau);
  return st != CKV_OK ? st : workspace_ok(w, workspace, workspace_bytes);
}

ckv_status ckv::utility_of(const ckv_params *params, const Shape &s, const Workspace &w, const void *q_win, const void *k,
                           const void *v, const float *lse, const float *w_head, const float *head_share, const float *t_gate,
                           int32_t n_ent, int32_t n_ppl, const int32_t *risk_bins, float *scores_scratch, float *vnorm_ratio,
                           float *utility, int32_t *budget, float *tau, void *workspace, size_t workspace_bytes,
                           hipStream_t stream, const Exchange &exchange) {
  const ckv_status st = utility_refused(params, w, q_win, k, v, w_head, t_gate, n_ent, n_ppl, risk_bins, scores_scratch, vnorm_ratio,
                                        utility, budget, tau, workspace, workspace_bytes);
  if (st != CKV_OK) return st;
  const bool vn = params->flags & CKV_FLAG_VALUE_NORM;
  float *ratio = vn ? vnorm_ratio : nullptr;
  if (vn && !norms_in_scan(params, s, lse != nullptr) &&
      launch_value_norm(params, s, w, v, ratio, (char *)workspace, stream) != hipSuccess)
    return CKV_EHIP;
  if (utility_fast_path(params, s)) {
    UtilityFusion fuse;
    fuse.w_row = w_head + (size_t)params->layer * s.Hq;
    fuse.utility = utility;
    fuse.pool = params->pool;
    const int kernel = params->pool == CKV_POOL_NONE ? 1 : params->pool_kernel;
    fuse.radius = kernel / 2;
    // rounded down, so that the rest is positive (never zero: an infinite sum stays infinite)
    fuse.inv_kernel = 1.0f / (float)kernel;
    if ((double)fuse.inv_kernel * kernel > 1.0) fuse.inv_kernel = nextafterf(fuse.inv_kernel, 0.0f);
    fuse.inv_kernel_rest = fmaxf((float)(1.0 / kernel - (double)fuse.inv_kernel), FLT_MIN);
    fuse.bud = budget_args(params, s, head_share, t_gate, n_ent, n_ppl, risk_bins, budget, tau);
    if (launch_window_scores(params, s, w, q_win, k, lse, nullptr, scores_scratch, (char *)workspace, stream,
                             &fuse, v, ratio, exchange) != hipSuccess)
      return CKV_EHIP;
    return CKV_OK;
  }
  if (launch_window_scores(params, s, w, q_win, k, lse, nullptr, scores_scratch, (char *)workspace, stream, nullptr,
                           v, ratio, exchange) != hipSuccess)
    return CKV_EHIP;
  if (launch_apply_tables(params, s, scores_scratch, vnorm_ratio, w_head, head_share, t_gate, n_ent, n_ppl,
                          risk_bins, utility, budget, tau, stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_window_utility(const ckv_params *params, const void *q_win, const void *k,
                                         const void *v, const float *lse, const float *w_head,
                                         const float *head_share, const float *t_gate, int32_t n_ent,
                                         int32_t n_ppl, const int32_t *risk_bins, float *scores_scratch,
                                         float *vnorm_ratio, float *utility, int32_t *budget, float *tau,
                                         void *workspace, size_t workspace_bytes, void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  return utility_of(params, s, w, q_win, k, v, lse, w_head, head_share, t_gate, n_ent, n_ppl, risk_bins, scores_scratch, vnorm_ratio,
                    utility, budget, tau, workspace, workspace_bytes, (hipStream_t)hip_stream, exchange_of(params, s, w, lse, workspace));
}

// The workspace is optional here: short prefixes are selected by one workgroup per unit, everything on chip; for long ones it
// lets the selection split a unit over several workgroups.
static bool select_workspace_short(const Shape &s, const Workspace &w, const void *workspace, size_t workspace_bytes) {
  return ((uintptr_t)workspace & 255) || workspace_bytes < w.select_off + select_split_bytes(s);
}
static ckv_status select_refused(const Shape &s, const Workspace &w, const float *utility, const int32_t *budget, const float *tau,
                                 const int32_t *idx, const int32_t *count, const void *workspace, size_t workspace_bytes) {
  if (!utility || !budget || !tau || !idx || !count) return CKV_EINVAL;
  const bool given = workspace && w.select_bytes > 0;
  return given && s.P % 4 == 0 && select_workspace_short(s, w, workspace, workspace_bytes) ? CKV_EWORKSPACE : CKV_OK;
}

static ckv_status select_of(const ckv_params *params, const Shape &s, const Workspace &w, const float *utility,
                            const int32_t *budget, const float *tau, int32_t *idx, int32_t *count, void *workspace,
                            size_t workspace_bytes, hipStream_t stream) {
  const ckv_status st = select_refused(s, w, utility, budget, tau, idx, count, workspace, workspace_bytes);
  if (st != CKV_OK) return st;
  const bool split = workspace && w.select_bytes > 0 && !select_workspace_short(s, w, workspace, workspace_bytes);
  if (launch_select(params, s, utility, budget, tau, idx, count, split ? (char *)workspace + w.select_off : nullptr,
                    split ? workspace_bytes - w.select_off : 0, stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_select_topk(const ckv_params *params, const float *utility,
                                      const int32_t *budget, const float *tau, int32_t *idx,
                                      int32_t *count, void *workspace, size_t workspace_bytes,
                                      void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  return select_of(params, s, w, utility, budget, tau, idx, count, workspace, workspace_bytes, (hipStream_t)hip_stream);
}

static ckv_status gather_refused(const void *k, const void *v, const int32_t *idx, const int32_t *count, const void *k_out,
                                 const void *v_out) {
  return !k || !v || !idx || !count || !k_out || !v_out ? CKV_EINVAL : CKV_OK;
}

static ckv_status gather_of(const ckv_params *params, const Shape &s, const void *k, const void *v, const int32_t *idx,
                            const int32_t *count, void *k_out, void *v_out, hipStream_t stream, bool shared_list) {
  const ckv_status st = gather_refused(k, v, idx, count, k_out, v_out);
  if (st != CKV_OK) return st;
  if (launch_gather(params, s, k, v, idx, count, k_out, v_out, stream, shared_list) != hipSuccess) return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_compact_kv(const ckv_params *params, const void *k, const void *v,
                                     const int32_t *idx, const int32_t *count, void *k_out,
                                     void *v_out, void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  derive(params, &s);
  return gather_of(params, s, k, v, idx, count, k_out, v_out, (hipStream_t)hip_stream, false);
}

// A layer's kernels queued by one call: what its separate calls cost the host besides the launches (marshalling of four calls,
// validation and the split of the key axis for each) is as much as a short layer takes on the GPU. us per layer on a stream of
// them, separate / one call: f32, 1024 keys, 4/4 heads 26.1 / 20.5, host time of 4096 keys, 32/32 heads 19.0 / 14.7.
extern "C" ckv_status ckv_retention_layer(const ckv_params *params, const void *q_win, const void *k, const void *v,
                                          const float *lse, const float *w_head, const float *head_share,
                                          const float *t_gate, int32_t n_ent, int32_t n_ppl, const int32_t *risk_bins,
                                          float *scores, int32_t scores_wanted, float *vnorm_ratio, float *utility,
                                          int32_t *budget, float *tau, int32_t *idx, int32_t *count, void *k_out,
                                          void *v_out, void *workspace, size_t workspace_bytes, void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  Workspace w;
  derive(params, &s);
  layout(params, s, &w);
  if (scores_wanted) {
    st = scores_refused(params, s, w, q_win, k, v, scores, vnorm_ratio, workspace, workspace_bytes);
    if (st == CKV_OK)
      st = tables_refused(params, scores, vnorm_ratio, w_head, t_gate, n_ent, n_ppl, risk_bins, utility, budget, tau);
  } else {
    st = utility_refused(params, w, q_win, k, v, w_head, t_gate, n_ent, n_ppl, risk_bins, scores, vnorm_ratio, utility, budget, tau,
                         workspace, workspace_bytes);
  }
  if (st == CKV_OK) st = select_refused(s, w, utility, budget, tau, idx, count, workspace, workspace_bytes);
  if (st == CKV_OK) st = gather_refused(k, v, idx, count, k_out, v_out);
  if (st != CKV_OK) return st;
  hipStream_t stream = (hipStream_t)hip_stream;
  const Exchange exchange = exchange_of(params, s, w, lse, workspace);
  if (scores_wanted) {
    st = scores_of(params, s, w, q_win, k, v, lse, scores, vnorm_ratio, workspace, workspace_bytes, stream, exchange);
    if (st == CKV_OK)
      st = tables_of(params, s, scores, vnorm_ratio, w_head, head_share, t_gate, n_ent, n_ppl, risk_bins, utility, budget, tau, stream);
  } else {
    st = utility_of(params, s, w, q_win, k, v, lse, w_head, head_share, t_gate, n_ent, n_ppl, risk_bins, scores, vnorm_ratio, utility,
                    budget, tau, workspace, workspace_bytes, stream, exchange);
  }
  const bool shares = head_share != nullptr;
  if (st == CKV_OK && keeps_in_one_launch(params, s, shares))
    return launch_keep(params, s, utility, budget, tau, k, v, idx, count, k_out, v_out, shares, stream) == hipSuccess ? CKV_OK : CKV_EHIP;
  if (st == CKV_OK) st = select_of(params, s, w, utility, budget, tau, idx, count, workspace, workspace_bytes, stream);
  if (st == CKV_OK) st = gather_of(params, s, k, v, idx, count, k_out, v_out, stream, false);
  return st;
}

extern "C" ckv_status ckv_alpha_accumulate(const ckv_params *params, const float *scores, float weight,
                                           float *alpha, void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!scores || !alpha || !isfinite(weight)) return CKV_EINVAL;
  Shape s;
  derive(params, &s);
  const int rows = (params->flags & CKV_FLAG_GROUP_MASS) ? s.Hkv : s.Hq;  // rows of scores per batch element
  if (launch_alpha_accumulate(s, rows, scores, weight, alpha, (hipStream_t)hip_stream) != hipSuccess) return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_risk_struct(const ckv_params *params, const float *alpha, const float *ent_edges,
                                      int32_t n_edges, float *risk, int32_t *bin, void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!alpha || !risk || n_edges < 0 || (bin && n_edges > 0 && !ent_edges)) return CKV_EINVAL;
  Shape s;
  derive(params, &s);
  if (launch_risk_struct(s, alpha, ent_edges, n_edges, risk, bin, (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_shared_utility(const ckv_params *params, const float *alpha, const float *vnorm_ratio,
                                         const float *w_head, const float *t_gate, int32_t n_ent, int32_t n_ppl,
                                         const int32_t *risk_bins, float *utility, float *tau, void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!alpha || !vnorm_ratio || !w_head || !utility || !tau) return CKV_EINVAL;
  if (t_gate && (n_ent < 1 || n_ppl < 1 || !risk_bins)) return CKV_EINVAL;
  Shape s;
  derive(params, &s);
  if (launch_shared_utility(params, s, alpha, vnorm_ratio, w_head, t_gate, n_ent, n_ppl, risk_bins, utility, tau,
                            (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_compact_kv_shared(const ckv_params *params, const void *k, const void *v,
                                            const int32_t *idx, const int32_t *count, void *k_out, void *v_out,
                                            void *hip_stream) {
  const ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  Shape s;
  derive(params, &s);
  return gather_of(params, s, k, v, idx, count, k_out, v_out, (hipStream_t)hip_stream, true);
}

extern "C" ckv_status ckv_map_table_depth(const float *table, int32_t n_layers_src, int32_t row_elems, float *mapped,
                                          int32_t n_layers_dst, void *hip_stream) {
  if (!table || !mapped || n_layers_src < 1 || n_layers_dst < 1 || row_elems < 1) return CKV_EINVAL;
  if ((int64_t)n_layers_dst * row_elems > (1 << 30)) return CKV_EUNSUPPORTED;
  if (launch_map_depth(table, n_layers_src, row_elems, mapped, n_layers_dst, (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

static ckv_status decode_args_ok(const ckv_params *p, int32_t n_q, int32_t n_rows, const int64_t *k_stride,
                                 const int64_t *v_stride) {
  if (n_q < 1 || n_rows < 1 || !k_stride || !v_stride) return CKV_EINVAL;
  const int64_t per16 = p->dtype == CKV_BF16 ? 8 : 4;
  for (int i = 0; i < 3; ++i)
    if (k_stride[i] < 0 || v_stride[i] < 0 || k_stride[i] % per16 || v_stride[i] % per16) return CKV_EINVAL;
  if (k_stride[2] < p->head_dim || v_stride[2] < p->head_dim) return CKV_EINVAL;
  if (n_rows > (1 << 24)) return CKV_EUNSUPPORTED;
  return CKV_OK;
}

extern "C" size_t ckv_decode_workspace_bytes(const ckv_params *params, int32_t n_q, int32_t n_rows) {
  if (validate(params) != CKV_OK || n_q < 1 || n_rows < 1) return 0;
  Shape s;
  derive(params, &s);
  const DecodePlan plan = plan_decode(s, n_q, n_rows);
  if (plan.grid_y > 65535) return 0;
  return align256(plan.workspace_bytes);
}

extern "C" ckv_status ckv_decode_attention(const ckv_params *params, const void *q_dec, int32_t n_q,
                                           const void *k_rows, const void *v_rows, const int64_t *k_stride,
                                           const int64_t *v_stride, int32_t n_rows, const int32_t *count,
                                           float *out, float *lse, void *workspace, size_t workspace_bytes,
                                           void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (!q_dec || !k_rows || !v_rows || !out || !lse) return CKV_EINVAL;
  st = decode_args_ok(params, n_q, n_rows, k_stride, v_stride);
  if (st != CKV_OK) return st;
  if (((uintptr_t)q_dec | (uintptr_t)k_rows | (uintptr_t)v_rows) & 15) return CKV_EINVAL;
  Shape s;
  derive(params, &s);
  const DecodePlan plan = plan_decode(s, n_q, n_rows);
  if (plan.grid_y > 65535) return CKV_EUNSUPPORTED;  // grid.y
  if (plan.workspace_bytes > 0 &&
      (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < plan.workspace_bytes))
    return CKV_EWORKSPACE;
  if (launch_decode_attention(params, s, q_dec, n_q, k_rows, v_rows, k_stride, v_stride, n_rows, count, out, lse,
                              (char *)workspace, (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" ckv_status ckv_discarded_mass(const ckv_params *params, int32_t n_q, const float *lse_full,
                                         const float *lse_kept, float *mass, float *eps_tail, void *hip_stream) {
  ckv_status st = validate(params);
  if (st != CKV_OK) return st;
  if (n_q < 1 || !lse_full || !lse_kept || !mass) return CKV_EINVAL;
  Shape s;
  derive(params, &s);
  if (launch_discarded_mass(s, n_q, lse_full, lse_kept, mass, eps_tail, (hipStream_t)hip_stream) != hipSuccess)
    return CKV_EHIP;
  return CKV_OK;
}

extern "C" const char *ckv_status_string(ckv_status status) {
  switch (status) {
    case CKV_OK: return "ok";
    case CKV_EINVAL: return "invalid argument";
    case CKV_EUNSUPPORTED: return "unsupported configuration";
    case CKV_EWORKSPACE: return "workspace missing, misaligned or too small";
    case CKV_EHIP: return "HIP launch failed";
  }
  return "unknown status";
}
