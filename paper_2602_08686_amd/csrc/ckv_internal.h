// Private declarations shared by the HIP translation units of libckv (not part of the ABI).
#ifndef CKV_INTERNAL_H_
#define CKV_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ckv.h"

namespace ckv {

constexpr int kWave = 64;          // CDNA wavefront width
constexpr int kTile = 32;          // MFMA 32x32 tile edge: query rows and keys per tile
constexpr int kMaxQTiles = 8;      // query-row tiles a wave keeps in registers (bf16; f32 kernels: kMaxQTilesF32)
constexpr int kMaxQTilesF32 = 4;
constexpr int kMaxQTilesNorms = 4; // up to here a wave of the scan's first pass leaves half of its SIMD's registers
constexpr int kMaxWindowTiles = 4; // 32-row tiles per query head: W <= 128
constexpr int kScoreWaves = 4;     // waves per workgroup in the scan kernels
// Compute units of the build target (gfx950: MI355X, 256). A constant on purpose, not a device query: the
// split of the key axis, and with it the workspace layout, must be the same for ckv_workspace_bytes
// (which may run where no device is visible) and for the calls that use the workspace.
constexpr int kComputeUnits = 256;
constexpr int kSelectThreads = 1024;
// Geometry of the fused utility form of the scan's second pass (ckv_scan.h). It works in rounds of
// kRing * kTile keys per wave; each round writes the utilities of the kRing * kTile keys that end
// kUtilShift keys before the round does and keeps its last kUtilCarry column sums in front of the next
// round's. The first four keys of a wave's range (its first kUtilHead column sums are kept for them), the last
// kUtilShift keys of its rounds and the keys behind the rounds follow when the workgroup's waves have their sums.
constexpr int kRing = 4;           // key-tile images per wave, and tiles per pipeline round
constexpr int kUtilShift = 32;
constexpr int kUtilCarry = 40;
constexpr int kUtilHead = 8;
constexpr int kUtilMaxRadius = 3;  // pooling kernels of up to 7 taps
static_assert(kUtilShift % 4 == 0 && kUtilCarry % 4 == 0 && kUtilHead % 4 == 0, "128-bit pieces");
static_assert(kUtilCarry >= kUtilShift + 4 + kUtilMaxRadius, "a round's first output window reaches this far back");
static_assert(kUtilHead >= 4 + kUtilMaxRadius, "the range's first four keys need their right neighbours");
static_assert(kUtilShift >= kUtilMaxRadius, "a round's last output window stays inside the round");
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kValueNormEps = 1e-6f;
constexpr int kVnormRows = 512;   // rows of V per workgroup of the value-norm kernel

// Derived quantities every entry point needs; filled by derive() after validation.
struct Shape {
  int Bz, Hq, Hkv, G, d, T, W, P;
  int esize;        // bytes per element of Q/K/V
  int WT;           // 32-row tiles per query head = ceil(W / 32)
  int n_tiles;      // G * WT, query-row tiles per KV head
  int NQ;           // tiles per wave (multiple of WT, <= kMaxQTiles)
  int n_groups;     // ceil(n_tiles / NQ): how often K is swept for one KV head
  int keys_per_wave;
  int n_chunks;     // workgroups along the key axis per (unit, group)
  float scale;      // softmax scale
};

// A 16-byte piece of a row; STREAM marks data that is used once (non-temporal: it should not displace
// what the caches hold).
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_d;
template <bool STREAM>
__device__ __forceinline__ uint4 load_piece(const char *p) {
  if (STREAM) {
    const u32x4_d v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_d *>(p));
    return make_uint4(v[0], v[1], v[2], v[3]);
  }
  return *reinterpret_cast<const uint4 *>(p);
}

// Sum over the LPR (8, 16 or 32) consecutive lanes that hold one row; every lane ends with the total.
// Lane exchanges inside a row of 16 lanes are DPP operands of the add (quad permutes give the xor-1 and
// xor-2 partners; once quads agree, mirroring a half row or a row pairs each lane with its xor-4 /
// xor-8 partner's value); only 32-lane rows need one exchange through the LDS crossbar.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  const int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false);
  return x + __int_as_float(y);
}
template <int LPR>
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0xB1>(x);                  // quad_perm [1,0,3,2]
  x = dpp_add<0x4E>(x);                  // quad_perm [2,3,0,1]
  x = dpp_add<0x141>(x);                 // row_half_mirror
  if (LPR >= 16) x = dpp_add<0x140>(x);  // row_mirror
  if (LPR >= 32) x += __shfl_xor(x, 16);
  return x;
}

// Scans and reductions over the wave with lane moves inside the vector unit (row shifts by 1, 2, 4, 8, then the
// last lane of a row of 16 to the next row and of the lower half to the upper): a shuffle through LDS costs over
// a hundred cycles per step, and these chains are most of what a short selection waits for.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_from(uint32_t identity, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)identity, (int)x, CTRL, ROWS, 0xF, false);
}
template <class Op>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x, uint32_t identity, Op op) {  // inclusive; lane 63: the total
  x = op(x, dpp_from<0x111, 0xF>(identity, x));
  x = op(x, dpp_from<0x112, 0xF>(identity, x));
  x = op(x, dpp_from<0x114, 0xF>(identity, x));
  x = op(x, dpp_from<0x118, 0xF>(identity, x));
  x = op(x, dpp_from<0x142, 0xA>(identity, x));
  x = op(x, dpp_from<0x143, 0xC>(identity, x));
  return x;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane) {  // lane is wave-uniform
  return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}
__device__ __forceinline__ int wave_inclusive(int x) {
  return (int)wave_scan((uint32_t)x, 0u, [](uint32_t p, uint32_t q) { return p + q; });
}

// c + the set bits of the mask below this lane
__device__ __forceinline__ uint32_t lanes_below(unsigned long long mask, uint32_t c) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, c));
}

// Values that pass between workgroups of one launch: past the first-level caches and the XCD's own L2, both ways (agent scope).
template <class T>
__device__ __forceinline__ void store_across(T *p, T v) {
  __scoped_atomic_store_n(p, v, __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
}
template <class T>
__device__ __forceinline__ T load_across(const T *p) {
  return __scoped_atomic_load_n(p, __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
}
template <class T>
__device__ __forceinline__ void replace_across(T *p, T old, T v) {  // nothing where *p is not `old` any more
  __scoped_atomic_compare_exchange_n(p, &old, v, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __MEMORY_SCOPE_DEVICE);
}
// Marks that workgroups of a launch leave for one another in memory that nobody has cleared: equal to the launch's tag or not.
// A launch takes its marks back before it ends, so that a replay of it, which has the same tag, finds none; what else the memory
// may have held is no tag (launch_tag: another value for every launch of the process, such as nothing else leaves there).
typedef uint64_t tag_t;
tag_t launch_tag();

ckv_status validate(const ckv_params *p);
void derive(const ckv_params *p, Shape *s);

// Workspace layout (bytes, 256-aligned sections), all sized from Shape.
struct Workspace {
  size_t part_off, part_bytes;   // float2 [units][groups][n_chunks][NQ*32] row-stat partials
  size_t lse_off, lse_bytes;     // float  [Bz][Hq][W]
  size_t vsum_off, vsum_bytes;   // float  [units][vnorm blocks] partial sums of value norms
  size_t select_off, select_bytes;  // the long selection's: slices' pairs, or the split's histograms, counts and thresholds
  size_t least;  // what a call has to be given: less than total where total has room for the slices' pairs
  size_t total;
};
void layout(const ckv_params *p, const Shape &s, Workspace *w);
int vnorm_blocks_per_unit(const Shape &s);

// Kernel launchers (each returns hipGetLastError() after its launches).
// tau and the per-head budgets of a call (paper Sec. 4.3), written beside the utilities.
struct BudgetArgs {
  const float *share_row;   // head_share + layer*Hkv or null
  const float *gate_layer;  // t_gate + layer*n_ent*n_ppl or null
  const int32_t *risk_bins;
  int n_ent, n_ppl;
  int32_t *budget;
  float *tau;
  int Hkv, T, W;
  int B;  // nominal budget per KV head
};
BudgetArgs budget_args(const ckv_params *p, const Shape &s, const float *head_share, const float *t_gate, int n_ent,
                       int n_ppl, const int32_t *risk_bins, int32_t *budget, float *tau);

// Fused utility form of pass 2 (see ckv_window_utility): where `fuse` is given, the second pass writes the
// utilities, tau and the budgets, and no column sums.
struct UtilityFusion {
  const float *w_row;  // w_head + layer * Hq
  float *utility;      // [Bz][Hkv][P]
  int pool, radius;
  float inv_kernel, inv_kernel_rest;  // 1 / kernel: the largest float that is not above it, and what that leaves
  BudgetArgs bud;
};
// Both passes as one launch, whose workgroups keep their keys on chip and exchange the row sums: where the shape allows it
// (one_launch) and the call gives marks.
struct Exchange {
  tag_t *marks = nullptr;  // one for each workgroup, or null: two launches
  uint32_t wait = 0;       // how long a workgroup waits for another's part of the row sums, in units of 10 ns
};
bool one_launch(const ckv_params *p, const Shape &s);
// lse_in == nullptr: pass 1 first, LSE into lse_out (or the workspace). scores == nullptr: pass 1 only.
// ratio: if given, pass 2 makes it of the value norms that launch_value_norm, or with norms_in_scan() and v pass 1, left there
// (and, in the fused form, multiplies the utilities by it).
hipError_t launch_window_scores(const ckv_params *p, const Shape &s, const Workspace &w, const void *q,
                                const void *k, const float *lse_in, float *lse_out, float *scores,
                                char *ws, hipStream_t stream, const UtilityFusion *fuse = nullptr,
                                const void *v = nullptr, float *ratio = nullptr, const Exchange &exchange = {});
// What ckv_window_scores and ckv_window_utility do behind validate(), derive() and layout(), with the exchange that exchange_of()
// gives them (or none: two launches).
Exchange exchange_of(const ckv_params *p, const Shape &s, const Workspace &w, const float *lse, void *workspace);
ckv_status scores_of(const ckv_params *params, const Shape &s, const Workspace &w, const void *q_win, const void *k, const void *v,
                     const float *lse, float *scores, float *vnorm_ratio, void *workspace, size_t workspace_bytes,
                     hipStream_t stream, const Exchange &exchange);
ckv_status utility_of(const ckv_params *params, const Shape &s, const Workspace &w, const void *q_win, const void *k, const void *v,
                      const float *lse, const float *w_head, const float *head_share, const float *t_gate, int32_t n_ent,
                      int32_t n_ppl, const int32_t *risk_bins, float *scores_scratch, float *vnorm_ratio, float *utility,
                      int32_t *budget, float *tau, void *workspace, size_t workspace_bytes, hipStream_t stream,
                      const Exchange &exchange);
// Whether pass 1 of a call takes the value norms beside its scan; the norms and sums are those of launch_value_norm.
bool norms_in_scan(const ckv_params *p, const Shape &s, bool lse_given);
// the norms into `ratio` and their sums per block into the workspace; launch_window_scores turns them into the ratio
hipError_t launch_value_norm(const ckv_params *p, const Shape &s, const Workspace &w, const void *v,
                             float *ratio, char *ws, hipStream_t stream);
hipError_t launch_apply_tables(const ckv_params *p, const Shape &s, const float *scores,
                               const float *vnorm_ratio, const float *w_head, const float *head_share,
                               const float *t_gate, int n_ent, int n_ppl, const int32_t *risk_bins,
                               float *utility, int32_t *budget, float *tau, hipStream_t stream);
// ws: nullptr, or ws_bytes bytes (256-byte aligned), at least select_split_bytes(), that let long prefixes be split
// over several workgroups per unit; with select_workspace_bytes() it is the form that suits the budget. The
// result is the same either way. The split's bytes follow from the shape alone, so one buffer serves any budget.
size_t select_split_bytes(const Shape &s);
size_t select_workspace_bytes(const ckv_params *p, const Shape &s);
hipError_t launch_select(const ckv_params *p, const Shape &s, const float *utility,
                         const int32_t *budget, const float *tau, int32_t *idx, int32_t *count,
                         char *ws, size_t ws_bytes, hipStream_t stream);
// Selection and gather together, where keeps_in_one_launch(); without shares no head's budget is above the nominal one.
bool keeps_in_one_launch(const ckv_params *p, const Shape &s, bool shares);
hipError_t launch_keep(const ckv_params *p, const Shape &s, const float *utility, const int32_t *budget, const float *tau, const void *k,
                       const void *v, int32_t *idx, int32_t *count, void *k_out, void *v_out, bool shares, hipStream_t stream);
hipError_t launch_gather(const ckv_params *p, const Shape &s, const void *k, const void *v,
                         const int32_t *idx, const int32_t *count, void *k_out, void *v_out,
                         hipStream_t stream, bool shared_list = false);
// layer-shared mode (Alg. 1 as printed)
hipError_t launch_alpha_accumulate(const Shape &s, int rows, const float *scores, float weight, float *alpha,
                                   hipStream_t stream);
hipError_t launch_risk_struct(const Shape &s, const float *alpha, const float *edges, int n_edges, float *risk,
                              int32_t *bin, hipStream_t stream);
hipError_t launch_shared_utility(const ckv_params *p, const Shape &s, const float *alpha, const float *rho,
                                 const float *w_head, const float *t_gate, int n_ent, int n_ppl,
                                 const int32_t *risk_bins, float *utility, float *tau, hipStream_t stream);

hipError_t launch_map_depth(const float *src, int n_src, int row, float *dst, int n_dst, hipStream_t stream);
// decode-side consumer (Proposition 1): attention over a ragged KV set, discarded mass
struct DecodePlan {
  int rq;              // query heads of a group that share one sweep over the rows (1, 2, 4 or 8)
  int head_chunks;     // ceil(G / rq)
  bool mfma;           // the bf16 matrix-core kernel, else the vector kernel
  int n_chunks;
  int64_t grid_y;      // Bz * Hkv * n_q * head_chunks
  int col_chunks;      // bf16: 16-wide tiles of a KV head's G * n_q query columns
  int64_t workgroups;  // bf16: Bz * Hkv * col_chunks
  size_t workspace_bytes;
};
DecodePlan plan_decode(const Shape &s, int n_q, int n_rows);
hipError_t launch_decode_attention(const ckv_params *p, const Shape &s, const void *q_dec, int n_q, const void *k_rows,
                                   const void *v_rows, const int64_t *k_stride, const int64_t *v_stride, int n_rows,
                                   const int32_t *count, float *out, float *lse, char *ws, hipStream_t stream);
hipError_t launch_discarded_mass(const Shape &s, int n_q, const float *lse_full, const float *lse_kept, float *mass,
                                 float *eps, hipStream_t stream);

}  // namespace ckv
#endif
