// Pooling + compiled-table application (paper Eq. 4 u = alpha * rho, Eq. 6 weighted max over heads,
// Sec. 4.3 gate lookup; 1-D pooling and the per-head budget split are workload definitions).
//
// Windows of up to 17 taps are pooled from registers, four positions to a thread (tables_window_kernel), whatever the
// alignment of the rows. Longer ones: one workgroup owns one tile of kTablesTile prefix positions of one (batch, KV
// head); for each query head of the group it stages the tile plus a halo of pool_kernel/2 positions in LDS, pools,
// multiplies by rho and by the head's weight, and keeps the running maximum in registers. Two barriers per head and a
// read of LDS per tap make that the slower form (10006 positions, 32 units, 7 taps: 15.1 us against 5.7), so it is
// left where the register window would not fit.
#include "ckv_tables.h"

namespace ckv {

// Tau and the budgets of a batch element are for one wave, alone in its workgroup: with shares a longer chain than the pooling of four
// positions. These workgroups fill the launch's first rows, which they share with up to n_tiles - 1 idle ones. As a column behind the
// tiles they and the idle ones among them put more tiles on some XCDs than on others, and launches that fill the CUs evenly waited
// for those (us, column / rows in front: 5960 positions, batch 31, 8/4 heads 4.5 / 4.2; 6705, batch 35, 28/4 9.5 / 8.1; 20989, batch 3,
// 32/4, 15 taps 6.4 / 5.4; 23011, batch 11, 32/8, 41 taps 32.5 / 28.7; without shares 32768, batch 2, 28/4 5.0 / 4.3, and 4.4
// by the last tile's workgroup behind its pooling).
__device__ __forceinline__ void budgets_in_front(const TablesArgs &a, int unit) {
  const int b = (int)blockIdx.y * a.n_tiles + (int)blockIdx.x;
  if (threadIdx.x >= kTablesThreads - kWave && unit < 0 && b < a.Bz) write_tau_and_budgets(a.bud, b, threadIdx.x & (kWave - 1));
}

__global__ void __launch_bounds__(kTablesThreads) tables_kernel(TablesArgs a) {
  __shared__ float sm[kTablesTile + 2 * kMaxHalo];
  const int unit = (int)blockIdx.y - a.budget_rows, tile = blockIdx.x;
  budgets_in_front(a, unit);
  if (unit < 0) return;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int t0 = tile * kTablesTile;

  float best[kTablesPerThread];
  float rho[kTablesPerThread];
#pragma unroll
  for (int e = 0; e < kTablesPerThread; ++e) {
    best[e] = -INFINITY;
    const int t = t0 + threadIdx.x + e * kTablesThreads;
    rho[e] = (a.rho && t < a.P) ? a.rho[(size_t)unit * a.T + t] : 1.0f;
  }
  const int span = kTablesTile + 2 * a.radius;
  const float pad = a.pool == CKV_POOL_MAX ? -INFINITY : 0.0f;
  for (int hg = 0; hg < a.G; ++hg) {
    const int h = g * a.G + hg;
    const float *row = a.scores + ((size_t)b * a.Hq + h) * a.T;
    __syncthreads();  // previous head's tile fully consumed
    for (int i = threadIdx.x; i < span; i += kTablesThreads) {
      const int t = t0 - a.radius + i;
      sm[i] = (t >= 0 && t < a.P) ? row[t] : pad;  // pooling sees the prefix only
    }
    __syncthreads();
    const float wgt = a.w_row[h];
#pragma unroll
    for (int e = 0; e < kTablesPerThread; ++e) {
      const int i = threadIdx.x + e * kTablesThreads + a.radius;  // centre in sm
      float c;
      if (a.pool == CKV_POOL_AVG) {
        c = 0.0f;
        for (int dt = -a.radius; dt <= a.radius; ++dt) c += sm[i + dt];
        c = c / (float)a.kernel;
      } else if (a.pool == CKV_POOL_MAX) {
        c = -INFINITY;
        for (int dt = -a.radius; dt <= a.radius; ++dt) c = fmaxf(c, sm[i + dt]);
      } else {
        c = sm[i];
      }
      best[e] = fmaxf(best[e], wgt * (c * rho[e]));
    }
  }
#pragma unroll
  for (int e = 0; e < kTablesPerThread; ++e) {
    const int t = t0 + threadIdx.x + e * kTablesThreads;
    if (t < a.P) a.utility[(size_t)unit * a.P + t] = best[e];
  }
}

template <int POOL, int R>
__global__ void __launch_bounds__(kTablesThreads) tables_window_kernel(TablesArgs a) {
  const int unit = (int)blockIdx.y - a.budget_rows;
  const int t = (blockIdx.x * kTablesThreads + threadIdx.x) * 4;  // first of this thread's positions
  if (unit >= 0 && t < a.P) pool_four<POOL, R>(a, unit, t);
  budgets_in_front(a, unit);  // behind the pooling's code: in front of it 1 to 3 % slower
}

template <int POOL>
static bool launch_window_pool(const TablesArgs &a, dim3 grid, hipStream_t stream) {
  const dim3 block(kTablesThreads);
#define CKV_WINDOW(R) \
  case R: hipLaunchKernelGGL((tables_window_kernel<POOL, R>), grid, block, 0, stream, a); return true;
  switch (a.radius) {
    CKV_WINDOW(0) CKV_WINDOW(1) CKV_WINDOW(2) CKV_WINDOW(3) CKV_WINDOW(4) CKV_WINDOW(5) CKV_WINDOW(6) CKV_WINDOW(7) CKV_WINDOW(8)
  }
#undef CKV_WINDOW
  return false;
}

// `rows` rows of workgroups, the first a.budget_rows of which write tau and the budgets.
static void launch_rows(const TablesArgs &a, int rows, hipStream_t stream) {
  const dim3 grid(a.n_tiles, rows);
  bool done = false;
  if (a.T >= 4 && a.kernel <= kWindowTaps)
    done = a.pool == CKV_POOL_MAX ? launch_window_pool<CKV_POOL_MAX>(a, grid, stream) : launch_window_pool<CKV_POOL_AVG>(a, grid, stream);
  if (!done) hipLaunchKernelGGL(tables_kernel, grid, dim3(kTablesThreads), 0, stream, a);
}

BudgetArgs budget_args(const ckv_params *p, const Shape &s, const float *head_share, const float *t_gate, int n_ent,
                       int n_ppl, const int32_t *risk_bins, int32_t *budget, float *tau) {
  BudgetArgs a;
  a.share_row = head_share ? head_share + (size_t)p->layer * s.Hkv : nullptr;
  a.gate_layer = t_gate ? t_gate + (size_t)p->layer * n_ent * n_ppl : nullptr;
  a.risk_bins = risk_bins;
  a.n_ent = n_ent;
  a.n_ppl = n_ppl;
  a.budget = budget;
  a.tau = tau;
  a.Hkv = s.Hkv; a.T = s.T; a.W = s.W;
  a.B = p->budget_per_kv_head;
  return a;
}

hipError_t launch_apply_tables(const ckv_params *p, const Shape &s, const float *scores,
                               const float *vnorm_ratio, const float *w_head, const float *head_share,
                               const float *t_gate, int n_ent, int n_ppl, const int32_t *risk_bins,
                               float *utility, int32_t *budget, float *tau, hipStream_t stream) {
  TablesArgs a = tables_args(p, s, scores, vnorm_ratio, w_head, head_share, t_gate, n_ent, n_ppl, risk_bins,
                             utility, budget, tau);
  const int units = s.P > 0 ? s.Bz * s.Hkv : 0;
  if (a.budget_rows + units <= 65535) {  // the grid's second dimension, and what units are limited to
    launch_rows(a, a.budget_rows + units, stream);
  } else {
    launch_rows(a, a.budget_rows, stream);
    a.budget_rows = 0;
    launch_rows(a, units, stream);
  }
  return hipGetLastError();
}

}  // namespace ckv
