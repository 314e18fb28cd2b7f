// Device code of the tables kernels (ckv_tables.hip): the argument block, the four-position pooling + weighted group
// maximum (paper Eq. 6), and the budget rule and the gate lookup (paper Sec. 4.3), which the fused utility form of
// the scan's second pass (ckv_scan.h) runs as well.
#ifndef CKV_TABLES_H_
#define CKV_TABLES_H_
#include "ckv_internal.h"

namespace ckv {

constexpr int kTablesThreads = 256;
constexpr int kTablesPerThread = 4;
constexpr int kTablesTile = kTablesThreads * kTablesPerThread;  // 1024 positions
constexpr int kMaxHalo = 31;                                    // pool_kernel <= 63
// Four floats at any multiple of four bytes: rows of T and P floats start on such addresses when the length is no
// multiple of four, and the 128-bit global accesses need no more.
typedef float f32x4_t __attribute__((ext_vector_type(4), aligned(4)));

struct TablesArgs {
  const float *scores;  // [Bz][Hq][T]
  const float *rho;     // [Bz][Hkv][T] or null
  const float *w_row;   // w_head + layer*Hq
  float *utility;  // [Bz][Hkv][P]
  int Bz, Hq, Hkv, G, T, W, P;
  int pool, radius, kernel;
  int n_tiles;
  int budget_rows;  // rows of workgroups in front of the tiles' that write tau and the budgets
  BudgetArgs bud;
};

// Per-head budgets of one batch element (same rule for every b; written per b for the ABI's layout), by one whole wave: lane i
// has heads i, i + 64, ... A thread going over the heads by itself was the longest path of the tables kernels (4 heads
// 2.5 us, 8 heads 4 to 5 with the shares' loads one behind the other).
__device__ __forceinline__ void write_budgets(const BudgetArgs &a, int b, int lane) {
  int32_t *out = a.budget + (size_t)b * a.Hkv;
  if (!a.share_row) {
    for (int g = lane; g < a.Hkv; g += kWave) out[g] = min(a.B, a.T);
    return;
  }
  const auto sum = [](uint32_t p, uint32_t q) { return p + q; };
  const auto larger = [](uint32_t p, uint32_t q) { return max(p, q); };
  const auto total_of = [&](uint32_t x) { return (int)lane_value(wave_scan(x, 0u, sum), kWave - 1); };
  const auto largest_of = [&](uint32_t x) { return (int)lane_value(wave_scan(x, 0u, larger), kWave - 1); };
  const long long b_tot = (long long)a.B * a.Hkv;
  // up to 64 heads a lane's only value stays in a register, beyond that its values are in out
  const bool one = a.Hkv <= kWave;
  int mine = 0;
  const auto get = [&](int g) { return one ? mine : out[g]; };
  const auto set = [&](int g, int v) {
    if (one) mine = v;
    else out[g] = v;
  };
  int total = 0;  // Hkv * T < 2^29
  for (int g = lane; g < a.Hkv; g += kWave) {
    // a share that is no number gives W; told from its bits, since the scan's translation units are compiled without NaNs
    const uint32_t bits = reinterpret_cast<const uint32_t *>(a.share_row)[g];
    double want = floor((double)__uint_as_float(bits) * (double)b_tot);
    if (want < (double)a.W) want = (double)a.W;
    if (want > (double)a.T) want = (double)a.T;
    const int keep = (bits & 0x7fffffffu) > 0x7f800000u ? a.W : (int)want;
    set(g, keep);
    total += keep;
  }
  // "While the sum exceeds B_tot, the largest budget above W (lowest head on ties) loses one", done
  // a level at a time: the n1 leaders drop together to the runner-up's value (never below W), or,
  // when the excess runs out first, share it evenly with the remainder going to the lowest heads.
  long long excess = (long long)total_of((uint32_t)total) - b_tot;
  while (excess > 0) {  // uniform
    int v1 = a.W, v2 = a.W, n1 = 0;
    for (int g = lane; g < a.Hkv; g += kWave) v1 = max(v1, get(g));
    v1 = largest_of((uint32_t)v1);
    if (v1 <= a.W) break;
    for (int g = lane; g < a.Hkv; g += kWave) {
      const int v = get(g);
      if (v == v1) ++n1;
      else v2 = max(v2, v);
    }
    v2 = largest_of((uint32_t)v2);
    n1 = total_of((uint32_t)n1);
    const long long drop = v1 - v2;
    if ((long long)n1 * drop <= excess) {
      for (int g = lane; g < a.Hkv; g += kWave)
        if (get(g) == v1) set(g, v2);
      excess -= (long long)n1 * drop;
    } else {
      const int each = (int)(excess / n1), extra = (int)(excess % n1);
      int before = 0;  // leaders among the heads in front of these 64
      for (int g0 = 0; g0 < a.Hkv; g0 += kWave) {
        const int g = g0 + lane;
        const bool leads = g < a.Hkv && get(g) == v1;
        const unsigned long long mask = __ballot(leads);
        if (leads) set(g, v1 - each - ((int)lanes_below(mask, (uint32_t)before) < extra ? 1 : 0));
        before += __popcll(mask);
      }
      excess = 0;
    }
  }
  if (one && lane < a.Hkv) out[lane] = mine;
}

__device__ __forceinline__ void write_tau_and_budgets(const BudgetArgs &a, int b, int lane) {
  if (lane == 0) {
    uint32_t tau = 0u;
    if (a.gate_layer) {
      const int be = min(max(a.risk_bins[2 * b], 0), a.n_ent - 1);
      const int bp = min(max(a.risk_bins[2 * b + 1], 0), a.n_ppl - 1);
      tau = reinterpret_cast<const uint32_t *>(a.gate_layer)[be * a.n_ppl + bp];
    }
    reinterpret_cast<uint32_t *>(a.tau)[b] = tau;
  }
  write_budgets(a, b, lane);
}

// Fast path for pooling kernels of at most kWindowTaps taps: a thread owns four consecutive positions and reads them
// plus what the window needs on either side as 128-bit loads per head (the neighbours' loads hit L1), pools
// from registers with the taps unrolled, and writes one 128-bit store. No LDS and no barriers, and no branch around
// a load (they would go out one after the other): addresses are clamped into the row, what lies outside the prefix is
// masked afterwards. Only a prefix that ends less than four elements before its row reads vectors that would not
// fit element by element. The caller has checked T >= 4.
// Utilities of the four positions t .. t + 3 (t a multiple of four, t < P) of one (batch, KV head).
constexpr int kWindowTaps = 17;
template <int POOL, int R>
__device__ __forceinline__ void pool_four(const TablesArgs &a, int unit, int t) {
  constexpr int SIDE = (R + 3) / 4;  // vectors on either side
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const float pad = POOL == CKV_POOL_MAX ? -INFINITY : 0.0f;
  const bool short_end = a.W < 4;  // the same for the whole launch
  float rho[4] = {1.0f, 1.0f, 1.0f, 1.0f};
  if (a.rho) {
    const float *row = a.rho + (size_t)unit * a.T;
    const f32x4_t r4 = *reinterpret_cast<const f32x4_t *>(row + min(t, a.T - 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) rho[e] = short_end ? row[min(t + e, a.T - 1)] : r4[e];
  }
  float best[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  // The head's weight comes by a vector load behind those of the row: with a scalar one the compiler puts the four quotients one
  // behind the other (32768 positions, batch 2, 28/4 heads 4.6 -> 4.9 us).
  uint32_t no_offset = 0;
  asm("" : "+v"(no_offset));
  for (int hg = 0; hg < a.G; ++hg) {
    const int h = g * a.G + hg;
    const float *row = a.scores + ((size_t)b * a.Hq + h) * a.T;
    float w[4 * (2 * SIDE + 1)];  // positions t - 4 SIDE ..
#pragma unroll
    for (int q = 0; q < 2 * SIDE + 1; ++q) {
      const f32x4_t v = *reinterpret_cast<const f32x4_t *>(row + max(0, min(t + 4 * (q - SIDE), a.T - 4)));
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * q + e] = v[e];
    }
    if (short_end) {
#pragma unroll
      for (int x = 0; x < 4 * (2 * SIDE + 1); ++x) w[x] = row[max(0, min(t - 4 * SIDE + x, a.T - 1))];
    }
#pragma unroll
    for (int x = 0; x < 4 * (2 * SIDE + 1); ++x) {
      const int at = t - 4 * SIDE + x;
      w[x] = at >= 0 && at < a.P ? w[x] : pad;
    }
    const float wgt = (a.w_row + h)[no_offset];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float c = w[4 * SIDE + e - R];
#pragma unroll
      for (int d = 1 - R; d <= R; ++d) c = POOL == CKV_POOL_MAX ? fmaxf(c, w[4 * SIDE + e + d]) : c + w[4 * SIDE + e + d];
      if (POOL == CKV_POOL_AVG) c = c / (float)(2 * R + 1);
      best[e] = fmaxf(best[e], wgt * (c * rho[e]));
    }
  }
  float *out = a.utility + (size_t)unit * a.P + t;
  if (t + 4 <= a.P) {
    *reinterpret_cast<f32x4_t *>(out) = f32x4_t{best[0], best[1], best[2], best[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (t + e < a.P) out[e] = best[e];
  }
}

// Host side: the argument block for one call.
inline TablesArgs tables_args(const ckv_params *p, const Shape &s, const float *scores,
                              const float *vnorm_ratio, const float *w_head, const float *head_share,
                              const float *t_gate, int n_ent, int n_ppl, const int32_t *risk_bins,
                              float *utility, int32_t *budget, float *tau) {
  TablesArgs a;
  a.scores = scores;
  a.rho = (p->flags & CKV_FLAG_VALUE_NORM) ? vnorm_ratio : nullptr;
  a.w_row = w_head + (size_t)p->layer * s.Hq;
  a.utility = utility;
  a.bud = budget_args(p, s, head_share, t_gate, n_ent, n_ppl, risk_bins, budget, tau);
  a.Bz = s.Bz; a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = s.G; a.T = s.T; a.W = s.W; a.P = s.P;
  a.pool = p->pool;
  a.kernel = p->pool == CKV_POOL_NONE ? 1 : p->pool_kernel;
  a.radius = a.kernel / 2;
  a.n_tiles = s.P > 0 ? (s.P + kTablesTile - 1) / kTablesTile : 1;
  a.budget_rows = (s.Bz + a.n_tiles - 1) / a.n_tiles;
  return a;
}

}  // namespace ckv
#endif
