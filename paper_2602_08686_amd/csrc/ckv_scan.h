// Kernel templates of the observation-window scan (paper Sec. 3 attention definition, Eq. 3, Eq. 4's alpha per query head):
//   pass 1  rowstats kernels : stream K, QK^T on the matrix cores, online (max, sum) per window row
//           lse_kernel       : merge the per-chunk partials into LSE_j
//   pass 2  colsum kernels   : stream K again, recompute QK^T, exp(z - LSE_j), sum over window rows;
//                              in the fused form also the pooling, head weights and group maximum of
//                              Eq. 6 (Alg. 1 Stage 3), so that the per-head mass is never written
//   scan_short_kernel        : both passes of a short call, whose keys stay in LDS between them
//
// Work decomposition. A "unit" is one (batch, KV head): its G*W window query rows all contract with
// the same K. Rows are cut into 32-row tiles (one MFMA 32x32 edge), whole heads only; a wave keeps its
// tiles of Q (up to eight for bf16, four for f32) in registers for its lifetime and takes 32-key tiles of
// K in MFMA operand layout: lane (m, hh) = (lane % 32, lane / 32) owns row m of a tile and the 16-byte
// chunks 2c+hh of that row. The contraction index may be permuted freely as long as both operands use
// the same permutation, so whole 16-byte chunks become MFMA k-groups and no transpose is needed. The
// four waves of a workgroup sweep four adjacent key ranges.
//
// The two passes use opposite operand orders on purpose:
//   pass 1: D = K Q^T, lane <-> query row: the running (max, sum) of a row never leaves its lane;
//   pass 2: D = Q K^T, lane <-> key: the sum over window rows is 16 in-lane adds and one half swap.
//
// Two families of kernels: plain ones that load every operand straight from global memory (f32,
// whose workloads are small), and LDS-staged, software-pipelined ones for bf16.
#ifndef CKV_SCAN_H_
#define CKV_SCAN_H_
#include "ckv_tables.h"

namespace ckv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t chunk_t;  // 16 bytes of one Q or K row

struct ScoreArgs {
  const char *q, *k;
  int64_t qs_b, qs_h, qs_w;  // byte strides
  int64_t ks_b, ks_h, ks_t;
  int Hq, Hkv, G, T, W, P;
  int WT, n_tiles, n_groups, keys_per_wave, n_chunks;
  float c2;     // softmax scale * log2(e): logits are kept in the log2 domain
  float norm;   // T / W
  float2 *part;      // [unit][group][n_chunks][NQ*32] (max, sum) in the log2 domain
  const float *lse;  // [Bz][Hq][W] natural log
  int lse_from_part; // both passes in one call: pass 2 merges the row partials of pass 1 itself
  float *lse_out;
  float *scores;     // [Bz][Hq][T]; with group_sum: [Bz][Hkv][T], the sum over each KV head's query heads
  int group_sum;
  float *ratio;      // [Bz][Hkv][T] or null: the norms of V's rows, which pass 2 turns into their ratio to the mean
  float *vsum;       // [Bz][Hkv][vnorm_blocks] partial sums of the norms
  int vnorm_blocks;
  const char *v;     // pass 1 takes the norms, or null
  int64_t vs_b, vs_h, vs_t;  // byte strides
  // fused utility form of pass 2 only
  const float *w_row;  // w_head + layer * Hq
  float *utility;      // [Bz][Hkv][P]
  int pool, radius;    // pooling mode and radius (kernel / 2, at most kUtilMaxRadius)
  float inv_kernel, inv_kernel_rest;  // 1 / pool_kernel in two terms
  BudgetArgs bud;
  // one-launch form only
  tag_t *marks;  // [workgroups]: the tag when the workgroup has left its row sums, tag + 1 when it has read all of its unit's
  tag_t tag;
  uint32_t wait;  // units of 10 ns
};

template <int DT> struct Mma;
template <> struct Mma<CKV_BF16> {
  static __device__ __forceinline__ void step(f32x16 &acc, const chunk_t &a, const chunk_t &b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                  __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
  }
};
template <> struct Mma<CKV_F32> {
  static __device__ __forceinline__ void step(f32x16 &acc, const chunk_t &a, const chunk_t &b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // copy the lanes out first: a bit_cast applied directly to a vector element reads element 0
      const uint32_t ua = a[e], ub = b[e];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(ua), __uint_as_float(ub), acc, 0, 0, 0);
    }
  }
};

// acc = sum over the row's chunks of a[c] . b[c]  (a: the 32 rows of D, b: the 32 columns of D)
template <int DT, int NCH>
__device__ __forceinline__ void mma_chain(f32x16 &acc, const chunk_t (&a)[NCH], const chunk_t (&b)[NCH]) {
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) Mma<DT>::step(acc, a[c], b[c]);
}

// Row of the 32x32 accumulator that element r of lane (m, hh) holds; its column is m.
__device__ __forceinline__ int acc_row(int r, int hh) { return 8 * (r >> 2) + 4 * hh + (r & 3); }

__device__ __forceinline__ void merge_stats(float &m, float &l, float om, float ol) {
  const float mn = fmaxf(m, om);
  l = l * __builtin_amdgcn_exp2f(m - mn) + ol * __builtin_amdgcn_exp2f(om - mn);
  m = mn;
}

template <int NCH>
__device__ __forceinline__ void load_row(chunk_t (&f)[NCH], const char *row, int hh) {
#pragma unroll
  for (int c = 0; c < NCH; ++c) f[c] = *reinterpret_cast<const chunk_t *>(row + (2 * c + hh) * 16);
}

struct BlockCoord {
  int chunk, grp, unit, b, g;
};
__device__ __forceinline__ BlockCoord decode_block(const ScoreArgs &a) {
  BlockCoord c;
  int bid = blockIdx.x;
  c.chunk = bid % a.n_chunks;
  bid /= a.n_chunks;
  c.grp = bid % a.n_groups;
  c.unit = bid / a.n_groups;
  c.b = c.unit / a.Hkv;
  c.g = c.unit % a.Hkv;
  // wave-uniform by construction; the divisions run on the vector ALU, so say it (addresses derived from
  // these feed scalar operands)
  c.chunk = __builtin_amdgcn_readfirstlane(c.chunk);
  c.grp = __builtin_amdgcn_readfirstlane(c.grp);
  c.unit = __builtin_amdgcn_readfirstlane(c.unit);
  c.b = __builtin_amdgcn_readfirstlane(c.b);
  c.g = __builtin_amdgcn_readfirstlane(c.g);
  return c;
}

// Loads this lane's rows of the group's NQ query tiles; jrow[i] = window row index of tile i, row m
// (or -1 where the tile or the row is padding).
template <int NCH, int NQ>
__device__ __forceinline__ void load_q_tiles(const ScoreArgs &a, const BlockCoord &bc, int m, int hh,
                                             chunk_t (&qf)[NQ][NCH], int (&jrow)[NQ]) {
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int tile = bc.grp * NQ + i;
    const int j = (tile % a.WT) * kTile + m;
    const bool valid = tile < a.n_tiles && j < a.W;
    jrow[i] = valid ? j : -1;
    if (valid) {
      const int h = bc.g * a.G + tile / a.WT;
      load_row<NCH>(qf[i], a.q + bc.b * a.qs_b + h * a.qs_h + j * a.qs_w, hh);
    } else {
#pragma unroll
      for (int c = 0; c < NCH; ++c) qf[i][c] = chunk_t{0u, 0u, 0u, 0u};
    }
  }
}

// Pass 1, vector part: online (max, sum) update of this lane's query row with the 16 logits it holds
// of one tile. The maximum is taken on the raw dot products (the scale is positive); scale and
// subtraction are one FMA per element.
template <bool EDGE, bool PLAIN = false>
__device__ __forceinline__ void rowstats_update(const f32x16 &acc, float c2, int t0, int hh, int limit, float &rm, float &rl) {
  float v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = acc[r];
  if (EDGE) {  // keys beyond `limit` do not count
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (PLAIN ? t0 + acc_row(r, hh) > limit : acc_row(r, hh) > limit - t0) v[r] = -INFINITY;
  }
  float t[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = fmaxf(fmaxf(v[4 * e], v[4 * e + 1]), fmaxf(v[4 * e + 2], v[4 * e + 3]));
  const float tmax = fmaxf(fmaxf(t[0], t[1]), fmaxf(t[2], t[3]));
  const float mn = fmaxf(rm, tmax * c2);
  float s[4];  // begun with the first weights: a zero added to them would be an instruction
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const float p = __builtin_amdgcn_exp2f(fmaf(v[r], c2, -mn));
    s[r & 3] = r < 4 ? p : s[r & 3] + p;
  }
  rl = fmaf(rl, __builtin_amdgcn_exp2f(rm - mn), (s[0] + s[1]) + (s[2] + s[3]));
  rm = mn;
}

// Merges the (max, sum) pairs of the two half-waves and of the workgroup's waves, one partial per chunk.
template <int NQ>
__device__ __forceinline__ void store_row_partials(const ScoreArgs &a, const BlockCoord &bc, int wave, int m,
                                                   int hh, float (&rm)[NQ], float (&rl)[NQ]) {
  __shared__ float2 sm[kScoreWaves][NQ * kTile];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const float om = __shfl_xor(rm[i], 32), ol = __shfl_xor(rl[i], 32);
    merge_stats(rm[i], rl[i], om, ol);
    if (hh == 0) sm[wave][i * kTile + m] = make_float2(rm[i], rl[i]);
  }
  __syncthreads();
  if (threadIdx.x < NQ * kTile) {
    float2 s = sm[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kScoreWaves; ++w) merge_stats(s.x, s.y, sm[w][threadIdx.x].x, sm[w][threadIdx.x].y);
    a.part[(((size_t)bc.unit * a.n_groups + bc.grp) * a.n_chunks + bc.chunk) * (NQ * kTile) + threadIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------------------------
// Plain kernels (f32): every tile count. Two waves per SIMD, K double-buffered in registers; one wave where two or
// more query tiles of 512-byte rows would not fit 256 registers beside it (they spilled 100 to 400).
// ---------------------------------------------------------------------------------------------
__host__ __device__ constexpr int plain_waves(int dt, int dh, int nq) { return dt == CKV_F32 && dh == 128 && nq >= 2 ? 1 : 2; }
template <int DT, int DH, int NQ>
__global__ void __launch_bounds__(kScoreWaves *kWave, plain_waves(DT, DH, NQ)) rowstats_kernel(ScoreArgs a) {
  constexpr int NCH = DH * (DT == CKV_BF16 ? 2 : 4) / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 31, hh = lane >> 5;
  const BlockCoord bc = decode_block(a);

  chunk_t qf[NQ][NCH];
  int jrow[NQ], limit[NQ];
  load_q_tiles<NCH, NQ>(a, bc, m, hh, qf, jrow);
  float rm[NQ], rl[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    limit[i] = jrow[i] < 0 ? -1 : a.P + jrow[i];  // last key this row may see (causal)
    rm[i] = -1e30f;
    rl[i] = 0.0f;
  }

  const char *kbase = a.k + bc.b * a.ks_b + bc.g * a.ks_h;
  const int t_begin = (bc.chunk * kScoreWaves + wave) * a.keys_per_wave;
  const int t_end = min(t_begin + a.keys_per_wave, a.T);
  auto tile_body = [&](const chunk_t (&kf)[NCH], int t0) {
    f32x16 acc;
    if (t0 + kTile > a.P) {  // the tile touches the window (causal mask) or the end of the keys
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        mma_chain<DT, NCH>(acc, kf, qf[i]);  // rows: keys, cols: query rows
        rowstats_update<true, true>(acc, a.c2, t0, hh, limit[i], rm[i], rl[i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        mma_chain<DT, NCH>(acc, kf, qf[i]);
        rowstats_update<false>(acc, a.c2, t0, hh, limit[i], rm[i], rl[i]);
      }
    }
  };
  // two K tiles in registers, used alternately: one is computed on while the other is in flight
  chunk_t ka[NCH], kb[NCH];
  if (t_begin < t_end) load_row<NCH>(ka, kbase + (int64_t)min(t_begin + m, a.T - 1) * a.ks_t, hh);
  for (int t0 = t_begin; t0 < t_end; t0 += 2 * kTile) {
    load_row<NCH>(kb, kbase + (int64_t)min(t0 + kTile + m, a.T - 1) * a.ks_t, hh);
    tile_body(ka, t0);
    if (t0 + kTile >= t_end) break;
    load_row<NCH>(ka, kbase + (int64_t)min(t0 + 2 * kTile + m, a.T - 1) * a.ks_t, hh);
    tile_body(kb, t0 + kTile);
  }
  store_row_partials<NQ>(a, bc, wave, m, hh, rm, rl);
}

// LSE_j = ln2 * (M + log2 sum_c l_c 2^(m_c - M)) from the n_chunks partials of one row (`stride` apart), in chunk order, eight
// loads in flight.
__device__ __forceinline__ void merge_eight(const float2 *v, float &M, float &L) {
  float top = M;
#pragma unroll
  for (int e = 0; e < 8; ++e) top = fmaxf(top, v[e].x);
  L *= __builtin_amdgcn_exp2f(M - top);
#pragma unroll
  for (int e = 0; e < 8; ++e) L += v[e].y * __builtin_amdgcn_exp2f(v[e].x - top);
  M = top;
}
__device__ __forceinline__ float merge_row_partials(const float2 *p, int n_chunks, int stride) {
  float M = -1e30f, L = 0.0f;
  for (int c0 = 0; c0 < n_chunks; c0 += 8) {
    float2 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = c0 + e < n_chunks ? p[(size_t)(c0 + e) * stride] : make_float2(-1e30f, 0.0f);
    merge_eight(v, M, L);
  }
  return (M + __log2f(L)) * kLn2;
}
// The same of partials that other workgroups of the launch have left; these loads take a microsecond, so 32 are in flight.
__device__ __forceinline__ float merge_partials_across(const float2 *p, int n_chunks, int stride) {
  constexpr int AHEAD = 32;
  float M = -1e30f, L = 0.0f;
  for (int c0 = 0; c0 < n_chunks; c0 += AHEAD) {
    float2 v[AHEAD];
#pragma unroll
    for (int b = 0; b < AHEAD; b += 8) {
      if (c0 + b >= n_chunks) continue;
#pragma unroll
      for (int e = b; e < b + 8; ++e)
        v[e] = __builtin_bit_cast(float2, load_across(reinterpret_cast<const uint64_t *>(p + (size_t)min(c0 + e, n_chunks - 1) * stride)));
    }
#pragma unroll
    for (int b = 0; b < AHEAD; b += 8) {
      if (c0 + b >= n_chunks) continue;
#pragma unroll
      for (int e = b; e < b + 8; ++e)
        if (c0 + e >= n_chunks) v[e] = make_float2(-1e30f, 0.0f);
      merge_eight(v + b, M, L);
    }
  }
  return (M + __log2f(L)) * kLn2;
}

// One thread per (unit, group, tile row).
template <int NQ>
__global__ void lse_kernel(ScoreArgs a, int n_rows_total) {
  const int row = blockIdx.x * blockDim.x + threadIdx.x;
  if (row >= n_rows_total) return;
  const int per_group = NQ * kTile;
  const int in_group = row % per_group, ug = row / per_group;
  const int grp = ug % a.n_groups;
  const int unit = ug / a.n_groups;
  const int tile = grp * NQ + in_group / kTile;
  const int j = (tile % a.WT) * kTile + in_group % kTile;
  if (tile >= a.n_tiles || j >= a.W) return;
  const int b = unit / a.Hkv, g = unit % a.Hkv, h = g * a.G + tile / a.WT;
  a.lse_out[((size_t)b * a.Hq + h) * a.W + j] =
      merge_row_partials(a.part + (size_t)ug * a.n_chunks * per_group + in_group, a.n_chunks, per_group);
}

// One 32-row x 32-key tile of pass 2 for the plain kernel. The accumulator starts at -LSE_row / scale
// (read from LDS before the MFMA chain, so the LDS latency hides behind it), the chain adds <q, k>, and
// the weight is exp2(c2 * acc) = exp(z - LSE). Returns this lane's sum over its 16 rows.
template <int DT, int NCH, bool EDGE>
__device__ __forceinline__ float colsum_tile(const chunk_t (&qf)[NCH], const chunk_t (&kf)[NCH], float c2,
                                             const float *init_tile, int hh, int first_masked_row) {
  f32x16 acc;
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const f32x4 ini = *reinterpret_cast<const f32x4 *>(init_tile + 8 * q4 + 4 * hh);
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[4 * q4 + e] = ini[e];
  }
#pragma unroll
  for (int c = 0; c < NCH; ++c) Mma<DT>::step(acc, qf[c], kf[c]);  // rows: query rows, cols: keys
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float pr = __builtin_amdgcn_exp2f(acc[r] * c2);
    // causal: key kt is visible to window row j iff kt <= P + j, i.e. tile row >= kt - P - j0
    if (EDGE && acc_row(r, hh) < first_masked_row) pr = 0.0f;
    s[r & 3] += pr;
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Value-norm ratio of the workgroup's key range: norm / (mean + eps), in place, by pass 2 (as a kernel of its own it took 4 to
// 5 us). What it reads is asked for before anything else (load) and used while the first key tiles are on their way.
typedef float f32x4_r __attribute__((ext_vector_type(4), aligned(4)));  // rows start at any multiple of four bytes
struct RatioScale {
  static constexpr int AHEAD = 2, BATCH = 4, STEP = kScoreWaves * kWave * 4;
  bool on;  // the same for the whole workgroup
  int begin, end;
  float *row;
  float part;
  f32x4_r r[AHEAD];
  __device__ __forceinline__ void load(const ScoreArgs &a, const BlockCoord &bc) {
    on = a.ratio && bc.grp == 0;
    if (!on) return;
    begin = bc.chunk * kScoreWaves * a.keys_per_wave;
    end = min(begin + kScoreWaves * a.keys_per_wave, a.T);
    row = a.ratio + (size_t)bc.unit * a.T;
    const float *vsum = a.vsum + (size_t)bc.unit * a.vnorm_blocks;
    const int lane = threadIdx.x & 63;
    part = lane < a.vnorm_blocks ? vsum[lane] : 0.0f;
#pragma unroll
    for (int e = 0; e < AHEAD; ++e) {
      const int t = begin + threadIdx.x * 4 + e * STEP;
      r[e] = f32x4_r{0.0f, 0.0f, 0.0f, 0.0f};
      if (t + 4 <= end) r[e] = *reinterpret_cast<const f32x4_r *>(row + t);
    }
  }
  __device__ __forceinline__ void store(const ScoreArgs &a, const BlockCoord &bc) {
    if (!on) return;
    float total = part;
    for (int i = kWave + (threadIdx.x & 63); i < a.vnorm_blocks; i += kWave)
      total += a.vsum[(size_t)bc.unit * a.vnorm_blocks + i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) total += __shfl_xor(total, o);
    const float inv = 1.0f / (total / (float)a.T + kValueNormEps);
    const auto scale = [&](int t0, const f32x4_r &x) {
      if (t0 + 4 <= end) *reinterpret_cast<f32x4_r *>(row + t0) = x * inv;
      else
        for (int t = t0; t < end; ++t) row[t] *= inv;
    };
    int t0 = begin + threadIdx.x * 4;
#pragma unroll
    for (int e = 0; e < AHEAD; ++e, t0 += STEP) scale(t0, r[e]);
    for (; t0 < end; t0 += BATCH * STEP) {  // longer ranges: several loads in flight
      f32x4_r x[BATCH];
#pragma unroll
      for (int e = 0; e < BATCH; ++e) x[e] = *reinterpret_cast<const f32x4_r *>(row + max(0, min(t0 + e * STEP, end - 4)));
#pragma unroll
      for (int e = 0; e < BATCH; ++e) scale(t0 + e * STEP, x[e]);
    }
  }
};

template <int DT, int DH, int NQ, bool RATIO>
__global__ void __launch_bounds__(kScoreWaves *kWave, plain_waves(DT, DH, NQ)) colsum_kernel(ScoreArgs a) {
  constexpr int NCH = DH * (DT == CKV_BF16 ? 2 : 4) / 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, m = lane & 31, hh = lane >> 5;
  const BlockCoord bc = decode_block(a);

  // accumulator start value -LSE / scale of every row of the group's tiles; -inf on padding rows so
  // that their weights come out as exp2(-inf) = 0
  __shared__ __attribute__((aligned(16))) float s_init[NQ * kTile];
  if (threadIdx.x < NQ * kTile) {
    const int tile = bc.grp * NQ + threadIdx.x / kTile;
    const int j = (tile % a.WT) * kTile + threadIdx.x % kTile;
    const int h = bc.g * a.G + tile / a.WT;
    const bool valid = tile < a.n_tiles && j < a.W;
    float lse_j = 0.0f;
    if (a.lse_from_part)  // as lse_kernel would have it, which this saves when both passes run in one call
      lse_j = merge_row_partials(a.part + ((size_t)bc.unit * a.n_groups + bc.grp) * a.n_chunks * (NQ * kTile) + threadIdx.x,
                                 a.n_chunks, NQ * kTile);
    else if (valid) lse_j = a.lse[((size_t)bc.b * a.Hq + h) * a.W + j];
    s_init[threadIdx.x] = valid ? -lse_j * (kLog2e / a.c2) : -INFINITY;
  }
  chunk_t qf[NQ][NCH];
  int jrow[NQ];
  RatioScale rs;
  if constexpr (RATIO) rs.load(a, bc);
  load_q_tiles<NCH, NQ>(a, bc, m, hh, qf, jrow);
  if constexpr (RATIO) rs.store(a, bc);
  __syncthreads();

  const char *kbase = a.k + bc.b * a.ks_b + bc.g * a.ks_h;
  const int t_begin = (bc.chunk * kScoreWaves + wave) * a.keys_per_wave;
  const int t_end = min(t_begin + a.keys_per_wave, a.T);

  auto tile_body = [&](const chunk_t (&kf)[NCH], int t0) {
    const int kt = t0 + m;  // this lane's key
    float cs[NQ];
    if (t0 + kTile > a.P) {
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int j0 = ((bc.grp * NQ + i) % a.WT) * kTile;
        cs[i] = colsum_tile<DT, NCH, true>(qf[i], kf, a.c2, s_init + i * kTile, hh, kt - a.P - j0);
      }
    } else {
#pragma unroll
      for (int i = 0; i < NQ; ++i) cs[i] = colsum_tile<DT, NCH, false>(qf[i], kf, a.c2, s_init + i * kTile, hh, 0);
    }
    // the other half-wave holds the other 16 rows of each tile: swap and add (all swaps in flight together)
    float other[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) other[i] = __shfl_xor(cs[i], 32);
#pragma unroll
    for (int i = 0; i < NQ; ++i) cs[i] += other[i];
    // one output per head: add the tiles of a head (WT of them), scale by T/W, lanes 0..31 store
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      if (i % a.WT) continue;
      float v = cs[i];
#pragma unroll
      for (int e = 1; e < kMaxWindowTiles; ++e)
        if (e < a.WT && i + e < NQ) v += cs[(i + e) < NQ ? (i + e) : i];
      const int tile = bc.grp * NQ + i;
      if (tile < a.n_tiles && hh == 0 && kt < a.T) {
        const int h = bc.g * a.G + tile / a.WT;
        a.scores[((size_t)bc.b * a.Hq + h) * a.T + kt] = v * a.norm;
      }
    }
  };

  chunk_t ka[NCH], kb[NCH];
  if (t_begin < t_end) load_row<NCH>(ka, kbase + (int64_t)min(t_begin + m, a.T - 1) * a.ks_t, hh);
  for (int t0 = t_begin; t0 < t_end; t0 += 2 * kTile) {
    load_row<NCH>(kb, kbase + (int64_t)min(t0 + kTile + m, a.T - 1) * a.ks_t, hh);
    tile_body(ka, t0);
    if (t0 + kTile >= t_end) break;
    load_row<NCH>(ka, kbase + (int64_t)min(t0 + 2 * kTile + m, a.T - 1) * a.ks_t, hh);
    tile_body(kb, t0 + kTile);
  }
}

// ---------------------------------------------------------------------------------------------
// LDS-staged kernels for bf16 (rows of 128 or 256 bytes).
//
// A load instruction in which every lane addresses a different row touches 32 cache lines and keeps
// the texture-address unit busy several times longer than a contiguous one; with four waves per CU
// the scan then runs at the address unit's pace. These kernels therefore move K (and once per
// workgroup, Q) with global -> LDS loads in which the 64 lanes of one instruction read 1 KiB of whole
// rows, and pick the MFMA operand layout up from LDS with 128-bit reads. Each wave owns a ring of
// four tile images. The image of a 32-row tile holds chunk kappa of row r at
// r * ROW + ((kappa ^ (r & SW)) * 16) so that the operand reads (32 lanes, same chunk, consecutive
// rows) spread over all banks; the load writes lane l's 16 bytes at image offset 16 * (64 * i + l),
// so the swizzle is applied to the source address instead.
//
// One wave per SIMD runs a two-stage software pipeline over (key tile, query tile) pairs: the MFMA
// chain of the next pair is issued in between the vector instructions that consume the current
// pair's logits (two accumulator sets). A lone wave issues one instruction at a time, so everything
// that is not vector arithmetic is kept out of the loop: the loop is unrolled over the ring (image
// addresses become immediates), key tiles are addressed by a running scalar pointer, and the loads
// use the scalar-base form with one M0 write per four instructions (their immediate offset moves the
// global and the LDS address alike, which the per-lane offsets compensate). In pass 2 the -LSE of the
// accumulator rows is folded into the contraction as one more MFMA step whose Q-side operand holds
// -LSE / scale split into three bf16 terms (exact to 2^-24) and whose K-side operand is ones.
// Tiles that touch the window or the end of the keys are handled after the pipeline, masked.
// ---------------------------------------------------------------------------------------------
// Cache policy of the pipeline's output stores (column sums, group sums, utilities): sc1. The outputs
// are consumed by a later kernel, never by this one; with the default policy the stores, although a
// few percent of the pass's bytes, cost it 6-8 us more (measured on the 32k / batch-16 shape).
#ifndef CKV_OUT_STORE_AUX
#define CKV_OUT_STORE_AUX 16
#endif
constexpr int kOutStoreAux = CKV_OUT_STORE_AUX;

template <int DT, int DH>
struct Geom {
  static constexpr int ROW = DH * (DT == CKV_BF16 ? 2 : 4);  // bytes per row
  static constexpr int CH = ROW / 16;                        // 16-byte chunks per row
  static constexpr int NCH = CH / 2;                         // chunks per lane (the other half-wave holds the rest)
  static constexpr int TILE = kTile * ROW;                   // bytes per 32-row tile image
  static constexpr int NDMA = TILE / 1024;                   // load instructions per tile
  static constexpr int SW = (CH < 16 ? CH : 16) - 1;         // swizzle mask
  static_assert(ROW == 128 || ROW == 256, "row size");
};

// Row and chunk of a tile that lane `lane` moves in load instruction i (the lane's 16 bytes land at
// image offset 16 * (64 * i + lane)).
template <class G>
__device__ __forceinline__ void dma_source(int i, int lane, int &r, int &kappa) {
  const int s = i * 64 + lane;
  r = s / G::CH;
  kappa = (s % G::CH) ^ (r & G::SW);
}

template <class G>
__device__ __forceinline__ int image_offset(int r, int kappa) {
  return r * G::ROW + ((kappa ^ (r & G::SW)) << 4);
}

// Waits until at most N of this wave's vector memory operations are still in flight (they complete
// in issue order); also keeps the compiler from moving LDS accesses across the wait.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}

// A wave-uniform pointer as a scalar register pair. The compiler may form uniform 64-bit address
// arithmetic on the vector ALU; operands of the scalar-base loads below must be told apart from that.
__device__ __forceinline__ const char *uniform_ptr(const char *p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char *)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// Four loads with one M0 write: instruction j reads 16 bytes per lane at sbase + voff_j + 1024 * j
// and writes them at LDS address lds + 1024 * j + 16 * lane. STREAM: keys that are not read again before everything else has gone through
// the caches are marked non-temporal, which measurably raises the rate at which HBM delivers them and leaves L2 and the
// memory-side cache to the data that is reused (Q, the column sums on their way to the next kernel). Without it the first pass leaves
// them to the second in the memory-side cache: kKeptKeyBytes draws the line.
template <bool STREAM>
__device__ __forceinline__ void dma_quad(const char *sbase, uint32_t lds, uint32_t v0, uint32_t v1, uint32_t v2,
                                         uint32_t v3) {
  if constexpr (STREAM)
    asm volatile(
        "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %1 offset:0 nt\n\t"
        "global_load_lds_dwordx4 %3, %1 offset:1024 nt\n\t"
        "global_load_lds_dwordx4 %4, %1 offset:2048 nt\n\t"
        "global_load_lds_dwordx4 %5, %1 offset:3072 nt"
        :
        : "s"(lds), "s"(sbase), "v"(v0), "v"(v1), "v"(v2), "v"(v3)
        : "memory");
  else
    asm volatile(
        "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, %1 offset:0\n\t"
        "global_load_lds_dwordx4 %3, %1 offset:1024\n\t"
        "global_load_lds_dwordx4 %4, %1 offset:2048\n\t"
        "global_load_lds_dwordx4 %5, %1 offset:3072"
        :
        : "s"(lds), "s"(sbase), "v"(v0), "v"(v1), "v"(v2), "v"(v3)
        : "memory");
}

// The same with an address of its own for every lane: lane l of instruction j moves 16 bytes from p_j to lds + 1024 * j + 16 * l. In asm like
// the others, since the compiler waits for every load into LDS that it knows of before the next barrier, and by then the first
// key tiles are among them (a barrier behind vmcnt(0) where Q alone had to be there): all waits for these loads are wait_vm()'s. us per
// layer, known to the compiler / not: 4096 keys, 32/32 heads 31.1 / 30.0, 20011, batch 2 56.4 / 55.0, 32768, batch 16 394.3 / 392.7.
__device__ __forceinline__ void dma_quad_rows(uint32_t lds, const char *p0, const char *p1, const char *p2, const char *p3) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "global_load_lds_dwordx4 %2, off offset:1024\n\t"
      "global_load_lds_dwordx4 %3, off offset:2048\n\t"
      "global_load_lds_dwordx4 %4, off offset:3072"
      :
      : "s"(lds), "v"(p0), "v"(p1 - 1024), "v"(p2 - 2048), "v"(p3 - 3072)
      : "memory");
}

// 16 bytes per lane from p to lds + 16 * lane.
__device__ __forceinline__ void dma_one(uint32_t lds, const char *p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(p) : "memory");
}

// A tile of 32 rows whose row r starts at row_of(r), into the image at LDS address lds.
template <class G, class Row>
__device__ __forceinline__ void dma_rows(Row row_of, int lane, uint32_t lds) {
#pragma unroll
  for (int q = 0; q < G::NDMA; q += 4) {
    const char *src[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int r, kappa;
      dma_source<G>(q + i, lane, r, kappa);
      src[i] = row_of(r) + kappa * 16;
    }
    dma_quad_rows(lds + q * 1024, src[0], src[1], src[2], src[3]);
  }
}

// One whole tile whose first row starts at tile_base. voff[i] already holds the lane's source offset in the first quad
// minus the immediate of its instruction plus kDmaBias, so the scalar base is tile_base - kDmaBias; the second quad reads the
// same chunks (the swizzle repeats every sixteen rows) quad_stride = 16 rows further on.
constexpr int kDmaBias = 3072;
template <class G, bool STREAM>
__device__ __forceinline__ void dma_tile(const char *tile_base, const uint32_t (&voff)[4], int64_t quad_stride, uint32_t lds_image) {
  static_assert(G::NDMA == 4 || (G::NDMA == 8 && G::CH == 16), "a quad is sixteen rows of sixteen chunks");
#pragma unroll
  for (int q = 0; q < G::NDMA / 4; ++q)
    dma_quad<STREAM>(tile_base - kDmaBias + q * quad_stride, lds_image + q * 4096, voff[0], voff[1], voff[2], voff[3]);
}

template <class G>
__device__ __forceinline__ void read_image(chunk_t (&f)[G::NCH], const char *image, const int (&roff)[G::NCH]) {
#pragma unroll
  for (int c = 0; c < G::NCH; ++c) f[c] = *reinterpret_cast<const chunk_t *>(image + roff[c]);
}

// Scheduling hint for one pipeline step: N_MFMA groups of one MFMA, (where the step also picks up the
// next key tile) one LDS read, and a few vector instructions.
template <int N_MFMA, int VALU_PER, int N_DS>
__device__ __forceinline__ void interleave_hint() {
#pragma unroll
  for (int u = 0; u < N_MFMA; ++u) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                 // one MFMA
    if (u < N_DS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
    __builtin_amdgcn_sched_group_barrier(0x002, VALU_PER, 0);          // then a few vector instructions
  }
}

// Key tiles per unrolled body of the pipelines. Up to four query tiles per wave the body is a whole ring
// cycle (every ring image address is an immediate). Beyond that a body of four tiles holds so many
// scheduling-hint groups that the compiler's solver for them needs minutes per kernel; half a cycle
// keeps it at seconds, and the ring image of a body's first tile becomes a run-time (scalar) value.
__host__ __device__ constexpr int unroll_tiles(int nq) { return nq > 4 ? 2 : kRing; }
static_assert(kRing % 2 == 0, "half a ring cycle starts at an even image");

// Vector instructions that the hint places behind each MFMA of the next pair's chain. Fewer than an even
// spread (pass 1 has ~59 per 8 MFMAs, pass 2 ~48 per 9): the chain is then issued early, and what is left
// of the current pair's vector work runs after its last MFMA -- the 18 wait states between an MFMA and the
// first read of its result are filled with work instead of s_nop (one `s_nop 11` per pair with an even
// spread). us per layer (passes 1 / 2, instructions per MFMA): 131072 keys, W = 64, eight tiles per wave: 172.2 (6 / 4), 175.0 (6 / 5), 169.7
// (6 / 3), 170.8 (5 / 4); another card 176.9 (6 / 3), 175.5 (5 / 3), 178.3 (4 / 3), 180.6 (5 / 2); 65536 keys, seven tiles, the same order. Four tiles,
// 32768 keys, batch 16: 399.2 (5 / 5), 401.0 (5 / 6), 398.9 (5 / 4), pass 1 at 6 or 4 another 1 to 2 % slower; 20011, batch 2 56.0, 56.2, 56.4; 10006
// with value norms 69.2, 69.4, 69.3.
__host__ __device__ constexpr int vector_per_mfma_pass1(int nq) { return 5; }
__host__ __device__ constexpr int vector_per_mfma_pass2(int nq) { return nq > 4 ? 3 : 5; }

// The tiles behind the pipeline run the same two stages over the query tiles of one key tile (the masks make their vector part
// half as long again).
constexpr int kTailVectorPerMfma = 8;

// Geometry of a wave's key range: wave-uniform values live in scalar registers.
struct WaveRange {
  int wave, t_begin, t_end;
  int n_full;   // tiles wholly inside the prefix
  int n_whole;  // tiles wholly inside the keys
  int n_all;    // the tiles to take: one more than n_whole where the keys end inside a tile
};
// `last`: the keys whose sums are wanted end here, T or (utilities) P.
__device__ __forceinline__ WaveRange wave_range(const ScoreArgs &a, const BlockCoord &bc, int last) {
  WaveRange r;
  r.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  r.t_begin = (bc.chunk * kScoreWaves + r.wave) * a.keys_per_wave;
  r.t_end = min(r.t_begin + a.keys_per_wave, a.T);
  r.n_full = max(0, (min(r.t_end, a.P) - r.t_begin) / kTile);
  r.n_whole = max(0, r.t_end - r.t_begin) / kTile;
  r.n_all = (max(0, min(r.t_end, last) - r.t_begin) + kTile - 1) / kTile;
  return r;
}

// Everything the two staged kernels share: the ring, the per-lane offsets, Q in registers.
#ifndef CKV_PIN_Q_ABOVE
#define CKV_PIN_Q_ABOVE 4
#endif
// The barriers of Staged::start, in order. A barrier waits for every wave of the workgroup, so waves that do other work beside the
// scan's pass all of them as well: one more or one less is a line here, and theirs follow.
enum StartBarrier { kQueriesLanded, kQueriesRead, kStartBarriers };
template <int WHICH>
__device__ __forceinline__ void start_barrier() {
  static_assert(WHICH < kStartBarriers, "every barrier of the start has a name");
  __syncthreads();
}

// LEAN: registers are short (another wave shares the SIMD), operand addresses are formed at each read.
template <int DT, int DH, int NQ, bool STREAM, bool LEAN = false>
struct Staged {
  using G = Geom<DT, DH>;
  static constexpr int NCH = G::NCH;
  typedef char Ring[kScoreWaves][kRing][G::TILE];
  uint32_t voff[4];        // lane's biased source offset inside a K tile, per load instruction of a quad
  int roff[NCH];           // lane's operand chunks inside a tile image
  uint32_t rbase;          // LEAN: the first of them in the wave's first image (the others differ in three bits)
  const char *kbase;       // first key row of the unit
  const char *kcur;        // first row of the key tile the pipeline is working on
  const char *kend;        // first row of the wave's last tile (what the loads beyond it fetch again)
  int64_t tile_stride;
  uint32_t lds_ring;       // LDS address of this wave's first image

  // Starts the loads of Q (wave w moves query tiles w and w + 4 into the last images of its ring) and of the
  // first key tiles, then hands every wave all NQ query tiles in registers; on return the wave's first
  // tiles_asked() key tiles are in flight, in order. jrow[i] = window row of tile i, row m, or -1 on padding.
  static constexpr int QI = (NQ + kScoreWaves - 1) / kScoreWaves;  // ring images per wave that first hold Q
  static_assert(QI >= 1 && QI <= kRing - 2, "query tiles pass through the ring's last images");
  static constexpr int N_PRE = kRing - QI;  // key tiles whose images are free while Q passes through
  // Key tiles of a wave with any whose loads start() has queued; the only tile of a sequence shorter than one fills the images
  // that are free beside Q, and no more.
  static __device__ __forceinline__ int tiles_asked(const ScoreArgs &a) { return a.T < kTile ? N_PRE : kRing - 1; }
  // `first` queues loads in front of all others, which have landed as Q has; `between` runs when every wave's have, with the query
  // tiles still in their images (image_of_tile), in front of the start's last barrier.
  template <class First, class Between>
  __device__ __forceinline__ void start(const ScoreArgs &a, const BlockCoord &bc, const WaveRange &wr, Ring &ring, int lane, int m,
                                        int hh, chunk_t (&qf)[NQ][NCH], int (&jrow)[NQ], First first, Between between) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      int r, kappa;
      dma_source<G>(i, lane, r, kappa);
      voff[i] = (uint32_t)(r * a.ks_t + kappa * 16 + kDmaBias - i * 1024);
    }
#pragma unroll
    for (int c = 0; c < NCH; ++c) roff[c] = image_offset<G>(m, c + NCH * hh);
    kbase = uniform_ptr(a.k + bc.b * a.ks_b + bc.g * a.ks_h);
    kcur = uniform_ptr(kbase + (int64_t)wr.t_begin * a.ks_t);
    tile_stride = (int64_t)kTile * a.ks_t;
    kend = uniform_ptr(wr.n_all > wr.n_whole ? kbase + (int64_t)max(a.T - kTile, 0) * a.ks_t
                                             : kcur + max(wr.n_whole - 1, 0) * tile_stride);
    lds_ring = (uint32_t)(uintptr_t)&ring[wr.wave][0][0];
    if (LEAN) rbase = lds_ring + image_offset<G>(m, NCH * hh);

    first();
#pragma unroll
    for (int qi = 0; qi < QI; ++qi) {
      if (wr.wave + qi * kScoreWaves < NQ) {
        const int tile = min(bc.grp * NQ + wr.wave + qi * kScoreWaves, a.n_tiles - 1);
        const char *qhead = a.q + bc.b * a.qs_b + (bc.g * a.G + tile / a.WT) * a.qs_h;
        const int j0 = (tile % a.WT) * kTile;
        dma_rows<G>([&](int r) { return qhead + (int64_t)min(j0 + r, a.W - 1) * a.qs_w; }, lane, lds_ring + (kRing - 1 - qi) * G::TILE);
      }
    }
    const bool tiny = a.T < kTile;
    if (wr.n_all > 0) {
      if (!tiny) {
#pragma unroll
        for (int d = 0; d < N_PRE; ++d)
          dma_tile<G, STREAM>(d < wr.n_whole ? kcur + d * tile_stride : kend, voff, tile_stride / 2, lds_ring + d * G::TILE);
      } else {  // the only tile of a sequence shorter than one: rows are clamped (whoever uses them masks their logits)
#pragma unroll
        for (int d = 0; d < N_PRE; ++d)
          dma_rows<G>([&](int r) { return kbase + (int64_t)min(r, a.T - 1) * a.ks_t; }, lane, lds_ring + d * G::TILE);
      }
      wait_vm<N_PRE * G::NDMA>();  // Q has landed, the key tiles may still be on their way
    } else {
      wait_vm<0>();
    }
    start_barrier<kQueriesLanded>();
#pragma unroll
    for (int i = 0; i < NQ; ++i) read_image<G>(qf[i], image_of_tile(ring, i), roff);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int tile = bc.grp * NQ + i;
      const int j = (tile % a.WT) * kTile + m;
      const bool valid = tile < a.n_tiles && j < a.W;
      jrow[i] = valid ? j : -1;
      if (!valid) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) qf[i][c] = chunk_t{0u, 0u, 0u, 0u};
      }
      // With more than four query tiles the ordinary vector registers are what runs out (the logits, the key
      // tile and the vector work's temporaries must live there), while the matrix cores take their operands
      // from accumulation registers just as well: say where Q is to live, or the allocator keeps a tile of it
      // in vector registers and serialises the exponentials through one temporary.
      if constexpr (NQ > CKV_PIN_Q_ABOVE) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) asm volatile("" : "+a"(qf[i][c]));
      }
    }
    between();
    start_barrier<kQueriesRead>();  // the images that held Q are free for key tiles from here on
    if (wr.n_all > 0 && !tiny) {
#pragma unroll
      for (int d = N_PRE; d < kRing - 1; ++d)
        dma_tile<G, STREAM>(d < wr.n_whole ? kcur + d * tile_stride : kend, voff, tile_stride / 2, lds_ring + d * G::TILE);
    }
  }

  static __device__ __forceinline__ const char *image_of_tile(Ring &ring, int i) {
    return ring[i % kScoreWaves][kRing - 1 - i / kScoreWaves];
  }

  // Load of the tile three ahead of the one at kcur (tile index t + 3) into ring image `slot`; past
  // the last tile the last one is fetched again (in bounds, unused).
  __device__ __forceinline__ void prefetch(int t, int n_whole, int slot) {
    dma_tile<G, STREAM>(t + 3 < n_whole ? kcur + 3 * tile_stride : kend, voff, tile_stride / 2, lds_ring + slot * G::TILE);
  }

  // Operand chunks of the tile in ring image `slot`.
  __device__ __forceinline__ void read(chunk_t (&f)[NCH], const WaveRange &wr, Ring &ring, int slot) {
    if constexpr (LEAN) {
      typedef __attribute__((address_space(3))) const chunk_t lds_chunk_t;
      uint32_t at = rbase;
      asm volatile("" : "+v"(at));  // or the eight addresses are kept in registers
#pragma unroll
      for (int c = 0; c < NCH; ++c) f[c] = *(lds_chunk_t *)(uintptr_t)((at ^ (c << 4)) + slot * G::TILE);
    } else {
      read_image<G>(f, ring[wr.wave][slot], roff);
    }
  }

  // Tile t (behind the pipeline, at kcur) into registers: its load was issued three tiles ago, as the pipeline's are. A tile that
  // the keys end in comes as the last 32 rows of them, `shift` rows in front of it; lanes beyond the keys take the last one.
  __device__ __forceinline__ void tail_tile(const WaveRange &wr, Ring &ring, int t, int shift, int m, int hh, chunk_t (&kf)[NCH]) {
    if (t + 3 < wr.n_all) {
      prefetch(t, wr.n_whole, (t + 3) % kRing);
      wait_vm<(kRing - 1) * G::NDMA>();
    } else {
      wait_vm<0>();
    }
    read_tail(wr, ring, t, shift, m, hh, kf);
    kcur += tile_stride;
  }
  __device__ __forceinline__ void read_tail(const WaveRange &wr, Ring &ring, int t, int shift, int m, int hh, chunk_t (&kf)[NCH]) {
    if (t < wr.n_whole) {
      read(kf, wr, ring, t % kRing);
    } else {
      // fewer than 32 keys at all: the image's rows are clamped already
      const int row = shift > t * kTile + wr.t_begin ? m : min(m + shift, kTile - 1);
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        kf[c] = *reinterpret_cast<const chunk_t *>(ring[wr.wave][t % kRing] + image_offset<G>(row, c + NCH * hh));
    }
  }
};

// Value norms (paper Eq. 4, r_t = ||v_t||) of the workgroup's key range by four more waves of pass 1. Wave w takes the rows that
// wave w of vnorm_rows_kernel takes, and the sums of blocks of kVnormRows rows are formed in that kernel's order: the same
// bits. DEPTH - 1 steps' loads are in flight beside a step; the norm of a row ends in one lane of those that hold it, so
// that a step takes one root and one store. Bound by memory: 16384 keys, batch 4, K and V 50 us at 5.4 TB/s over the launch, one
// behind the other 32 + 23; four steps in registers, or a higher priority for either kind of wave, 0 to 2 % slower.
template <int DH>
struct NormWaves {
  static constexpr int LPR = DH / 8;                     // lanes (16-byte pieces) per row
  static constexpr int RPL = kWave / LPR;                // adjacent rows per load
  static constexpr int APART = kScoreWaves * RPL;        // rows from one load to the next
  static constexpr int U = 8, STEP = U * APART;          // loads of a step, rows of a step of all waves
  static constexpr int DEPTH = 3;                        // steps in registers
  static_assert(U <= LPR, "a lane per load keeps its row's norm");
  static_assert(kVnormRows % STEP == 0, "whole steps per block");
  typedef float Sums[4096 * kScoreWaves / kVnormRows][kScoreWaves];  // per block of the longest range and wave
  static __device__ __forceinline__ void load(uint4 (&c)[U], const char *base, int64_t stride, int row, int end, int sub) {
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = load_piece<true>(base + (int64_t)min(row + u * APART, end - 1) * stride + sub * 16);
  }
  static __device__ __forceinline__ void run(const ScoreArgs &a, const BlockCoord &bc, int wave, int lane, Sums &sums) {
    const int begin = bc.chunk * kScoreWaves * a.keys_per_wave, end = min(begin + kScoreWaves * a.keys_per_wave, a.T);
    const char *base = a.v + bc.b * a.vs_b + bc.g * a.vs_h;
    float *out = a.ratio + (size_t)bc.unit * a.T;
    const int sub = lane % LPR;
    float local = 0.0f;
    uint4 c[DEPTH][U];
    int row = begin + wave * RPL + lane / LPR;  // of the step's first load
#pragma unroll
    for (int i = 0; i < DEPTH - 1; ++i) load(c[i], base, a.vs_t, row + i * STEP, end, sub);
    const auto step = [&](uint4 (&now)[U], uint4 (&next)[U]) {
      load(next, base, a.vs_t, row + (DEPTH - 1) * STEP, end, sub);
      float mine = 0.0f;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t w[4] = {now[u].x, now[u].y, now[u].z, now[u].w};
        float sq = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __uint_as_float(w[e] << 16), hi = __uint_as_float(w[e] & 0xffff0000u);
          sq = fmaf(lo, lo, sq);
          sq = fmaf(hi, hi, sq);
        }
        sq = row_sum<LPR>(sq);
        mine = sub == u ? sq : mine;
      }
      const int t = row + sub * APART;
      float nrm = sqrtf(mine);
      if (sub < U && t < end) out[t] = nrm;
      nrm = t < end ? nrm : 0.0f;
      // lane 0 of a row's lanes adds the step's norms in the order of the rows
      local += nrm;
      local += from_lane<1>(nrm);
      local += from_lane<2>(nrm);
      local += from_lane<3>(nrm);
      local += from_lane<4>(nrm);
      local += from_lane<5>(nrm);
      local += from_lane<6>(nrm);
      local += from_lane<7>(nrm);
      row += STEP;
    };
#pragma unroll
    for (int i = 0; i < kStartBarriers; ++i) __builtin_amdgcn_s_barrier();  // with the first loads on their way
    for (int first = begin, i = 0; first < end;) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        if (first >= end) break;
        step(c[d], c[(d + DEPTH - 1) % DEPTH]);
        first += STEP;
        if ((first - begin) % kVnormRows == 0 || first >= end) {
          float s = sub == 0 ? local : 0.0f;
#pragma unroll
          for (int o = 32; o >= LPR; o >>= 1) s += __shfl_xor(s, o);
          if (lane == 0) sums[i][wave] = s;
          ++i;
          local = 0.0f;
        }
      }
    }
    __syncthreads();  // the one of store_row_partials
    const int block = wave * kWave + lane, n_blocks = (end - begin + kVnormRows - 1) / kVnormRows;
    if (block < n_blocks)
      a.vsum[(size_t)bc.unit * a.vnorm_blocks + begin / kVnormRows + block] =
          (sums[block][0] + sums[block][1]) + (sums[block][2] + sums[block][3]);
  }
  template <int N>
  static __device__ __forceinline__ float from_lane(float x) {  // of N lanes further on in the row of sixteen
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x100 + N, 0xF, 0xF, true));
  }
};

template <int DT, int DH, int NQ, bool NORMS = false, bool KEEP = false>
__global__ void __launch_bounds__(kScoreWaves *kWave * (NORMS ? 2 : 1)) rowstats_lds_kernel(ScoreArgs a) {
  using G = Geom<DT, DH>;
  constexpr int NCH = G::NCH;
  constexpr int N_MFMA = NCH * (DT == CKV_BF16 ? 1 : 4);
  constexpr bool STREAM = !KEEP;
  constexpr bool LEAN = NORMS && NQ == kMaxQTilesNorms;
  // query tile during which the next key tile is picked up; LEAN: when the last chain of the present one has been issued, into
  // the same registers (with a second set 18 registers spilled, and a reload waits for the loads in flight: 54 us for 50)
  constexpr int READ_AT = LEAN ? NQ - 1 : NQ >= 2 ? NQ - 2 : 0;
  constexpr int NEXT = LEAN ? 0 : 1;
  __shared__ __attribute__((aligned(1024))) typename Staged<DT, DH, NQ, STREAM>::Ring ring;
  const int lane = threadIdx.x & 63, m = lane & 31, hh = lane >> 5;
  const BlockCoord bc = decode_block(a);
  if constexpr (NORMS) {
    __shared__ typename NormWaves<DH>::Sums s_norms;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - kScoreWaves;
    if (wave >= 0) {
      NormWaves<DH>::run(a, bc, wave, lane, s_norms);
      return;
    }
  }
  const WaveRange wr = wave_range(a, bc, a.T);

  Staged<DT, DH, NQ, STREAM, LEAN> st;
  chunk_t qf[NQ][NCH];
  int jrow[NQ];
  st.start(a, bc, wr, ring, lane, m, hh, qf, jrow, [] {}, [] {});
  float rm[NQ], rl[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    rm[i] = -1e30f;
    rl[i] = 0.0f;
  }

  chunk_t kreg[1 + NEXT][NCH];
  f32x16 acc[2];
  const int n_piped = wr.n_full / kRing * kRing;  // the pipeline takes key tiles one ring at a time
  if (n_piped > 0) {
    wait_vm<(kRing - 2) * G::NDMA>();
    st.read(kreg[0], wr, ring, 0);
    mma_chain<DT, NCH>(acc[0], kreg[0], qf[0]);
  }
  constexpr int UR = unroll_tiles(NQ);
  for (int t0 = 0; t0 < n_piped; t0 += UR) {
    const int slot0 = UR == kRing ? 0 : (t0 & (kRing - 1));  // ring image of tile t0
#pragma unroll
    for (int v = 0; v < UR; ++v) {  // tile t0 + v lives in image u and in kreg[v & 1]
      const int u = slot0 + v;
      st.prefetch(t0 + v, wr.n_whole, (u + kRing - 1) % kRing);
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int cur = (v * NQ + i) & 1;  // accumulator set holding this pair's logits
        if (i == READ_AT) {
          wait_vm<(kRing - 2) * G::NDMA>();  // tile t0 + v + 1 has landed
          st.read(kreg[(v + 1) & NEXT], wr, ring, (u + 1) % kRing);
        }
        // logits of the next pair; the last pair of a key tile already starts the next key tile
        if (i + 1 < NQ) mma_chain<DT, NCH>(acc[cur ^ 1], kreg[v & NEXT], qf[i + 1]);
        else mma_chain<DT, NCH>(acc[cur ^ 1], kreg[(v + 1) & NEXT], qf[0]);
        rowstats_update<false>(acc[cur], a.c2, 0, hh, 0, rm[i], rl[i]);
        if (LEAN && i == READ_AT) {  // the chain waits for the reads
          __builtin_amdgcn_sched_group_barrier(0x100, NCH, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 32, 0);
          interleave_hint<N_MFMA, 4, 0>();
        } else if (i == READ_AT) interleave_hint<N_MFMA, vector_per_mfma_pass1(NQ), NCH>();
        else interleave_hint<N_MFMA, vector_per_mfma_pass1(NQ), 0>();
      }
      st.kcur += st.tile_stride;
    }
  }
  // What the pipeline left: up to a ring of whole tiles and the masked ones.
  for (int t = n_piped; t < wr.n_all; ++t) {
    const int t0 = wr.t_begin + t * kTile;
    st.tail_tile(wr, ring, t, t0 - (a.T - kTile), m, hh, kreg[0]);
    mma_chain<DT, NCH>(acc[0], kreg[0], qf[0]);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      if (i + 1 < NQ) mma_chain<DT, NCH>(acc[(i + 1) & 1], kreg[0], qf[i + 1]);
      const int tile = bc.grp * NQ + i, j = (tile % a.WT) * kTile + m;
      const int limit = tile < a.n_tiles && j < a.W ? a.P + j : -1;  // last key this row may see (causal)
      rowstats_update<true>(acc[i & 1], a.c2, t0, hh, limit, rm[i], rl[i]);
      if (i + 1 < NQ) interleave_hint<N_MFMA, kTailVectorPerMfma, 0>();
    }
  }
  store_row_partials<NQ>(a, bc, wr.wave, m, hh, rm, rl);
  wait_vm<0>();  // the loads beyond the last tile write LDS: not after the wave
}

// The extra contraction step of pass 2 that adds bias_j = -LSE_j / scale to every logit of query row j: the bias as hi + mid + lo
// bf16 terms in the first three slots of the Q-side operand of the lanes with hh = 0, ones in the same slots on the K side. The
// terms are made once per row (pack) and reach the lanes through LDS. (In registers, as the addend of the scale's multiplication, the
// normalisers save the ninth MFMA of a pair and 0.5 to 1.4 % of a layer; but they round differently, and keys within 1e-6 of a
// threshold change places.) Padding rows (q = 0) get exp2(kNoWeight) = 0 as weight.
constexpr float kNoWeight = -1000.0f;
__device__ __forceinline__ uint32_t bf16_bits(float x) {  // round to nearest even; x is finite
  const uint32_t u = __float_as_uint(x);
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
struct RowBias {
  chunk_t q;
  static __device__ __forceinline__ uint2 pack(float bias) {
    const uint32_t hi = bf16_bits(bias);
    const float r1 = bias - __uint_as_float(hi << 16);
    const uint32_t mid = bf16_bits(r1);
    const float r2 = r1 - __uint_as_float(mid << 16);
    return make_uint2(hi | (mid << 16), bf16_bits(r2));
  }
  __device__ __forceinline__ void set(const uint2 *rows, int m, int hh) {  // rows: of the tile
    const uint2 v = rows[m];
    q = hh == 0 ? chunk_t{v.x, v.y, 0u, 0u} : chunk_t{0u, 0u, 0u, 0u};
  }
  __device__ __forceinline__ void add(f32x16 &acc, int hh) const {
    Mma<CKV_BF16>::step(acc, q, hh == 0 ? chunk_t{0x3f803f80u, 0x3f80u, 0u, 0u} : chunk_t{0u, 0u, 0u, 0u});
  }
};

// Weights exp(z - LSE) of one tile from acc = <q, k> - LSE / scale, summed over this lane's 16 rows.
template <bool EDGE>
__device__ __forceinline__ float colsum_weights(const f32x16 &acc, float c2, int hh, int first_masked_row) {
  float s[4];
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float pr = __builtin_amdgcn_exp2f(acc[r] * c2);
    // causal: key kt is visible to window row j iff kt <= P + j, i.e. tile row >= kt - P - j0
    if (EDGE && acc_row(r, hh) < first_masked_row) pr = 0.0f;
    s[r & 3] = r < 4 ? pr : s[r & 3] + pr;
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Adds the two half-waves' row sums and stores one value per (head, key). Heads are taken in pairs:
// v_permlane32_swap turns (x, y) into ([x.lo, y.lo], [x.hi, y.hi]), so one add leaves head x's
// totals in lanes 0..31 and head y's in lanes 32..63, and all 64 lanes store.
template <int NQ>
__device__ __forceinline__ void store_column_sums(const ScoreArgs &a, const BlockCoord &bc, const float (&cs)[NQ],
                                                  int WT, int kt, int hh) {
  float hv[NQ];  // per head of the group (NQ / WT of them), the sum over its tiles
  int nh = 0;
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    if (i % WT == 0) hv[nh++] = cs[i];
    else hv[nh - 1] += cs[i];
  }
  const int head0 = bc.g * a.G + (bc.grp * NQ) / WT;  // first head of the group
  const int heads_left = a.G - (bc.grp * NQ) / WT;    // heads of the KV group from there on
#pragma unroll
  for (int h = 0; h < NQ; h += 2) {
    if (h >= nh) break;
    const float x = hv[h], y = hv[(h + 1 < nh) ? h + 1 : h];
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    const float tot = (__uint_as_float(sw[0]) + __uint_as_float(sw[1])) * a.norm;
    const int mine = h + hh;  // lanes 32..63 carry the second head of the pair
    if (mine < nh && mine < heads_left && kt < a.T) a.scores[((size_t)bc.b * a.Hq + head0 + mine) * a.T + kt] = tot;
  }
}

// Group-sum form of the same: one value per key, the sum over the group's heads.
template <int NQ>
__device__ __forceinline__ void store_group_sum(const ScoreArgs &a, const BlockCoord &bc, const float (&cs)[NQ], int kt,
                                                int hh) {
  float x = cs[0];  // padding heads have zero query rows and kNoWeight: their weights are exactly 0
#pragma unroll
  for (int i = 1; i < NQ; ++i) x += cs[i];
  const float tot = (x + __shfl_xor(x, 32)) * a.norm;
  if (hh == 0 && kt < a.T) a.scores[((size_t)bc.b * a.Hkv + bc.g) * a.T + kt] = tot;
}

// Pipeline form of the same: the totals of one key tile go to a per-wave LDS stage
// [head of the group][key of the ring cycle], and once per ring cycle (4 tiles, 128 keys) every lane
// stores four consecutive keys of one head with one 128-bit buffer store per pair of heads.
template <int NQ, int WT, int ROW = kRing * kTile>
__device__ __forceinline__ void stage_column_sums(const float (&cs)[NQ], float norm, float *stage, int at, int hh) {
  constexpr int NH = NQ / WT;
  float hv[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    hv[h] = cs[h * WT];
#pragma unroll
    for (int e = 1; e < WT; ++e) hv[h] += cs[h * WT + e];
  }
#pragma unroll
  for (int h = 0; h < NH; h += 2) {
    const float x = hv[h], y = hv[(h + 1 < NH) ? h + 1 : h];
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    const float tot = (__uint_as_float(sw[0]) + __uint_as_float(sw[1])) * norm;
    if (h + hh < NH) stage[(h + hh) * ROW + at] = tot;
  }
}

// The stage is written by one set of lanes and read by another of the same wave. The hardware keeps a
// wave's LDS operations in order, but the compiler, reasoning per lane, sees a store and a load that can
// never touch the same word and may swap them: this keeps every memory access on its side of the line.
__device__ __forceinline__ void stage_fence() { asm volatile("" ::: "memory"); }

template <int NQ, int WT>
__device__ __forceinline__ void flush_column_sums(const ScoreArgs &a, const BlockCoord &bc, const float *stage,
                                                  int t_first, int lane, __amdgpu_buffer_rsrc_t rsrc) {
  constexpr int NH = NQ / WT;
  const int head0 = bc.g * a.G + (bc.grp * NQ) / WT;
  const int heads_left = a.G - (bc.grp * NQ) / WT;
#pragma unroll
  for (int h = 0; h < NH; h += 2) {
    const int mine = h + (lane >> 5), key4 = 4 * (lane & 31);
    const bool valid = mine < NH && mine < heads_left;
    const f32x4 v = *reinterpret_cast<const f32x4 *>(stage + (valid ? mine : 0) * (kRing * kTile) + key4);
    const uint32_t off = valid ? (uint32_t)(((head0 + mine) * a.T + t_first + key4) * 4) : 0x80000000u;
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), rsrc, off, 0, kOutStoreAux);
  }
}

// Group-sum form of the flush (layer-shared mode: the prompt's alpha is a mean over heads, so only the
// sum over a KV head's query heads is needed): lanes 0..31 add the even heads of the stage, lanes
// 32..63 the odd ones, four consecutive keys each; the halves are added and lanes 0..31 store one
// 128-bit piece of the single output row -- a quarter of the per-head form's bytes for groups of four.
template <int NQ>
__device__ __forceinline__ void flush_group_sums(const ScoreArgs &a, const BlockCoord &bc, const float *stage,
                                                 int t_first, int lane, __amdgpu_buffer_rsrc_t rsrc_g) {
  const int half = lane >> 5, key4 = 4 * (lane & 31);
  const int heads_left = a.G - bc.grp * NQ;
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int h = 0; h < NQ; h += 2) {
    const int mine = h + half;
    if (mine < NQ && mine < heads_left) acc += *reinterpret_cast<const f32x4 *>(stage + mine * (kRing * kTile) + key4);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], 32);
  const uint32_t off = half == 0 ? (uint32_t)((bc.g * a.T + t_first + key4) * 4) : 0x80000000u;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, acc), rsrc_g, off, 0, kOutStoreAux);
}

// Fused form of the flush (ckv_window_utility): instead of the column sums, the wave writes the
// UTILITY -- pooled along the keys, weighted per head, maximum over the group's heads (paper Eq. 6) --
// straight from the stage. A stage row holds, in front of the block's 128 values, the last 40 of the
// previous block, and each flush covers the 128 keys that END 32 keys before the block does: every
// pooling window (radius <= 3) lies inside the row and every store covers whole 128-byte lines
// (partial lines proved expensive). What this leaves out per wave range -- the first four keys, the
// last 32 keys of the pipelined part, and the tail tiles -- finish_utility writes behind a barrier, when the
// neighbours' sums are known. Lanes 0..31 take the even heads of the group, lanes 32..63 the odd ones,
// four consecutive keys each (three 128-bit reads per head); the halves then swap so that each lane
// ends up with the group maximum of two adjacent keys and stores them with one 64-bit store. The taps
// are combined left to right, as the stand-alone tables kernel does.
constexpr int kUtilRow = kUtilCarry + kRing * kTile;
// win[hp]: the twelve values around this lane's four keys (win[hp][4 .. 7]) of head 2 hp + half.
template <int NH, int POOL, int R>
__device__ __forceinline__ void pooled_group_max(const ScoreArgs &a, const float (&win)[(NH + 1) / 2][12], int lane,
                                                 int heads_left, const float (&wgt)[NH], float (&best)[4]) {
  const int half = lane >> 5;
#pragma unroll
  for (int e = 0; e < 4; ++e) best[e] = -INFINITY;
#pragma unroll
  for (int hp = 0; hp < (NH + 1) / 2; ++hp) {
    const int h = 2 * hp + half;
    const bool live = h < NH && h < heads_left;
    float wg = 0.0f;
#pragma unroll
    for (int x = 0; x < NH; ++x) wg = (x == h) ? wgt[x] : wg;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float c = win[hp][4 + e - R];
#pragma unroll
      for (int d = 1 - R; d <= R; ++d) c = POOL == CKV_POOL_MAX ? fmaxf(c, win[hp][4 + e + d]) : c + win[hp][4 + e + d];
      // the quotient to the last bit, as the tables kernel's division has it (c times the rounded reciprocal was up to 9 % further
      // from 64 bits over whole layers: a bias of its own)
      if (POOL == CKV_POOL_AVG) c = fmaf(c, a.inv_kernel, c * a.inv_kernel_rest);
      // a select, not a branch: heads that do not exist leave the maximum alone
      best[e] = fmaxf(best[e], live ? wg * c : -INFINITY);
    }
  }
}

template <int NH>
__device__ __forceinline__ void pooled_best(const ScoreArgs &a, const float (&win)[(NH + 1) / 2][12], int lane,
                                            int heads_left, const float (&wgt)[NH], float (&best)[4]) {
  if (a.pool == CKV_POOL_MAX) {
    switch (a.radius) {
      case 1: pooled_group_max<NH, CKV_POOL_MAX, 1>(a, win, lane, heads_left, wgt, best); break;
      case 2: pooled_group_max<NH, CKV_POOL_MAX, 2>(a, win, lane, heads_left, wgt, best); break;
      case 3: pooled_group_max<NH, CKV_POOL_MAX, 3>(a, win, lane, heads_left, wgt, best); break;
      default: pooled_group_max<NH, CKV_POOL_MAX, 0>(a, win, lane, heads_left, wgt, best); break;
    }
  } else {
    switch (a.radius) {
      case 1: pooled_group_max<NH, CKV_POOL_AVG, 1>(a, win, lane, heads_left, wgt, best); break;
      case 2: pooled_group_max<NH, CKV_POOL_AVG, 2>(a, win, lane, heads_left, wgt, best); break;
      case 3: pooled_group_max<NH, CKV_POOL_AVG, 3>(a, win, lane, heads_left, wgt, best); break;
      default: pooled_group_max<NH, CKV_POOL_AVG, 0>(a, win, lane, heads_left, wgt, best); break;
    }
  }
}

// rows: the wave's stage rows (carry included); edge: where the first block leaves its first kUtilHead sums; t_first:
// first key of the block just staged. Every LDS read of the flush is issued before anything waits for one (the wave is alone on its SIMD: a read's
// latency is otherwise paid once per dependent step).
template <int NQ, int WT>
__device__ __forceinline__ void flush_utility(const ScoreArgs &a, const BlockCoord &bc, float *rows, float *edge,
                                              int t_first, bool first_block, int lane, __amdgpu_buffer_rsrc_t rsrc_u,
                                              const float (&wgt)[NQ / WT]) {
  constexpr int NH = NQ / WT;
  constexpr int NP = (NH + 1) / 2;  // pairs of heads: lanes 0..31 take the even head, lanes 32..63 the odd one
  constexpr int BLK = kRing * kTile;
  const int heads_left = a.G - (bc.grp * NQ) / WT;
  const int half = lane >> 5, grp = lane & 31, key4 = 4 * grp;
  typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  // -- reads: the pooling windows, the pieces of the carry
  float win[NP][12];
#pragma unroll
  for (int hp = 0; hp < NP; ++hp) {
    const int mine = 2 * hp + half;
    const float *row = rows + (mine < NH ? mine : 0) * kUtilRow;
    const float *w0 = row + (kUtilCarry - kUtilShift - 4) + key4;  // w0[4 .. 7]: keys 4 grp - 32 .. of the block
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const f32x4 v = *reinterpret_cast<const f32x4 *>(w0 + 4 * q);
#pragma unroll
      for (int e = 0; e < 4; ++e) win[hp][4 * q + e] = v[e];
    }
  }
  constexpr int PER = kUtilCarry / 4;  // 128-bit pieces of the carry per head
  constexpr int NC = (PER * NH + kWave - 1) / kWave;
  static_assert(NC <= 2, "at most two pieces per lane");
  f32x4 carry[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int piece = lane + i * kWave;
    const int pc = piece < PER * NH ? piece : 0;
    carry[i] = *reinterpret_cast<const f32x4 *>(rows + (pc / PER) * kUtilRow + BLK + 4 * (pc % PER));
  }
  // -- carry: the block's last kUtilCarry values move in front of the rows for the next block (LDS operations
  // of a wave complete in order: the windows above were read before these writes land)
  stage_fence();
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int piece = lane + i * kWave;
    if (piece < PER * NH) *reinterpret_cast<f32x4 *>(rows + (piece / PER) * kUtilRow + 4 * (piece % PER)) = carry[i];
  }
  if (first_block && key4 < kUtilHead) {
#pragma unroll
    for (int hp = 0; hp < NP; ++hp) {
      const int mine = 2 * hp + half;
      if (mine < NH)
        *reinterpret_cast<f32x4 *>(edge + mine * kUtilHead + key4) =
            *reinterpret_cast<const f32x4 *>(rows + mine * kUtilRow + kUtilCarry + key4);
    }
  }
  float best[4];
  pooled_best<NH>(a, win, lane, heads_left, wgt, best);
  // (x, y) -> ([x.lo, y.lo], [x.hi, y.hi]): lanes 0..31 get both halves' values of keys 0 and 1 of their
  // group, lanes 32..63 those of keys 2 and 3
  const auto s02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[0]), __float_as_uint(best[2]), false, false);
  const auto s13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[1]), __float_as_uint(best[3]), false, false);
  const f32x2 out = {fmaxf(__uint_as_float(s02[0]), __uint_as_float(s02[1])),
                     fmaxf(__uint_as_float(s13[0]), __uint_as_float(s13[1]))};
  // groups 0..7 lie in front of the block; in the range's first block they and group 8 (the range's
  // first four keys, whose windows reach in front of the range) are left to finish_utility
  const bool emit = grp >= kUtilShift / 4 + 1 || !first_block;
  const uint32_t off_u =
      emit ? (uint32_t)((bc.g * a.P + t_first - kUtilShift + 4 * grp + 2 * half) * 4) : 0x80000000u;
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, out), rsrc_u, off_u, 0, kOutStoreAux);
}

// The first and last keys around a workgroup's range, four on either side, for the pooling windows that reach over its ends:
// eight rows in a small LDS image, loaded first of all and contracted while the first key tiles are on their way
// (each wave takes the heads w and w + 4). The neighbours' ranges inside the workgroup go through its stages.
constexpr int kHaloKeys = 4;
static_assert(kHaloKeys >= kUtilMaxRadius && 2 * kHaloKeys == kUtilHead, "one row of eight sums");
template <class G>
__device__ __forceinline__ void dma_halo(const char *kbase, int64_t ks_t, int begin, int end, int T, int lane, uint32_t lds) {
#pragma unroll
  for (int i = 0; i < 2 * kHaloKeys * G::ROW / 1024; ++i) {
    int r, kappa;
    dma_source<G>(i, lane, r, kappa);
    const int t = r < kHaloKeys ? max(begin - kHaloKeys + r, 0) : min(end + r - kHaloKeys, T - 1);
    dma_one(lds + i * 1024, kbase + (int64_t)min(t, T - 1) * ks_t + kappa * 16);
  }
}

// The utilities a wave's rounds leave out: groups of four keys as in flush_utility, the first at the front of the range
// (where there were rounds), the others from the last kUtilShift keys of the rounds to the end of the range or of the prefix.
// A group's twelve sums come from the wave's stage, and over the ends of its range from the wave in front (`prev`, four sums
// per head), its own first ones (`edge`) and the wave behind (`next`). A separate kernel for them, from sums in global memory,
// took 5 to 7 us of every call (4096 keys, 32/32 heads 33.6 us with it; 16384 keys with given normalisers 51.8).
template <int NQ, int WT>
__device__ __forceinline__ void finish_utility(const ScoreArgs &a, const BlockCoord &bc, const WaveRange &wr, int n_piped,
                                               const float *rows, const float *edge, const float *prev, int prev_stride,
                                               const float *next, int next_stride, int lane,
                                               __amdgpu_buffer_rsrc_t rsrc_u, const float (&wgt)[NQ / WT]) {
  constexpr int NH = NQ / WT;
  constexpr int NP = (NH + 1) / 2;
  typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
  const int heads_left = a.G - (bc.grp * NQ) / WT;
  const int half = lane >> 5;
  const int limit = min(wr.t_end, a.P), tail0 = wr.t_begin + n_piped * kTile;
  const int n_front = n_piped > 0 ? 1 : 0, first = tail0 - (n_piped > 0 ? kUtilShift : 0);
  const int n = n_front + (limit - first + 3) / 4;
  const uint32_t pad = a.pool == CKV_POOL_MAX ? 0xff800000u : 0u;
  for (int g0 = 0; g0 < n; g0 += kWave / 2) {
    const int grp = g0 + (lane & 31), i = min(grp, n - 1);
    const bool front = i < n_front;
    const int t = front ? wr.t_begin : first + 4 * (i - n_front), rel = t - tail0;
    float win[NP][12];
#pragma unroll
    for (int hp = 0; hp < NP; ++hp) {
      const int head = 2 * hp + half < NH ? 2 * hp + half : 0;
      const float *row = rows + head * kUtilRow + kUtilCarry + (front ? 0 : rel);
      const float *own = edge + head * kUtilHead;
      const float *from[3] = {t == wr.t_begin ? prev + head * prev_stride : row - 4, front ? own : row,
                              front ? own + 4 : t + 4 >= limit ? next + head * next_stride : row + 4};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const u32x4_t v = *reinterpret_cast<const u32x4_t *>(from[q]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t x = v[e];  // what lies outside the prefix may be anything: masked as bits
          win[hp][4 * q + e] = __uint_as_float((uint32_t)(t - 4 + 4 * q + e) < (uint32_t)a.P ? x : pad);
        }
      }
    }
    float best[4];
    pooled_best<NH>(a, win, lane, heads_left, wgt, best);
    const auto s02 = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[0]), __float_as_uint(best[2]), false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap(__float_as_uint(best[1]), __float_as_uint(best[3]), false, false);
    const float out[2] = {fmaxf(__uint_as_float(s02[0]), __uint_as_float(s02[1])),
                          fmaxf(__uint_as_float(s13[0]), __uint_as_float(s13[1]))};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int at = t + 2 * half + e;
      const uint32_t off = grp < n && at < limit ? (uint32_t)((bc.g * a.P + at) * 4) : 0x80000000u;
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(out[e]), rsrc_u, off, 0, kOutStoreAux);
    }
  }
}

// Beyond six query tiles a wave has its SIMD to itself, whatever LDS would allow: the scheduler is told so, or it saves registers where rows
// are short enough for two workgroups of LDS per CU, misses the half of them that a second wave would need, and puts the
// exponentials one behind the other (us, 64 dimensions, windows of 100: 70827 keys, batch 8, 32/4 heads 557 -> 483, 4/2 heads 62.9 -> 54.4;
// 28/4 heads, windows of 32: 40000 keys, batch 4 34.3 -> 31.8). In pass 1, where seven and eight tiles do leave room for a second wave,
// it gains 5 % in launches of one workgroup per CU and loses 6 % in larger ones.
template <int DT, int DH, int NQ, int WT, bool UTIL = false, bool GSUM = false>
__global__ void __launch_bounds__(kScoreWaves *kWave) __attribute__((amdgpu_waves_per_eu(1, NQ > 6 ? 1 : 8))) colsum_lds_kernel(ScoreArgs a) {
  static_assert(!(UTIL && GSUM) && (!GSUM || WT == 1), "one epilogue at a time; group sums take one tile per head");
  static_assert(NQ % WT == 0, "whole heads");
  using G = Geom<DT, DH>;
  constexpr int NCH = G::NCH;
  constexpr bool STREAM = true;
  static_assert(DT == CKV_BF16, "row biases");
  constexpr int N_MFMA = NCH + 1;
  constexpr int READ_AT = NQ >= 2 ? NQ - 2 : 0;
  __shared__ __attribute__((aligned(1024))) typename Staged<DT, DH, NQ, STREAM>::Ring ring;
  const int lane = threadIdx.x & 63, m = lane & 31, hh = lane >> 5;
  const BlockCoord bc = decode_block(a);
  const WaveRange wr = wave_range(a, bc, UTIL ? a.P : a.T);  // utilities: of the prefix only

  constexpr int NH = NQ / WT;
  __shared__ __attribute__((aligned(1024))) char s_halo_keys[UTIL ? 2 * kHaloKeys * G::ROW : 16];
  __shared__ __attribute__((aligned(16))) float s_halo[UTIL ? NH * kUtilHead : 4];
  __shared__ __attribute__((aligned(16))) float s_edge[UTIL ? kScoreWaves : 1][UTIL ? NH * kUtilHead : 4];
  __shared__ __attribute__((aligned(1024))) float s_stage[kScoreWaves][NH * (UTIL ? kUtilRow : kRing * kTile)];
  RatioScale rs;
  rs.load(a, bc);
  Staged<DT, DH, NQ, STREAM> st;
  chunk_t qf[NQ][NCH];
  int jrow[NQ];
  // The biases that the normalisers make, a thread per row (NQ * 32 <= 256 of them): given, or, both passes in one call, merged from the first
  // pass's row partials by every workgroup of a unit. (A kernel in between cost 5 us, 11 with eight tiles and 32
  // workgroups along the keys; a lane merging all its rows by itself cost more than that from 16 partials on.) What they are made
  // of comes into the stage, which is not used yet, in front of everything else: a load into registers would have to be waited
  // for behind the first key tiles, since the compiler does not know of those. More partials than the stage holds are loaded that way.
  // With that, and the sums around the range contracted while the query tiles are in their images, 16384 keys with given normalisers
  // 45.5 -> 44.9 us per layer, 32/8 heads of 131072 177.8 -> 175.9.
  constexpr int ROWS = NQ * kTile;
  constexpr int STAGED_CHUNKS = (int)sizeof(s_stage) / 1024 * 1024 / (ROWS * (int)sizeof(float2));  // whole loads of 1 KiB
  static_assert(ROWS <= kScoreWaves * kWave && sizeof(s_stage) >= kScoreWaves * kWave * sizeof(float), "a thread per row");
  __shared__ uint2 s_bias[ROWS];
  const float2 *part = a.part + ((size_t)bc.unit * a.n_groups + bc.grp) * a.n_chunks * ROWS;
  // The sums around the workgroup's range (fused form): wave w takes the heads w and w + 4, the tiles of a head one after the other
  constexpr int HALO_TILES = UTIL ? WT * ((NH + kScoreWaves - 1) / kScoreWaves) : 1;
  const auto halo_head = [&](int u) { return wr.wave + u / WT * kScoreWaves; };
  f32x16 halo[HALO_TILES];
  st.start(
      a, bc, wr, ring, lane, m, hh, qf, jrow,
      [&] {
        const uint32_t stage_lds = (uint32_t)(uintptr_t)&s_stage[0][0];
        if (a.lse_from_part) {
          const int bytes = a.n_chunks * ROWS * (int)sizeof(float2);
          if (a.n_chunks <= STAGED_CHUNKS)
            for (int at = wr.wave * 1024; at < bytes; at += kScoreWaves * 1024)
              dma_one(stage_lds + at, reinterpret_cast<const char *>(part) + min(at + lane * 16, bytes - 16));
        } else if (wr.wave * kWave < ROWS) {
          const int row = wr.wave * kWave + lane, tile = min(bc.grp * NQ + row / kTile, a.n_tiles - 1);
          const int j = min(tile % WT * kTile + row % kTile, a.W - 1);
          const float *src = a.lse + ((size_t)bc.b * a.Hq + bc.g * a.G + tile / WT) * a.W + j;
          asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(stage_lds + wr.wave * (kWave * 4)), "v"(src) : "memory");
        }
        if constexpr (UTIL) {
          const int begin = bc.chunk * kScoreWaves * a.keys_per_wave;
          if (wr.wave == 0)
            dma_halo<G>(a.k + bc.b * a.ks_b + bc.g * a.ks_h, a.ks_t, begin, begin + kScoreWaves * a.keys_per_wave, a.T, lane,
                        (uint32_t)(uintptr_t)s_halo_keys);
        }
      },
      [&] {
        if constexpr (UTIL) {
          int hoff[NCH];
#pragma unroll
          for (int c = 0; c < NCH; ++c) hoff[c] = image_offset<G>(m & (kUtilHead - 1), c + NCH * hh);
          chunk_t kh[NCH], qh[NCH];
          read_image<G>(kh, s_halo_keys, hoff);
#pragma unroll
          for (int u = 0; u < HALO_TILES; ++u) {
            if (halo_head(u) >= NH) continue;
            const int tile = halo_head(u) * WT + u % WT;
            read_image<G>(qh, Staged<DT, DH, NQ, STREAM>::image_of_tile(ring, tile), st.roff);
            if (bc.grp * NQ + tile >= a.n_tiles || tile % WT * kTile + m >= a.W) {
#pragma unroll
              for (int c = 0; c < NCH; ++c) qh[c] = chunk_t{0u, 0u, 0u, 0u};
            }
            mma_chain<DT, NCH>(halo[u], qh, kh);
          }
        }
        if (threadIdx.x < ROWS) {
          float v;
          if (!a.lse_from_part) v = s_stage[0][threadIdx.x];
          else if (a.n_chunks <= STAGED_CHUNKS)
            v = merge_row_partials(reinterpret_cast<const float2 *>(&s_stage[0][0]) + threadIdx.x, a.n_chunks, ROWS);
          else v = merge_row_partials(part + threadIdx.x, a.n_chunks, ROWS);
          const bool valid = bc.grp * NQ + (int)threadIdx.x / kTile < a.n_tiles && (int)threadIdx.x / kTile % WT * kTile + (int)threadIdx.x % kTile < a.W;
          s_bias[threadIdx.x] = RowBias::pack(valid ? v * (-kLog2e / a.c2) : kNoWeight / a.c2);
        }
      });
  if constexpr (UTIL) {  // tau and the budgets of a batch element: a wave of its first workgroup
    if (bc.g == 0 && bc.chunk == 0 && wr.wave == kScoreWaves - 1) write_tau_and_budgets(a.bud, bc.b, lane);
  }
  rs.store(a, bc);
  RowBias bias[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) bias[i].set(s_bias + i * kTile, m, hh);
  // Descriptor over scores[b]: Hq * T floats (the host checks that this stays below 2 GiB). Lanes with
  // nothing to store present an offset outside it, which the hardware drops: no branch splits the
  // pipeline's code, and every flush issues exactly N_STORES store instructions.
  const int score_rows = GSUM ? a.Hkv : a.Hq;  // rows of a batch element in the output
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(a.scores + (UTIL ? 0 : (size_t)bc.b * score_rows * a.T)), 0, UTIL ? 0 : score_rows * a.T * 4, 0x00020000);
  // Vector memory operations complete in issue order, stores included. When tile t + 1 is picked up,
  // the loads of tiles t + 2 and t + 3 were issued after its own, and so were the stores of the
  // previous ring cycle if t is the cycle's first or second tile; that many operations may still be
  // in flight. The first cycle has no such stores behind it: dropped stores (offset outside the
  // descriptor) issued after the first loads stand in.
  // per flush: one for the fused and for the group-sum form
  constexpr int N_STORES = GSUM || UTIL ? 1 : (NH + 1) / 2;
  // fused form: descriptor over utility[b] (Hkv * P floats) and the weights of this group's heads
  const __amdgpu_buffer_rsrc_t rsrc_u = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(UTIL ? a.utility + (size_t)bc.b * a.Hkv * a.P : a.scores), 0, UTIL ? a.Hkv * a.P * 4 : 0, 0x00020000);
  float wgt[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int head = bc.g * a.G + (bc.grp * NQ) / WT + h;
    wgt[h] = UTIL && head < a.Hq ? a.w_row[head] : 0.0f;
  }
  float *stage = s_stage[wr.wave];
  const int n_piped = wr.n_full / kRing * kRing;
  // (distinct offsets, all outside the descriptor: identical stores could be merged into one)
#pragma unroll
  for (int i = 0; i < N_STORES; ++i) __builtin_amdgcn_raw_buffer_store_b32(0u, UTIL ? rsrc_u : rsrc, 0x80000000u + 64u * i, 0, 0);

  chunk_t kreg[2][NCH];
  f32x16 acc[2];
  if constexpr (UTIL) {
#pragma unroll
    for (int u = 0; u < HALO_TILES; u += WT) {
      if (halo_head(u) >= NH) continue;
      float x = 0.0f;
#pragma unroll
      for (int e = 0; e < WT; ++e) {
        RowBias own;
        own.set(s_bias + (halo_head(u) * WT + e) * kTile, m, hh);
        own.add(halo[u + e], hh);
        const float w = colsum_weights<false>(halo[u + e], a.c2, hh, 0);
        x = e == 0 ? w : x + w;
      }
      const float tot = (x + __shfl_xor(x, 32)) * a.norm;
      if (lane < kUtilHead) s_halo[halo_head(u) * kUtilHead + lane] = tot;
    }
  }
  if (n_piped > 0) {
    wait_vm<(kRing - 2) * G::NDMA>();
    read_image<G>(kreg[0], ring[wr.wave][0], st.roff);
    mma_chain<DT, NCH>(acc[0], qf[0], kreg[0]);
    bias[0].add(acc[0], hh);
  }
  constexpr int UR = unroll_tiles(NQ);
  for (int t0 = 0; t0 < n_piped; t0 += UR) {
    const int slot0 = UR == kRing ? 0 : (t0 & (kRing - 1));  // ring image of tile t0
#pragma unroll
    for (int v = 0; v < UR; ++v) {
      const int u = slot0 + v;
      st.prefetch(t0 + v, wr.n_whole, (u + kRing - 1) % kRing);
      float cs[NQ];
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        const int cur = (v * NQ + i) & 1;
        if (i == READ_AT) {
          // tile t0 + v + 1 has landed. In the first half of a ring cycle the previous cycle's stores were
          // issued after its load and may still be in flight; where the half is only known at run time the
          // wait does not allow for them (stricter, never wrong).
          if (UR == kRing && v < 2) wait_vm<(kRing - 2) * G::NDMA + N_STORES>();
          else wait_vm<(kRing - 2) * G::NDMA>();
          read_image<G>(kreg[(v + 1) & 1], ring[wr.wave][(u + 1) % kRing], st.roff);
        }
        if (i + 1 < NQ) {
          mma_chain<DT, NCH>(acc[cur ^ 1], qf[i + 1], kreg[v & 1]);  // rows: query rows, cols: keys
          bias[i + 1].add(acc[cur ^ 1], hh);
        } else {
          mma_chain<DT, NCH>(acc[cur ^ 1], qf[0], kreg[(v + 1) & 1]);
          bias[0].add(acc[cur ^ 1], hh);
        }
        cs[i] = colsum_weights<false>(acc[cur], a.c2, hh, 0);
        if (i == READ_AT) interleave_hint<N_MFMA, vector_per_mfma_pass2(NQ), NCH>();
        else interleave_hint<N_MFMA, vector_per_mfma_pass2(NQ), 0>();
      }
      if constexpr (UTIL) stage_column_sums<NQ, WT, kUtilRow>(cs, a.norm, stage + kUtilCarry, u * kTile + m, hh);
      else stage_column_sums<NQ, WT>(cs, a.norm, stage, u * kTile + m, hh);
      st.kcur += st.tile_stride;
    }
    if (UR == kRing || slot0 + UR == kRing) {  // a ring cycle is complete
      const int c0 = t0 + UR - kRing;          // its first tile
      stage_fence();  // the tiles' sums are staged
      if constexpr (UTIL)
        flush_utility<NQ, WT>(a, bc, stage, s_edge[wr.wave], wr.t_begin + c0 * kTile, c0 == 0, lane, rsrc_u, wgt);
      else if constexpr (GSUM) flush_group_sums<NQ>(a, bc, stage, wr.t_begin + c0 * kTile, lane, rsrc);
      else flush_column_sums<NQ, WT>(a, bc, stage, wr.t_begin + c0 * kTile, lane, rsrc);
      stage_fence();  // and read, before the next cycle's overwrite them
    }
  }
  for (int t = n_piped; t < wr.n_all; ++t) {
    const int kt = wr.t_begin + t * kTile + m;  // this lane's key
    st.tail_tile(wr, ring, t, wr.t_begin + t * kTile - (a.T - kTile), m, hh, kreg[0]);
    float cs[NQ];
    mma_chain<DT, NCH>(acc[0], qf[0], kreg[0]);
    bias[0].add(acc[0], hh);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int j0 = ((bc.grp * NQ + i) % WT) * kTile;
      if (i + 1 < NQ) {
        mma_chain<DT, NCH>(acc[(i + 1) & 1], qf[i + 1], kreg[0]);
        bias[i + 1].add(acc[(i + 1) & 1], hh);
      }
      cs[i] = colsum_weights<!UTIL>(acc[i & 1], a.c2, hh, kt - a.P - j0);  // keys of the prefix: every row sees them
      if (i + 1 < NQ) interleave_hint<N_MFMA, kTailVectorPerMfma, 0>();
    }
    if constexpr (UTIL)
      stage_column_sums<NQ, WT, kUtilRow>(cs, a.norm, stage + kUtilCarry, (t - n_piped) * kTile + m, hh);
    else if constexpr (GSUM) store_group_sum<NQ>(a, bc, cs, kt, hh);
    else store_column_sums<NQ>(a, bc, cs, WT, kt, hh);
  }
  if constexpr (UTIL) {
    __syncthreads();
    if (wr.n_all > 0) {
      // the wave in front has a whole range of the prefix; the one behind left its first sums at s_edge if it had rounds
      const int w = wr.wave, round = kRing * kTile, behind = min(wr.t_end + a.keys_per_wave, a.P) - wr.t_end;
      const float *prev = w > 0 ? s_stage[w - 1] + kUtilCarry + a.keys_per_wave % round - kHaloKeys : s_halo;
      const float *next = w == kScoreWaves - 1 ? s_halo + kHaloKeys : behind >= round ? s_edge[w + 1] : s_stage[w + 1] + kUtilCarry;
      finish_utility<NQ, WT>(a, bc, wr, n_piped, stage, s_edge[w], prev, w > 0 ? kUtilRow : kUtilHead, next,
                             w == kScoreWaves - 1 || behind >= round ? kUtilHead : kUtilRow, lane, rsrc_u, wgt);
    }
    if (a.ratio) {
      // times the ratio, which this thread has scaled at the start; the utilities are other waves' stores: read past the L1
      wait_vm<0>();
      __syncthreads();
      const int begin = bc.chunk * kScoreWaves * a.keys_per_wave, end = min(begin + kScoreWaves * a.keys_per_wave, a.P);
      const float *ratio = a.ratio + (size_t)bc.unit * a.T;
      typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
      constexpr int STEP = kScoreWaves * kWave * 4, BATCH = 4;  // groups of four keys, BATCH of them in flight
      for (int t0 = begin + threadIdx.x * 4; t0 < end; t0 += BATCH * STEP) {
        u32x4_t u[BATCH];
        f32x4_r r[BATCH];
#pragma unroll
        for (int e = 0; e < BATCH; ++e) {
          const int t = t0 + e * STEP;
          u[e] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_u, t < end ? (uint32_t)((bc.g * a.P + t) * 4) : 0x80000000u, 0, kOutStoreAux);
          r[e] = *reinterpret_cast<const f32x4_r *>(ratio + min(t, a.T - 4));
        }
#pragma unroll
        for (int e = 0; e < BATCH; ++e) {
          const int t = t0 + e * STEP;
          if (t + 4 <= end && t + 4 <= a.T) {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const uint32_t bits = u[e][x];
              u[e][x] = __float_as_uint(__uint_as_float(bits) * r[e][x]);
            }
            __builtin_amdgcn_raw_buffer_store_b128(u[e], rsrc_u, (uint32_t)((bc.g * a.P + t) * 4), 0, kOutStoreAux);
          } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) {
              const uint32_t bits = u[e][x];
              if (t + x < end) a.utility[(size_t)bc.unit * a.P + t + x] = __uint_as_float(bits) * ratio[t + x];
            }
          }
        }
      }
    }
  }
  wait_vm<0>();  // the loads beyond the last tile write LDS: not after the wave
}

// The mark of a range whose sums another workgroup has made, unless the range's own one has left its mark, or changed it already.
__device__ __forceinline__ void leave_mark(tag_t *mark, tag_t tag) {
  const tag_t seen = load_across(mark);
  if ((seen | 1) != (tag | 1)) replace_across(mark, seen, tag);
}

// ---------------------------------------------------------------------------------------------
// Both passes of a fused call in one launch, for ranges that fit the ring: the key tiles stay in LDS between the passes. What a short
// call takes is launches, the way of the first loads and the fetch of code, not bytes or arithmetic; here the second pass has
// neither a launch nor loads of its own, and as a range is four tiles at most, nothing is unrolled over them.
//
// The workgroups of a unit exchange their row sums: each leaves its own and a mark (behind them, when they have arrived), waits until
// it sees all marks, and merges all sums. No workgroup depends on another one's progress: after a.wait it makes the sums of one of the missing
// ranges, from the keys in memory, the same ones to the last bit, leaves that range's mark and looks again (a launch whose workgroups do not all
// find a CU, because another stream's kernel holds some, would wait for workgroups that wait for it otherwise). Each begins at
// another of the missing ranges, so that they share them: with all of them made by every waiting workgroup, four streams of 65536 keys,
// batch 2, 8/1 heads (128 ranges a unit) took 646 us per call, now 51, two launches 33; beside matrix products 220 us more than two launches, now none
// (the same beside a scan that holds 136 CUs, us: 239, 151, 142; 8192 keys, batch 2, 32/4 heads 78, 78, 102).
// Who has read all sums changes its mark; who sees all of them changed at its end takes them back, and the last one to change its
// own does see that.
// us per layer on a stream of layers, two launches / one, keys in the memory-side cache before the call and from HBM: 4096 keys, 32/32 heads
// 26.3 / 24.1, 30.4 / 24.7; 8192, 32/8 27.6 / 25.1, 28.9 / 25.0; 4096, batch 4, 32/8 36.0 / 30.7, 38.2 / 31.4; 1000, 32/8 20.2 / 18.9, 20.5 / 19.9; seven
// tiles, 6000, batch 2, 28/4 30.2 / 28.8, 32.1 / 29.0; eight, 8192, batch 2, 32/4 33.4 / 30.9, 35.6 / 31.0; 3001, W = 64, 32/8 28.8 / 28.2, 30.7 / 28.7;
// 65536, batch 2, 8/1 60.7 / 57.2, 63.9 / 57.2. One layer that is waited for, keys from HBM (launch and host included): 45.1 / 39.8 for the first, 42.9 / 39.5
// for the second. The keys are streamed, since nothing reads them again (kept in the cache 1 to 5 % faster if they were there
// before, 2 to 7 % slower if not).
// ---------------------------------------------------------------------------------------------
template <int DT, int DH, int NQ, int WT, bool UTIL>
__global__ void __launch_bounds__(kScoreWaves *kWave) scan_short_kernel(ScoreArgs a) {
  static_assert(DT == CKV_BF16 && NQ % WT == 0, "whole heads");
  static_assert(kRing == 4, "the waits below");
  using G = Geom<DT, DH>;
  constexpr int NCH = G::NCH, NH = NQ / WT, ROWS = NQ * kTile;
  // Eight query tiles of 256-byte rows fill the registers: the sums around the range are contracted behind the exchange, not held through
  // it (eight registers spilled, and each reload waited for all key tiles in flight: us per layer 8192 keys, batch 2, 32/4 heads 31.7
  // with spills / 31.0, 3001 keys, W = 64 29.3 / 28.4, 65536 keys, batch 2, 8/1 56.5 / 55.4).
  constexpr bool FULL = NQ == kMaxQTiles && G::ROW == 256 && UTIL;
  typedef Staged<DT, DH, NQ, true> Scan;
  __shared__ __attribute__((aligned(1024))) typename Scan::Ring ring;
  __shared__ __attribute__((aligned(1024))) char s_halo_keys[UTIL ? 2 * kHaloKeys * G::ROW : 16];
  __shared__ __attribute__((aligned(16))) float s_halo[UTIL ? NH * kUtilHead : 4];
  __shared__ __attribute__((aligned(16))) float s_stage[kScoreWaves][UTIL ? NH * kUtilRow : 2 * ROWS];  // first: the waves' row sums
  __shared__ uint2 s_bias[ROWS];
  __shared__ uint64_t s_missing[kComputeUnits / kWave];
  static_assert(sizeof(s_stage) >= kScoreWaves * ROWS * sizeof(float2), "row sums pass through the stage");
  const int lane = threadIdx.x & 63, m = lane & 31, hh = lane >> 5;
  const BlockCoord bc = decode_block(a);
  const WaveRange wr = wave_range(a, bc, a.T);
  const int n_sums = wave_range(a, bc, UTIL ? a.P : a.T).n_all;  // tiles whose column sums are wanted

  Scan st;
  chunk_t qf[NQ][NCH];
  int jrow[NQ];
  constexpr int HALO_TILES = !UTIL ? 1 : WT * ((NH + kScoreWaves - 1) / kScoreWaves);  // as in colsum_lds_kernel
  const auto halo_head = [&](int u) { return wr.wave + u / WT * kScoreWaves; };
  f32x16 halo[HALO_TILES];
  const auto read_halo = [&](chunk_t(&kh)[NCH]) {
    int hoff[NCH];
#pragma unroll
    for (int c = 0; c < NCH; ++c) hoff[c] = image_offset<G>(m & (kUtilHead - 1), c + NCH * hh);
    read_image<G>(kh, s_halo_keys, hoff);
  };
  st.start(
      a, bc, wr, ring, lane, m, hh, qf, jrow,
      [&] {
        if constexpr (!UTIL) return;
        const int begin = bc.chunk * kScoreWaves * a.keys_per_wave;
        if (wr.wave == 0)
          dma_halo<G>(a.k + bc.b * a.ks_b + bc.g * a.ks_h, a.ks_t, begin, begin + kScoreWaves * a.keys_per_wave, a.T, lane,
                      (uint32_t)(uintptr_t)s_halo_keys);
      },
      [&] {
        if constexpr (!UTIL || FULL) return;
        chunk_t kh[NCH], qh[NCH];
        read_halo(kh);
#pragma unroll
        for (int u = 0; u < HALO_TILES; ++u) {
          if (halo_head(u) >= NH) continue;
          const int tile = halo_head(u) * WT + u % WT;
          read_image<G>(qh, Scan::image_of_tile(ring, tile), st.roff);
          if (bc.grp * NQ + tile >= a.n_tiles || tile % WT * kTile + m >= a.W) {
#pragma unroll
            for (int c = 0; c < NCH; ++c) qh[c] = chunk_t{0u, 0u, 0u, 0u};
          }
          mma_chain<DT, NCH>(halo[u], qh, kh);
        }
      });

  // -- pass 1: the rows' (max, sum) over a range, left for the unit's workgroups
  float2 *const parts = a.part + (size_t)bc.unit * a.n_chunks * ROWS;
  chunk_t kf[NCH];
  f32x16 acc[2];
  const auto row_sums = [&](const WaveRange &range, int chunk, auto read_tile) {
    float rm[NQ], rl[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      rm[i] = -1e30f;
      rl[i] = 0.0f;
    }
    for (int t = 0; t < range.n_all; ++t) {
      const int t0 = range.t_begin + t * kTile;
      read_tile(t, t0);
      mma_chain<DT, NCH>(acc[0], kf, qf[0]);
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        if (i + 1 < NQ) mma_chain<DT, NCH>(acc[(i + 1) & 1], kf, qf[i + 1]);
        if (t >= range.n_full) {  // uniform: the window's rows see no later keys, and there are none beyond T
          const int tile = bc.grp * NQ + i, j = tile % WT * kTile + m;
          const int limit = tile < a.n_tiles && j < a.W ? a.P + j : -1;
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i & 1][r] = acc_row(r, hh) > limit - t0 ? -INFINITY : acc[i & 1][r];
        }
        rowstats_update<false>(acc[i & 1], a.c2, 0, hh, 0, rm[i], rl[i]);
      }
    }
    float2 *sums = reinterpret_cast<float2 *>(&s_stage[0][0]);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const float om = __shfl_xor(rm[i], 32), ol = __shfl_xor(rl[i], 32);
      merge_stats(rm[i], rl[i], om, ol);
      if (hh == 0) sums[range.wave * ROWS + i * kTile + m] = make_float2(rm[i], rl[i]);
    }
    __syncthreads();
    if (threadIdx.x < ROWS) {
      float2 s = sums[threadIdx.x];
#pragma unroll
      for (int w = 1; w < kScoreWaves; ++w) merge_stats(s.x, s.y, sums[w * ROWS + threadIdx.x].x, sums[w * ROWS + threadIdx.x].y);
      store_across(reinterpret_cast<uint64_t *>(parts + chunk * ROWS + threadIdx.x), __builtin_bit_cast(uint64_t, s));
    }
    wait_vm<0>();  // what was left has arrived
    __syncthreads();
  };
  if (wr.n_all == kRing) st.prefetch(0, wr.n_whole, kRing - 1);
  const int asked = Scan::tiles_asked(a) + (wr.n_all == kRing ? 1 : 0);
  row_sums(wr, bc.chunk, [&](int t, int t0) {
    switch (asked - 1 - t) {  // tiles asked for behind this one
      case 3: wait_vm<3 * G::NDMA>(); break;
      case 2: wait_vm<2 * G::NDMA>(); break;
      case 1: wait_vm<G::NDMA>(); break;
      default: wait_vm<0>();
    }
    st.read_tail(wr, ring, t, t0 - (a.T - kTile), m, hh, kf);
  });
  tag_t *const marks = a.marks + (size_t)bc.unit * a.n_chunks;
  if (threadIdx.x == 0) store_across(marks + bc.chunk, a.tag);
  if (UTIL && bc.g == 0 && bc.chunk == 0 && wr.wave == kScoreWaves - 1) write_tau_and_budgets(a.bud, bc.b, lane);

  // -- the others' sums: all of them within a.wait, or one of the missing ranges by this workgroup, and the marks again
  for (;;) {
    if (wr.wave == 0) {
      const uint64_t start = __builtin_amdgcn_s_memrealtime();
      for (;;) {
        const uint64_t now = __builtin_amdgcn_s_memrealtime();
        bool some = false;
        for (int c0 = 0; c0 < a.n_chunks; c0 += kWave) {
          const int c = c0 + lane;
          const uint64_t missing = __ballot(c < a.n_chunks && (load_across(marks + c) | 1) != (a.tag | 1));
          if (lane == 0) s_missing[c0 / kWave] = missing;
          some |= missing != 0;
        }
        if (!some || now - start >= a.wait) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __syncthreads();
    const auto missing = [&](int c0) {
      const uint64_t x = s_missing[c0 / kWave];
      return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(x >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)x);
    };
    int n_missing = 0, rank = bc.chunk;  // rank: of this workgroup among those whose sums are there
    for (int c0 = 0; c0 < a.n_chunks; c0 += kWave) {
      const uint64_t x = missing(c0);
      const int in_front = bc.chunk - c0;
      n_missing += __popcll(x);
      rank -= in_front >= kWave ? __popcll(x) : in_front > 0 ? __popcll(x & ((1ull << in_front) - 1)) : 0;
    }
    if (n_missing == 0) break;
    int skip = rank % n_missing;
    BlockCoord other = bc;
    for (int c0 = 0; c0 < a.n_chunks; c0 += kWave) {
      uint64_t x = missing(c0);
      const int here = __popcll(x);
      if (skip >= here) {
        skip -= here;
        continue;
      }
      for (; skip > 0; --skip) x &= x - 1;
      other.chunk = c0 + __ffsll((long long)x) - 1;
      break;
    }
    row_sums(wave_range(a, other, a.T), other.chunk, [&](int, int t0) {
      const char *row = st.kbase + (int64_t)min(t0 + m, a.T - 1) * a.ks_t;
#pragma unroll
      for (int c = 0; c < NCH; ++c) kf[c] = *reinterpret_cast<const chunk_t *>(row + (c + NCH * hh) * 16);
    });
    if (threadIdx.x == 0) leave_mark(marks + other.chunk, a.tag);
    wait_vm<0>();
  }
  if (threadIdx.x < ROWS) {
    const int tile = bc.grp * NQ + (int)threadIdx.x / kTile;
    const bool valid = tile < a.n_tiles && tile % WT * kTile + (int)threadIdx.x % kTile < a.W;
    const float lse = merge_partials_across(parts + threadIdx.x, a.n_chunks, ROWS);
    s_bias[threadIdx.x] = RowBias::pack(valid ? lse * (-kLog2e / a.c2) : kNoWeight / a.c2);
  }
  __syncthreads();
  if (threadIdx.x == 0) store_across(marks + bc.chunk, a.tag | 1);

  // -- pass 2
  RowBias bias[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) bias[i].set(s_bias + i * kTile, m, hh);
  if constexpr (FULL) {
    chunk_t kh[NCH];
    read_halo(kh);
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (wr.wave == i / WT % kScoreWaves) mma_chain<DT, NCH>(halo[i / (WT * kScoreWaves) * WT + i % WT], qf[i], kh);
  }
  if constexpr (UTIL) {
#pragma unroll
    for (int u = 0; u < HALO_TILES; u += WT) {
      if (halo_head(u) >= NH) continue;
      float x = 0.0f;
#pragma unroll
      for (int e = 0; e < WT; ++e) {
        RowBias own;
        own.set(s_bias + (halo_head(u) * WT + e) * kTile, m, hh);
        own.add(halo[u + e], hh);
        const float w = colsum_weights<false>(halo[u + e], a.c2, hh, 0);
        x = e == 0 ? w : x + w;
      }
      const float tot = (x + __shfl_xor(x, 32)) * a.norm;
      if (lane < kUtilHead) s_halo[halo_head(u) * kUtilHead + lane] = tot;
    }
  }
  const __amdgpu_buffer_rsrc_t rsrc_u = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(UTIL ? a.utility + (size_t)bc.b * a.Hkv * a.P : a.scores), 0, UTIL ? a.Hkv * a.P * 4 : 0, 0x00020000);
  float wgt[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int head = bc.g * a.G + (bc.grp * NQ) / WT + h;
    wgt[h] = UTIL && head < a.Hq ? a.w_row[head] : 0.0f;
  }
  float *stage = s_stage[wr.wave];
  for (int t = 0; t < n_sums; ++t) {
    const int kt = wr.t_begin + t * kTile + m;  // this lane's key
    st.read_tail(wr, ring, t, kt - m - (a.T - kTile), m, hh, kf);
    float cs[NQ];
    mma_chain<DT, NCH>(acc[0], qf[0], kf);
    bias[0].add(acc[0], hh);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      if (i + 1 < NQ) {
        mma_chain<DT, NCH>(acc[(i + 1) & 1], qf[i + 1], kf);
        bias[i + 1].add(acc[(i + 1) & 1], hh);
      }
      // utilities: keys of the prefix, which every row sees
      cs[i] = colsum_weights<!UTIL>(acc[i & 1], a.c2, hh, kt - a.P - i % WT * kTile);
    }
    if constexpr (UTIL) stage_column_sums<NQ, WT, kUtilRow>(cs, a.norm, stage + kUtilCarry, t * kTile + m, hh);
    else store_column_sums<NQ>(a, bc, cs, WT, kt, hh);
  }
  if constexpr (UTIL) __syncthreads();
  // All marks, asked for when the workgroup's own one has arrived as it stays.
  constexpr int MARKS = kComputeUnits / kWave;
  bool all = true;
  if (wr.wave == 0) {
    wait_vm<0>();
#pragma unroll
    for (int e = 0; e < MARKS; ++e)
      if (e * kWave + lane < a.n_chunks) all &= load_across(marks + e * kWave + lane) == (a.tag | 1);
  }
  if (UTIL && n_sums > 0) {
    const int w = wr.wave;
    const float *prev = w > 0 ? s_stage[w - 1] + kUtilCarry + a.keys_per_wave - kHaloKeys : s_halo;
    const float *next = w == kScoreWaves - 1 ? s_halo + kHaloKeys : s_stage[w + 1] + kUtilCarry;
    finish_utility<NQ, WT>(a, bc, wr, 0, stage, s_halo, prev, w > 0 ? kUtilRow : kUtilHead, next,
                           w == kScoreWaves - 1 ? kUtilHead : kUtilRow, lane, rsrc_u, wgt);
  }
  if (wr.wave == 0 && __ballot(!all) == 0)
    for (int c = lane; c < a.n_chunks; c += kWave) store_across(marks + c, (tag_t)0);
  wait_vm<0>();
}

// ---------------------------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------------------------
// Bytes of K up to which the first pass of a call leaves the keys in the memory-side cache (256 MiB) for the second. us per
// layer, streamed / kept, keys in the cache before the call (as a prefill that has just written them leaves them, or a call on the
// same ones) and then keys from HBM: 4096 keys, 32/32 heads 30.5 / 27.5, 31.1 / 31.4; 16384, 32/8 37.2 / 34.5, 37.5 / 36.2; 1024, 32/32 19.3 / 18.7, 21.7
// / 20.7; 8192, 32/8 28.5 / 27.4, 29.3 / 29.7. At 57 and 61 MB (28000, 32/8; 7500, batch 4) 44.3 / 44.7, 45.1 / 44.9 and no gain from HBM,
// at 82 MB 55.4 / 56.0 from HBM, at 1 GiB 392 / 408. In the second pass, whose keys nobody reads again, the streaming form loses
// nothing (16384, 32/8: 34.9 against 34.1 from the cache, but 20011, batch 2 57.1 against 58.8 from HBM).
constexpr int64_t kKeptKeyBytes = 48 << 20;
template <int DT, int DH, int NQ>
static void launch_rowstats(const Shape &s, const ScoreArgs &a, dim3 grid, dim3 block, hipStream_t stream) {
  if constexpr (DT == CKV_BF16) {
    if (a.v) {
      if constexpr (NQ <= kMaxQTilesNorms)
        hipLaunchKernelGGL((rowstats_lds_kernel<DT, DH, NQ, true>), grid, dim3(2 * block.x), 0, stream, a);
    } else if (a.lse_from_part && (int64_t)s.Bz * s.Hkv * s.T * s.d * s.esize <= kKeptKeyBytes) {
      hipLaunchKernelGGL((rowstats_lds_kernel<DT, DH, NQ, false, true>), grid, block, 0, stream, a);
    } else {
      hipLaunchKernelGGL((rowstats_lds_kernel<DT, DH, NQ>), grid, block, 0, stream, a);
    }
  } else
    hipLaunchKernelGGL((rowstats_kernel<DT, DH, NQ>), grid, block, 0, stream, a);
  if (a.lse_from_part) return;  // the second pass of the same call merges the partials itself
  const int rows = s.Bz * s.Hkv * s.n_groups * NQ * kTile;
  hipLaunchKernelGGL(lse_kernel<NQ>, dim3((rows + 255) / 256), dim3(256), 0, stream, a, rows);
}

template <int DT, int DH, int NQ>
static void launch_colsum(const Shape &s, const ScoreArgs &a, dim3 grid, dim3 block, hipStream_t stream) {
  if constexpr (DT == CKV_BF16) {
    // NQ is a multiple of WT (whole heads per wave)
    if (s.WT == 1) {
      if (a.utility) hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 1, true>), grid, block, 0, stream, a);
      else if (a.group_sum) {
        if constexpr (NQ <= 4) hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 1, false, true>), grid, block, 0, stream, a);
      } else hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 1>), grid, block, 0, stream, a);
      return;
    }
    if constexpr (NQ % 2 == 0) {
      if (s.WT == 2) {
        if (a.utility) hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 2, true>), grid, block, 0, stream, a);
        else hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 2>), grid, block, 0, stream, a);
        return;
      }
    }
    if constexpr (NQ % 3 == 0) {
      if (s.WT == 3) {
        hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 3>), grid, block, 0, stream, a);
        return;
      }
    }
    if constexpr (NQ % 4 == 0) {
      if (s.WT == 4) {
        hipLaunchKernelGGL((colsum_lds_kernel<DT, DH, NQ, 4>), grid, block, 0, stream, a);
        return;
      }
    }
  } else if (a.ratio) {
    hipLaunchKernelGGL((colsum_kernel<DT, DH, NQ, true>), grid, block, 0, stream, a);
  } else {
    hipLaunchKernelGGL((colsum_kernel<DT, DH, NQ, false>), grid, block, 0, stream, a);
  }
}

template <int DT, int DH, int NQ, int WT>
static void launch_short_wt(const ScoreArgs &a, dim3 grid, dim3 block, hipStream_t stream) {
  if constexpr (NQ % WT == 0) {
    if constexpr (WT <= 2) {
      if (a.utility) {
        hipLaunchKernelGGL((scan_short_kernel<DT, DH, NQ, WT, true>), grid, block, 0, stream, a);
        return;
      }
    }
    hipLaunchKernelGGL((scan_short_kernel<DT, DH, NQ, WT, false>), grid, block, 0, stream, a);
  }
}
template <int DT, int DH, int NQ>
static void launch_short(const Shape &s, const ScoreArgs &a, dim3 grid, dim3 block, hipStream_t stream) {
  if constexpr (DT == CKV_BF16) {
    switch (s.WT) {  // NQ is a multiple of WT (whole heads per wave)
      case 1: launch_short_wt<DT, DH, NQ, 1>(a, grid, block, stream); break;
      case 2: launch_short_wt<DT, DH, NQ, 2>(a, grid, block, stream); break;
      case 3: launch_short_wt<DT, DH, NQ, 3>(a, grid, block, stream); break;
      default: launch_short_wt<DT, DH, NQ, 4>(a, grid, block, stream);
    }
  }
}

// Launches for the query-tile counts NQ_LO..NQ_HI (the instantiations are spread over several translation
// units, each covering a range, to keep compile times apart).
template <int DT, int DH, int NQ_LO, int NQ_HI>
static hipError_t launch_scores_t(const Shape &s, ScoreArgs &a, bool need_lse, bool need_scores, hipStream_t stream) {
  const int units = s.Bz * s.Hkv;
  const dim3 grid((unsigned)((size_t)units * s.n_groups * s.n_chunks)), block(kScoreWaves * kWave);
#define CKV_LAUNCH_NQ(NQ)                                                          \
  case NQ:                                                                         \
    if constexpr (NQ >= NQ_LO && NQ <= NQ_HI) {                                    \
      a.lse_from_part = need_lse && need_scores;                                   \
      if (a.marks) {                                                               \
        launch_short<DT, DH, NQ>(s, a, grid, block, stream);                       \
        break;                                                                     \
      }                                                                            \
      if (need_lse) launch_rowstats<DT, DH, NQ>(s, a, grid, block, stream);        \
      if (need_scores) launch_colsum<DT, DH, NQ>(s, a, grid, block, stream);       \
      break;                                                                       \
    }                                                                              \
    return hipErrorInvalidValue;
  switch (s.NQ) {
    CKV_LAUNCH_NQ(1)
    CKV_LAUNCH_NQ(2)
    CKV_LAUNCH_NQ(3)
    CKV_LAUNCH_NQ(4)
    CKV_LAUNCH_NQ(5)
    CKV_LAUNCH_NQ(6)
    CKV_LAUNCH_NQ(7)
    CKV_LAUNCH_NQ(8)
    default: return hipErrorInvalidValue;
  }
#undef CKV_LAUNCH_NQ
  return hipGetLastError();
}


// One definition per (element type, head size, range of query-tile counts), each in a translation unit of
// its own.
#define CKV_DECLARE_SCAN(name) \
  hipError_t name(const Shape &s, ScoreArgs &a, bool need_lse, bool need_scores, hipStream_t stream)
CKV_DECLARE_SCAN(launch_scores_bf16_d128);       // 1..4 query tiles per wave
CKV_DECLARE_SCAN(launch_scores_bf16_d128_nq56);
CKV_DECLARE_SCAN(launch_scores_bf16_d128_nq78);
CKV_DECLARE_SCAN(launch_scores_bf16_d64);
CKV_DECLARE_SCAN(launch_scores_bf16_d64_nq56);
CKV_DECLARE_SCAN(launch_scores_bf16_d64_nq78);
CKV_DECLARE_SCAN(launch_scores_f32_d128);
CKV_DECLARE_SCAN(launch_scores_f32_d64);

}  // namespace ckv
#endif
