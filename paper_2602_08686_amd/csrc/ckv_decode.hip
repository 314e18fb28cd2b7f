// Decode-side consumer of the compact cache (paper Sec. 4.5, Proposition 1 and its proof in App. A).
// A decoding query sits after the prompt, so it sees every row of a KV set; over the retained set its
// attention row is the full row restricted to S and renormalised (p~ of the Proposition), and the mass
// the full row had outside S is m = 1 - exp(lse_S - lse_full).
//
// Attention of decoding queries over a ragged KV set (the first count[b,g] rows of each (batch, KV head)). HBM-bound:
// every valid K and V row once, 2 * rows * d * e bytes per unit.
//
// bf16 (decode_mfma_kernel): both products on the matrix cores. All decoding queries of a KV head, G * n_q of them, are
// the columns of one 16-wide tile, so a row is read once for all heads and queries, and the cost of a
// row does not grow with them (on the vector ALUs four heads take ~110 instructions per four rows and
// hold the sweep at 5 TB/s; here 32 rows take ~130 instructions and 32 MFMAs). Keys x queries leaves a lane with
// the logits of eight keys of one query, which is the operand layout of the second product; the rows
// of V come with whole rows per load and are transposed in registers (32 byte permutes per 32 rows). The
// weights enter it as three bf16 terms that add up to the fp32 value exactly. A wave takes 32 rows at a time and
// asks for the next 32 as soon as the registers of the current ones are free. Waves are combined in LDS in wave
// order, chunks by decode_merge_kernel in chunk order (bit-stable).
// Measured, us per call, before (vector ALUs, a sweep per query and two to eight heads) -> now: batch 4, 32/8 heads, 32k rows
// 118.0 -> 86.1 (6.2 TB/s); 544 rows, batch 16: 13.6 -> 10.0; 20000 rows, batch 8, 32/4 heads, two queries 372 -> 60.
// RMS error against 64 bits 2.7e-7 -> 2.0e-7 on the first of them. Not faster: both blocks of two in registers at once
// (85.2, and 11.2 on 544 rows).
//
// f32, and long bf16 rows with one query column (decode_partial_kernel): dot products on the vector ALUs, a 16-byte piece of a row per
// lane, online softmax in the log2 domain, the query heads of a group sharing each row.
#include <type_traits>

#include "ckv_internal.h"

namespace ckv {

struct DecodeArgs {
  const void *q;         // [Bz][Hq][n_q][d]
  const void *k, *v;     // rows of (batch, kv head) through the strides below
  const int32_t *count;  // [Bz*Hkv] valid rows, or null: all n_rows
  int64_t ks[3], vs[3];  // element strides over (batch, kv head, row)
  float *part;           // [grid.y][n_chunks][RQ][d + 2]: weighted V sum, running max (log2), sum
  float *out;            // [Bz][Hq][n_q][d]
  float *lse;            // [Bz][Hq][n_q] natural log
  int Hq, Hkv, G, n_q, n_rows, n_chunks, head_chunks;
  int cols, col_chunks;  // bf16: query columns per KV head (G * n_q) and 16-column tiles of them
  int part_cols;         // columns of a tile's partial: min(16, cols)
  float scale2;          // softmax scale * log2(e)
};

constexpr int kXcds = 8;  // accelerator dies of the part; workgroup i of a launch runs on die i % 8
constexpr int kDecodeThreads = 256;
constexpr int kDecodeWaves = kDecodeThreads / kWave;

// A 16-byte piece of a row: four f32 or eight bf16.
__device__ __forceinline__ void piece_to_float(const uint4 &raw, float (&f)[4]) {
  f[0] = __uint_as_float(raw.x);
  f[1] = __uint_as_float(raw.y);
  f[2] = __uint_as_float(raw.z);
  f[3] = __uint_as_float(raw.w);
}
__device__ __forceinline__ void piece_to_float(const uint4 &raw, float (&f)[8]) {
  const uint32_t words[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f[2 * i] = __uint_as_float(words[i] << 16);
    f[2 * i + 1] = __uint_as_float(words[i] & 0xffff0000u);
  }
}

// Rows of a chunk: a unit's chunks share its valid rows evenly, in whole steps of the workgroup. (With chunks of n_rows instead, a
// cache with many more rows than counts left most of its workgroups without any.)
template <int STEP>
__device__ __forceinline__ int chunk_rows(const DecodeArgs &a, int n_valid) {
  return max(1, (int)((uint32_t)(n_valid + a.n_chunks * STEP - 1) / (uint32_t)(a.n_chunks * STEP))) * STEP;
}
constexpr int kVectorStep = 64;

// exp2(a - b) with the conventions of an online softmax: a = -inf gives 0 also when b was reset to 0
__device__ __forceinline__ float exp2_diff(float a, float b) { return exp2f(a - b); }

// NW waves per workgroup, U row steps whose loads are in flight together (PIPE: of the next block too). With one chunk per
// (unit, query) the workgroup writes the final result itself and no merge kernel follows.
template <int DT, int DH, int RQ, int NW, int U, bool PIPE>
__global__ void __launch_bounds__(NW *kWave) decode_partial_kernel(DecodeArgs a) {
  constexpr int ESIZE = DT == CKV_BF16 ? 2 : 4, E = 16 / ESIZE;
  // bf16: weights times V summed in 64 bits, which makes the result as exact as the matrix form's (RMS error against 64 bits, 9000 rows:
  // 2.1e-7 with an f32 sum, 1.9e-7; matrix 1.9e-7) for 1 to 8 % of the time.
  typedef typename std::conditional<DT == CKV_BF16, double, float>::type sum_t;
  constexpr int LPR = DH / E;        // lanes per row
  constexpr int KPW = kWave / LPR;   // rows per wave step
  constexpr int ROW = DH + 2;
  constexpr bool STREAM = NW == kDecodeWaves;  // the chunked form sweeps long caches once: streaming loads
  __shared__ float sm[NW][RQ][ROW];

  const int chunk = blockIdx.x;
  int y = blockIdx.y;
  // One launch over a short KV set: the workgroups that read the same rows (the head chunks of a unit) are
  // consecutive in y, and consecutive workgroups go to different XCDs, each with an L2 of its own -- the
  // rows would come from HBM once per head chunk. Within groups of 8 * head_chunks workgroups the index is
  // transposed, so that a unit's head chunks are 8 apart: same XCD, the second reader hits its L2.
  if (PIPE && a.head_chunks > 1) {
    const int span = kXcds * a.head_chunks, base = y / span * span;
    if (base + span <= (int)gridDim.y) {
      const int j = y - base;
      y = base + (j % kXcds) * a.head_chunks + j / kXcds;
    }
  }
  const int hc = y % a.head_chunks;
  y /= a.head_chunks;
  const int qi = y % a.n_q, unit = y / a.n_q;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sub = lane % LPR, slot = lane / LPR;
  int n_valid = a.n_rows;
  if (a.count) n_valid = min(max(a.count[unit], 0), a.n_rows);
  const bool single = a.n_chunks == 1;
  const int rows = single ? n_valid : chunk_rows<kVectorStep>(a, n_valid);
  const int r0 = chunk * rows, r1 = min(r0 + rows, n_valid);
  if (r0 >= r1 && !single) return;  // the merge reads the chunks below n_valid only

  float qv[RQ][E];
#pragma unroll
  for (int r = 0; r < RQ; ++r) {
    const int hg = hc * RQ + r;
    uint4 raw = make_uint4(0u, 0u, 0u, 0u);
    if (hg < a.G) {
      const size_t row = ((size_t)b * a.Hq + (size_t)g * a.G + hg) * a.n_q + qi;
      raw = *reinterpret_cast<const uint4 *>(static_cast<const char *>(a.q) + (row * DH + sub * E) * ESIZE);
    }
    piece_to_float(raw, qv[r]);
#pragma unroll
    for (int e = 0; e < E; ++e) qv[r][e] *= a.scale2;
  }

  float m[RQ], l[RQ];
  sum_t acc[RQ][E];
#pragma unroll
  for (int r = 0; r < RQ; ++r) {
    m[r] = -INFINITY;
    l[r] = 0.0f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[r][e] = 0;
  }

  const char *kb = static_cast<const char *>(a.k) + ((size_t)b * a.ks[0] + (size_t)g * a.ks[1]) * ESIZE;
  const char *vb = static_cast<const char *>(a.v) + ((size_t)b * a.vs[0] + (size_t)g * a.vs[1]) * ESIZE;
  // a wave takes KPW * U consecutive rows at a time; the workgroup's waves interleave such blocks
  // The loads of the wave's next block are issued before the current block is worked on: a short KV set
  // is a handful of dependent round trips otherwise.
  auto load_block = [&](int base, uint4 (&kraw)[U], uint4 (&vraw)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int row = base + u * KPW + slot;
      kraw[u] = make_uint4(0u, 0u, 0u, 0u);
      vraw[u] = make_uint4(0u, 0u, 0u, 0u);
      if (row < r1) {
        kraw[u] = load_piece<STREAM>(kb + ((size_t)row * a.ks[2] + sub * E) * ESIZE);
        vraw[u] = load_piece<STREAM>(vb + ((size_t)row * a.vs[2] + sub * E) * ESIZE);
      }
    }
  };
  uint4 kraw[U], vraw[U];
  const int base0 = r0 + wave * KPW * U;
  if (base0 < r1) load_block(base0, kraw, vraw);
  for (int base = base0; base < r1; base += NW * KPW * U) {
    uint4 knext[U], vnext[U];
    if (PIPE) load_block(base + NW * KPW * U, knext, vnext);  // rows at and beyond r1 are not read
    float s[U][RQ], vf[U][E];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float kf[E];
      piece_to_float(kraw[u], kf);
      piece_to_float(vraw[u], vf[u]);
      const bool ok = base + u * KPW + slot < r1;
#pragma unroll
      for (int r = 0; r < RQ; ++r) {
        float dot = 0.0f;
#pragma unroll
        for (int e = 0; e < E; ++e) dot = fmaf(qv[r][e], kf[e], dot);
        dot = row_sum<LPR>(dot);  // the row's lanes all end with the sum
        s[u][r] = ok ? dot : -INFINITY;
      }
    }
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      float mx = s[0][r];
#pragma unroll
      for (int u = 1; u < U; ++u) mx = fmaxf(mx, s[u][r]);
      const float m_new = fmaxf(m[r], mx);
      const float ref = m_new == -INFINITY ? 0.0f : m_new;
      const float keep = exp2_diff(m[r], ref);
      l[r] *= keep;
#pragma unroll
      for (int e = 0; e < E; ++e) acc[r][e] *= keep;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float p = exp2_diff(s[u][r], ref);
        l[r] += p;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[r][e] = fma((sum_t)p, (sum_t)vf[u][e], acc[r][e]);
      }
      m[r] = m_new;
    }
    if (PIPE) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        kraw[u] = knext[u];
        vraw[u] = vnext[u];
      }
    } else if (base + NW * KPW * U < r1) {
      load_block(base + NW * KPW * U, kraw, vraw);
    }
  }

  // the wave's row slots, in a fixed butterfly order
#pragma unroll
  for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
      const float m_o = __shfl_xor(m[r], o), l_o = __shfl_xor(l[r], o);
      const float m_new = fmaxf(m[r], m_o);
      const float ref = m_new == -INFINITY ? 0.0f : m_new;
      // both partners must add in the same order for identical results: lower lane's value first
      const bool low = (lane & o) == 0;
      const float f_self = exp2_diff(m[r], ref), f_other = exp2_diff(m_o, ref);
      l[r] = low ? fmaf(l[r], f_self, l_o * f_other) : fmaf(l_o, f_other, l[r] * f_self);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const sum_t a_o = __shfl_xor(acc[r][e], o), s = f_self, t = f_other;
        acc[r][e] = low ? fma(acc[r][e], s, a_o * t) : fma(a_o, t, acc[r][e] * s);
      }
      m[r] = m_new;
    }
  }
  if (slot == 0) {
#pragma unroll
    for (int r = 0; r < RQ; ++r) {
#pragma unroll
      for (int e = 0; e < E; ++e) sm[wave][r][sub * E + e] = (float)acc[r][e];
      if (sub == 0) {
        sm[wave][r][DH] = m[r];
        sm[wave][r][DH + 1] = l[r];
      }
    }
  }
  __syncthreads();
  if (single) {
    for (int i = tid; i < RQ * DH; i += NW * kWave) {
      const int r = i / DH, c = i % DH;
      const int hg = hc * RQ + r;
      if (hg >= a.G) continue;
      float top = sm[0][r][DH];
#pragma unroll
      for (int w = 1; w < NW; ++w) top = fmaxf(top, sm[w][r][DH]);
      const float ref = top == -INFINITY ? 0.0f : top;
      float num = 0.0f, den = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = exp2_diff(sm[w][r][DH], ref);
        num = fmaf(sm[w][r][c], f, num);
        den = fmaf(sm[w][r][DH + 1], f, den);
      }
      const size_t row = ((size_t)b * a.Hq + (size_t)g * a.G + hg) * a.n_q + qi;
      a.out[row * DH + c] = den > 0.0f ? num / den : 0.0f;
      if (c == 0) a.lse[row] = den > 0.0f ? (top + log2f(den)) * kLn2 : -INFINITY;
    }
    return;
  }
  float *part = a.part + ((size_t)blockIdx.y * a.n_chunks + chunk) * RQ * ROW;
  for (int i = tid; i < RQ * ROW; i += NW * kWave) {
    const int r = i / ROW, c = i % ROW;
    float top = sm[0][r][DH];
#pragma unroll
    for (int w = 1; w < NW; ++w) top = fmaxf(top, sm[w][r][DH]);
    const float ref = top == -INFINITY ? 0.0f : top;
    float val;
    if (c == DH) val = top;
    else {
      const int src = c < DH ? c : DH + 1;  // a V component, or the sum
      val = 0.0f;
#pragma unroll
      for (int w = 0; w < NW; ++w) val = fmaf(sm[w][r][src], exp2_diff(sm[w][r][DH], ref), val);
    }
    part[i] = val;
  }
}

// ---------------------------------------------------------------------------------------------
// bf16: matrix cores
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_d;
typedef __attribute__((ext_vector_type(4))) float f32x4_dec;
constexpr int kCols = 16;       // query columns of a tile
constexpr int kBlockRows = 32;  // rows a wave takes at a time
constexpr int kFlatStep = kDecodeWaves * kBlockRows;

__device__ __forceinline__ void mma16(f32x4_dec &acc, const u32x4_d &x, const u32x4_d &y) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_d, x), __builtin_bit_cast(bf16x8_d, y), acc, 0, 0, 0);
}
// Largest value / sum over the four lanes that hold one query column (lane, lane ^ 16, lane ^ 32, lane ^ 48).
template <class Op>
__device__ __forceinline__ float over_quarters(float x, Op op) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// High halves of two words side by side (x below y): two truncated bf16 of an operand.
__device__ __forceinline__ uint32_t high_halves(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x07060302); }
__device__ __forceinline__ uint32_t low_halves(uint32_t x, uint32_t y) { return __builtin_amdgcn_perm(y, x, 0x05040100); }

// SPLIT: workgroups that share a unit's columns, each with all of K and a SPLIT-th of V's components. One CU takes in about
// 60 GB/s; where units are fewer than CUs this is how more of them read (8 units of 4096 rows, four heads each: 40.6
// us with one, 34.5 with four).
template <int DH, int SPLIT, int NW, bool STREAM>
__global__ void __launch_bounds__(NW *kWave, 2) decode_mfma_kernel(DecodeArgs a) {
  constexpr int STEPS = DH / 32;     // MFMAs per 16 keys
  constexpr int DV = DH / SPLIT;     // components of V
  constexpr int VE = DV / 16;        // elements of a V row per lane: 8, 4 or 2
  constexpr int VW = VE / 2;         // words of them
  constexpr int ROW = DV + 2;
  __shared__ float sm[NW][kCols][ROW];
  const int chunk = blockIdx.x;
  int y = blockIdx.y;
  // Workgroups that read the same rows (the column tiles and splits of a unit) onto one XCD, whose L2 then serves all but the
  // first: consecutive workgroups go to different XCDs, so within groups of 8 x sharers the index is transposed.
  const int sharers = a.col_chunks * SPLIT;
  if (gridDim.x == 1 && sharers > 1) {
    const int span = kXcds * sharers, base = y / span * span;
    if (base + span <= (int)gridDim.y) {
      const int j = y - base;
      y = base + (j % kXcds) * sharers + j / kXcds;
    }
  }
  const int split = y % SPLIT;
  y /= SPLIT;
  const int cc = y % a.col_chunks, unit = y / a.col_chunks;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), m = lane & 15, quarter = lane >> 4;
  const int n_cols = min(kCols, a.cols - cc * kCols);  // columns of this tile that exist
  const size_t q_row = ((size_t)b * a.Hq + (size_t)g * a.G) * a.n_q + cc * kCols;  // first of them in q, out and lse
  const bool single = a.n_chunks == 1;

  u32x4_d qf[STEPS];  // lane (m, quarter): column m, the 16-byte pieces 4 * step + quarter of its row
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    qf[s] = u32x4_d{0u, 0u, 0u, 0u};
    if (m < n_cols)
      qf[s] = *reinterpret_cast<const u32x4_d *>(static_cast<const char *>(a.q) + ((q_row + m) * DH + (4 * s + quarter) * 8) * 2);
  }
  const char *kb = static_cast<const char *>(a.k) + ((size_t)b * a.ks[0] + (size_t)g * a.ks[1]) * 2 + quarter * 16;
  const char *vb = static_cast<const char *>(a.v) + ((size_t)b * a.vs[0] + (size_t)g * a.vs[1]) * 2 + (split * DV + m * VE) * 2;
  const int64_t ks = a.ks[2] * 2, vs = a.vs[2] * 2;  // bytes per row

  // K: key row 16 t + m of the block, as the query pieces. V: the rows whose logits the lane will hold,
  // j -> 16 (j / 4) + 4 quarter + j % 4, piece m. Rows at and beyond `end` are not read.
  u32x4_d kraw[2][STEPS];
  uint32_t vraw[8][VW];
  auto load_k = [&](int base, int end) {
    const bool whole = base + kBlockRows <= end;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int row = base + 16 * t + m;
      const char *p = kb + (int64_t)row * ks;
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
        if (!whole) kraw[t][s] = u32x4_d{0u, 0u, 0u, 0u};
        if (whole || row < end) {
          if (STREAM) kraw[t][s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_d *>(p + s * 64));
          else kraw[t][s] = *reinterpret_cast<const u32x4_d *>(p + s * 64);
        }
      }
    }
  };
  typedef __attribute__((ext_vector_type(VW))) uint32_t piece_v;
  auto load_v = [&](int base, int end) {
    const bool whole = base + kBlockRows <= end;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int row = base + 16 * (j / 4) + 4 * quarter + j % 4;
      piece_v v;
#pragma unroll
      for (int w = 0; w < VW; ++w) v[w] = 0u;
      if (whole || row < end) {
        const piece_v *p = reinterpret_cast<const piece_v *>(vb + (int64_t)row * vs);
        if (STREAM) v = __builtin_nontemporal_load(p);
        else v = *p;
      }
#pragma unroll
      for (int w = 0; w < VW; ++w) vraw[j][w] = v[w];
    }
  };

  // nothing behind the count is read: its rows need not even be mapped
  int n_valid = a.n_rows;
  if (a.count) n_valid = min(max(a.count[unit], 0), a.n_rows);
  const int rows = single ? n_valid : chunk_rows<kFlatStep>(a, n_valid);
  const int r0 = chunk * rows, r1 = min(r0 + rows, n_valid), base0 = r0 + wave * kBlockRows;
  if (r0 >= r1 && !single) return;  // the merge reads the chunks below n_valid only
  if (base0 < r1) {
    load_k(base0, r1);
    load_v(base0, r1);
  }

  float top = -INFINITY, sum = 0.0f;  // of column m: the running maximum (the wave's), this lane's share of the sum
  f32x4_dec acc[VE];                  // element e: D[4 quarter + r][column m] = component VE (4 quarter + r) + e
  // WITH_INFINITIES: infinite and NaN components of V by themselves, times one where the weight is above zero (the second and
  // third term of a weight may be zero, and zero times infinity is none of the results that the weight itself would give).
  auto sweep = [&](auto with_infinities) {
    constexpr bool WITH_INFINITIES = decltype(with_infinities)::value;
    top = -INFINITY;
    sum = 0.0f;
#pragma unroll
    for (int e = 0; e < VE; ++e) acc[e] = f32x4_dec{0.0f, 0.0f, 0.0f, 0.0f};
    for (int base = base0; base < r1; base += NW * kBlockRows) {
      const int next = base + NW * kBlockRows;
      f32x4_dec s2[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {  // two chains per tile: half the truncated additions
        f32x4_dec half[2] = {f32x4_dec{0.0f, 0.0f, 0.0f, 0.0f}, f32x4_dec{0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int s = 0; s < STEPS; ++s) mma16(half[s & 1], kraw[t][s], qf[s]);
        s2[t] = half[0] + half[1];
      }
      if (next < r1) load_k(next, r1);
      float z[8];  // logits (log2 domain) of rows 16 (j / 4) + 4 quarter + j % 4
#pragma unroll
      for (int j = 0; j < 8; ++j) z[j] = s2[j / 4][j % 4] * a.scale2;
      if (base + kBlockRows > r1) {  // rows that are not there were not read either: zeros
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (base + 16 * (j / 4) + 4 * quarter + j % 4 >= r1) z[j] = -INFINITY;
      }
      float mx = fmaxf(fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3])), fmaxf(fmaxf(z[4], z[5]), fmaxf(z[6], z[7])));
      mx = over_quarters(mx, [](float p, float q) { return fmaxf(p, q); });
      if (__any(mx > top)) {  // after the first blocks a new maximum is rare
        const float t_new = fmaxf(top, mx);
        const float keep = exp2_diff(top, t_new == -INFINITY ? 0.0f : t_new);
        sum *= keep;
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[e] *= keep;
        top = t_new;
      }
      const float ref = top == -INFINITY ? 0.0f : top;
      // weights, and their three bf16 terms: truncations, each of what the ones before left
      u32x4_d w0, w1, w2, w3;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        uint32_t t0[2], t1[2], t2[2], t3[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const float p = __builtin_amdgcn_exp2f(z[2 * h + x] - ref);
          sum += p;
          t1[x] = __float_as_uint(p);
          const float r = p - __uint_as_float(t1[x] & 0xffff0000u);
          t2[x] = __float_as_uint(r);
          t3[x] = __float_as_uint(r - __uint_as_float(t2[x] & 0xffff0000u));
          if (WITH_INFINITIES) t0[x] = z[2 * h + x] - ref > -150.0f ? 0x3f800000u : 0u;  // 2^-150 rounds to zero
        }
        w1[h] = high_halves(t1[0], t1[1]);
        w2[h] = high_halves(t2[0], t2[1]);
        w3[h] = high_halves(t3[0], t3[1]);
        if (WITH_INFINITIES) w0[h] = high_halves(t0[0], t0[1]);
      }
      u32x4_d vt[VE];  // V transposed: component e of the lane's piece, its eight rows
#pragma unroll
      for (int e = 0; e < VE; ++e)
#pragma unroll
        for (int h = 0; h < 4; ++h)
          vt[e][h] = e % 2 ? high_halves(vraw[2 * h][e / 2], vraw[2 * h + 1][e / 2]) : low_halves(vraw[2 * h][e / 2], vraw[2 * h + 1][e / 2]);
      if (next < r1) load_v(next, r1);
      // the block's sum by itself, then one rounded addition: the matrix cores truncate what they add to an accumulator
      // that is larger than the products, and over a long sweep that adds up (7e-7 instead of 3e-7 after 8192 rows)
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        f32x4_dec head = {0.0f, 0.0f, 0.0f, 0.0f}, rest = head;
        if (WITH_INFINITIES) {
          u32x4_d beyond;  // the components that are not finite, the others zero
#pragma unroll
          for (int h = 0; h < 4; ++h) {
            const uint32_t x = vt[e][h];
            beyond[h] = ((x & 0x7f800000u) == 0x7f800000u ? x & 0xffff0000u : 0u) | ((x & 0x7f80u) == 0x7f80u ? x & 0xffffu : 0u);
            vt[e][h] = x ^ beyond[h];
          }
          mma16(rest, beyond, w0);
        }
        mma16(head, vt[e], w1);
        mma16(rest, vt[e], w3);
        mma16(rest, vt[e], w2);
        acc[e] += head + rest;
      }
    }
  };
  sweep(std::false_type{});
  bool undefined = false;
#pragma unroll
  for (int e = 0; e < VE; ++e)
#pragma unroll
    for (int r = 0; r < 4; ++r) undefined |= acc[e][r] != acc[e][r];
  if (__any(undefined)) {  // V has components that are not finite (or the logits have): once more, for what they give
    load_k(base0, r1);
    load_v(base0, r1);
    sweep(std::true_type{});
  }
  sum = over_quarters(sum, [](float p, float q) { return p + q; });

  if (m < n_cols) {
    float *to = sm[wave][m];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int e = 0; e < VE; ++e) to[VE * (4 * quarter + r) + e] = acc[e][r];
    if (quarter == 0) {
      to[DV] = top;
      to[DV + 1] = sum;
    }
  }
  __syncthreads();
  // the waves, in wave order (more than one chunk: SPLIT is 1)
  float *part = single ? nullptr : a.part + (((size_t)blockIdx.y * a.n_chunks + chunk) * a.part_cols) * ROW;
  for (int i = threadIdx.x; i < n_cols * DV; i += NW * kWave) {
    const int c = i / DV, x = i % DV;
    float mx = sm[0][c][DV];
#pragma unroll
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, sm[w][c][DV]);
    const float ref = mx == -INFINITY ? 0.0f : mx;
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float *from = sm[w][c];
      const float f = exp2_diff(from[DV], ref);
      num = fmaf(from[x], f, num);
      den = fmaf(from[DV + 1], f, den);
    }
    if (single) {
      a.out[(q_row + c) * DH + split * DV + x] = den > 0.0f ? num / den : 0.0f;
      if (x == 0 && split == 0) a.lse[q_row + c] = den > 0.0f ? (mx + log2f(den)) * kLn2 : -INFINITY;
    } else {
      part[c * ROW + x] = num;
      if (x == 0) {
        part[c * ROW + DV] = mx;
        part[c * ROW + DV + 1] = den;
      }
    }
  }
}

// Chunks of one (unit, query row): a lane per chunk for the maximum and the weights, a thread per component for the
// sum, its loads independent. One workgroup per query row (the first form, one per unit, kept 32 workgroups of the
// chip busy for 16.7 us on the 32k / batch-4 cache).
// FLAT: partials of the bf16 kernel, [(unit, column tile)][chunk][part_cols][d + 2]; else [(unit, query, head chunk)][chunk][RQ][d + 2].
constexpr int kMaxChunks = 64;
template <int DH, int RQ, bool FLAT>
__global__ void __launch_bounds__(DH) decode_merge_kernel(DecodeArgs a) {
  constexpr int ROW = DH + 2;
  __shared__ float s_weight[kMaxChunks];
  __shared__ float s_top, s_den;
  const int row = blockIdx.x;  // of [Bz][Hq][n_q]
  const int head = row / a.n_q, qi = row % a.n_q, b = head / a.Hq, h = head % a.Hq, g = h / a.G, hg = h % a.G;
  const int unit = b * a.Hkv + g;
  size_t first;  // partial row of chunk 0
  if (FLAT) {
    const int c = hg * a.n_q + qi;
    first = ((size_t)unit * a.col_chunks + c / kCols) * a.n_chunks * a.part_cols + c % kCols;
  } else {
    first = (((size_t)unit * a.n_q + qi) * a.head_chunks + hg / RQ) * a.n_chunks * RQ + hg % RQ;
  }
  const int stride = (FLAT ? a.part_cols : RQ) * ROW;
  const float *part = a.part + first * ROW;
  int n_valid = a.n_rows;
  if (a.count) n_valid = min(max(a.count[unit], 0), a.n_rows);
  const int rows = chunk_rows<FLAT ? kFlatStep : kVectorStep>(a, n_valid);
  const int n_chunks = (n_valid + rows - 1) / rows;  // the chunks that were written
  if (threadIdx.x < kWave) {
    const int c = threadIdx.x;
    const float top = c < n_chunks ? part[(size_t)c * stride + DH] : -INFINITY;
    const float sum = c < n_chunks ? part[(size_t)c * stride + DH + 1] : 0.0f;
    float mx = top;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    const float w = exp2_diff(top, mx == -INFINITY ? 0.0f : mx);
    float den = sum * w;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) den += __shfl_xor(den, o);
    s_weight[c] = w;
    if (c == 0) {
      s_top = mx;
      s_den = den;
    }
  }
  __syncthreads();
  float num = 0.0f;
  const int x = threadIdx.x;
  constexpr int BATCH = 16;
  for (int c0 = 0; c0 < n_chunks; c0 += BATCH) {
    float v[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) v[j] = c0 + j < n_chunks ? part[(size_t)(c0 + j) * stride + x] : 0.0f;
#pragma unroll
    for (int j = 0; j < BATCH; ++j) num = fmaf(v[j], c0 + j < n_chunks ? s_weight[c0 + j] : 0.0f, num);
  }
  const float den = s_den;
  a.out[(size_t)row * DH + x] = den > 0.0f ? num / den : 0.0f;
  if (x == 0) a.lse[row] = den > 0.0f ? (s_top + log2f(den)) * kLn2 : -INFINITY;
}

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
static int query_rows_per_pass(int G) { return G >= 8 ? 8 : G > 2 ? 4 : G; }  // 1, 2, 4, 8 (G = 3 pads to 4)

static int64_t least64(int64_t x, int64_t y) { return x < y ? x : y; }

// bf16, long rows: rows per chunk. Two workgroups of four waves fit a CU, but one of them takes in nearly as much as both, so the
// work of the fullest CU counts: ceil(workgroups / 256) x (rows + set-up), the set-up (its partial's way through the merge
// included) being worth 16 rows per query column; a tenth more where a CU has one workgroup only, and a tenth of a chunk's rows
// where not all workgroups are resident from the start.
// Measured against what fills the chip once (512 / workgroups chunks, rounded down), us, rows of 128: 264 workgroups, 4200 rows 142
// -> 94 (11 chunks), 320, 9000 rows 315 -> 235 (4 or 8), 136, 9000 rows 118 -> 104 (15), 96, 9000 rows 80 -> 76 (8); the same chunks as
// before for 32 x 32768, 56 x 9000, 128 x 9000 and 512 x 4200.
static int64_t mfma_chunk_rows(int64_t workgroups, int64_t cols, int n_rows, int most) {
  constexpr int STEP = kFlatStep;
  const int64_t set_up = 4 + 16 * cols;
  int64_t best = 0, best_cost = INT64_MAX;
  for (int chunks = 1; chunks <= most; ++chunks) {
    const int64_t rows = (n_rows + chunks * STEP - 1) / (chunks * STEP) * STEP;
    const int64_t n = workgroups * ((n_rows + rows - 1) / rows), per_cu = (n + kComputeUnits - 1) / kComputeUnits;
    const int64_t cost = (per_cu == 1 ? 11 : 10 * per_cu) * (rows + set_up) + (n > 2 * kComputeUnits ? rows : 0);
    if (cost < best_cost) {
      best = rows;
      best_cost = cost;
    }
  }
  return best;
}

DecodePlan plan_decode(const Shape &s, int n_q, int n_rows) {
  DecodePlan p;
  p.mfma = s.esize == 2;
  p.rq = query_rows_per_pass(s.G);
  p.head_chunks = (s.G + p.rq - 1) / p.rq;
  p.grid_y = (int64_t)s.Bz * s.Hkv * n_q * p.head_chunks;
  p.col_chunks = (int)(((int64_t)s.G * n_q + kCols - 1) / kCols);
  p.workgroups = (int64_t)s.Bz * s.Hkv * p.col_chunks;
  // Short KV sets (a compact cache): one large workgroup per unit and query tile (f32: per query and pair of heads)
  // finishes the job in one launch -- a decoding step is a chain of dependent layers, and a second launch
  // costs more than it saves.
  if (n_rows <= 4096 || (p.grid_y >= 1024 && n_rows <= 16384)) {
    p.rq = s.G >= 2 ? 2 : 1;
    p.head_chunks = (s.G + p.rq - 1) / p.rq;
    p.grid_y = (int64_t)s.Bz * s.Hkv * n_q * p.head_chunks;
    p.n_chunks = 1;
    p.workspace_bytes = 0;
    return p;
  }
  // bf16 with one query column per KV head (no grouped heads, one query) has nothing for the other columns of a tile, and on the
  // vector ALUs sixteen waves per CU keep more rows in flight than the eight that the tile's registers leave. Long rows, us, vector
  // / matrix: 136 units of 128, counts of 2500 of 5000 35 / 45, of 1050 of 9000 22 / 30; 320 units, 1100 of 9000 39 / 52; 640 units, 4200 rows
  // 219 / 231; 320 units of 64, 9000 rows 118 / 164. With fewer units than half the CUs, and up to 4096 rows, the matrix form is about as
  // fast or faster (V is shared out over workgroups there).
  if (s.G * (int64_t)n_q == 1 && p.workgroups >= kComputeUnits / 2) p.mfma = false;
  // At most 64 chunks, of whole steps of a workgroup. On the vector ALUs: workgroups for several times the chip.
  const int64_t step = p.mfma ? kFlatStep : kVectorStep, most = least64(kMaxChunks, (n_rows + step - 1) / step);
  int64_t rows;
  if (p.mfma) {
    rows = mfma_chunk_rows(p.workgroups, least64(kCols, (int64_t)s.G * n_q), n_rows, (int)most);
  } else {
    const int64_t chunks = least64(most, (4096 + p.grid_y - 1) / p.grid_y);
    rows = ((n_rows + chunks - 1) / chunks + step - 1) / step * step;
  }
  p.n_chunks = (int)((n_rows + rows - 1) / rows);
  const size_t part_rows = p.mfma ? (size_t)p.workgroups * least64(kCols, (int64_t)s.G * n_q) : (size_t)p.grid_y * p.rq;
  p.workspace_bytes = part_rows * p.n_chunks * (s.d + 2) * sizeof(float);
  return p;
}

template <int DH, int SPLIT, int NW>
static void launch_decode_short(const DecodeArgs &a, const DecodePlan &p, hipStream_t stream) {
  hipLaunchKernelGGL((decode_mfma_kernel<DH, SPLIT, NW, false>), dim3(1, (unsigned)p.workgroups * SPLIT), dim3(NW * kWave), 0,
                     stream, a);
}

template <int DH>
static void launch_decode_bf16(const DecodeArgs &a, const DecodePlan &p, int rows, hipStream_t stream) {
  if (p.workspace_bytes == 0) {
    // as many splits as leave every workgroup a CU of its own
    if (DH == 128 && p.workgroups * 4 <= kComputeUnits) launch_decode_short<DH, DH / 32, 16>(a, p, stream);
    else if (p.workgroups * 2 <= kComputeUnits) launch_decode_short<DH, 2, DH == 64 ? 16 : 8>(a, p, stream);
    else launch_decode_short<DH, 1, 8>(a, p, stream);
    return;
  }
  hipLaunchKernelGGL((decode_mfma_kernel<DH, 1, kDecodeWaves, true>), dim3(p.n_chunks, (unsigned)p.workgroups),
                     dim3(kDecodeThreads), 0, stream, a);
  if (p.n_chunks > 1)  // one chunk: the workgroups wrote the results
    hipLaunchKernelGGL((decode_merge_kernel<DH, 1, true>), dim3((unsigned)rows), dim3(DH), 0, stream, a);
}

template <int DT, int DH, int RQ>
static void launch_decode_vector(const DecodeArgs &a, const DecodePlan &p, int rows, hipStream_t stream) {
  if constexpr (DT == CKV_F32 && RQ <= 2) {
    if (p.n_chunks == 1) {
      hipLaunchKernelGGL((decode_partial_kernel<DT, DH, RQ, 16, 2, true>), dim3(1, (unsigned)p.grid_y),
                         dim3(16 * kWave), 0, stream, a);
      return;
    }
  }
  hipLaunchKernelGGL((decode_partial_kernel<DT, DH, RQ, kDecodeWaves, 4, false>), dim3(p.n_chunks, (unsigned)p.grid_y),
                     dim3(kDecodeThreads), 0, stream, a);
  if (p.n_chunks > 1)  // one chunk: the workgroups wrote the results
    hipLaunchKernelGGL((decode_merge_kernel<DH, RQ, false>), dim3((unsigned)rows), dim3(DH), 0, stream, a);
}

template <int DH>
static void launch_decode_rq(const DecodeArgs &a, const DecodePlan &p, int rows, hipStream_t stream) {
  switch (p.rq) {
    case 1: launch_decode_vector<CKV_F32, DH, 1>(a, p, rows, stream); break;
    case 2: launch_decode_vector<CKV_F32, DH, 2>(a, p, rows, stream); break;
    case 4: launch_decode_vector<CKV_F32, DH, 4>(a, p, rows, stream); break;
    default: launch_decode_vector<CKV_F32, DH, 8>(a, p, rows, stream); break;
  }
}

hipError_t launch_decode_attention(const ckv_params *p, const Shape &s, const void *q_dec, int n_q, const void *k_rows,
                                   const void *v_rows, const int64_t *k_stride, const int64_t *v_stride, int n_rows,
                                   const int32_t *count, float *out, float *lse, char *ws, hipStream_t stream) {
  const DecodePlan plan = plan_decode(s, n_q, n_rows);
  DecodeArgs a;
  a.q = q_dec;
  a.k = k_rows;
  a.v = v_rows;
  a.count = count;
  for (int i = 0; i < 3; ++i) {
    a.ks[i] = k_stride[i];
    a.vs[i] = v_stride[i];
  }
  a.part = reinterpret_cast<float *>(ws);
  a.out = out;
  a.lse = lse;
  a.Hq = s.Hq; a.Hkv = s.Hkv; a.G = s.G;
  a.n_q = n_q;
  a.n_rows = n_rows;
  a.n_chunks = plan.n_chunks;
  a.head_chunks = plan.head_chunks;
  a.scale2 = s.scale * kLog2e;
  a.cols = s.G * n_q;
  a.col_chunks = plan.col_chunks;
  a.part_cols = (int)least64(kCols, a.cols);
  const int rows = s.Bz * s.Hq * n_q;
  if (p->dtype == CKV_BF16) {
    if (!plan.mfma && s.d == 128) launch_decode_vector<CKV_BF16, 128, 1>(a, plan, rows, stream);
    else if (!plan.mfma) launch_decode_vector<CKV_BF16, 64, 1>(a, plan, rows, stream);
    else if (s.d == 128) launch_decode_bf16<128>(a, plan, rows, stream);
    else launch_decode_bf16<64>(a, plan, rows, stream);
  } else {
    if (s.d == 128) launch_decode_rq<128>(a, plan, rows, stream);
    else launch_decode_rq<64>(a, plan, rows, stream);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Discarded mass and tail epsilon from the two normalisers
// ---------------------------------------------------------------------------------------------
struct MassArgs {
  const float *lse_full, *lse_kept;  // [rows][n_q]
  float *mass;                       // [rows][n_q]
  float *eps;                        // [rows] or null
  int rows, n_q;
};

__global__ void __launch_bounds__(256) discarded_mass_kernel(MassArgs a) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  if (row >= a.rows) return;
  float sq = 0.0f;
  for (int i = 0; i < a.n_q; ++i) {
    const size_t j = (size_t)row * a.n_q + i;
    // retained mass exp(lse_S - lse) <= 1; expm1 keeps small discarded masses accurate
    float m = -expm1f(a.lse_kept[j] - a.lse_full[j]);
    m = fminf(fmaxf(m, 0.0f), 1.0f);
    a.mass[j] = m;
    sq = fmaf(m, m, sq);
  }
  if (a.eps) a.eps[row] = sqrtf(sq / (float)a.n_q);
}

hipError_t launch_discarded_mass(const Shape &s, int n_q, const float *lse_full, const float *lse_kept, float *mass,
                                 float *eps, hipStream_t stream) {
  MassArgs a;
  a.lse_full = lse_full;
  a.lse_kept = lse_kept;
  a.mass = mass;
  a.eps = eps;
  a.rows = s.Bz * s.Hq;
  a.n_q = n_q;
  hipLaunchKernelGGL(discarded_mass_kernel, dim3((a.rows + 255) / 256), dim3(256), 0, stream, a);
  return hipGetLastError();
}

}  // namespace ckv
