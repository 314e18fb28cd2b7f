// Elastic candidate pool with budget clamp (paper Eq. 8, Alg. 1 Select) as a radix select.
//
// Utilities are non-negative floats, so their bit patterns order like integers: a key is the pattern of a
// candidate and -1 of anything else. Everything is counted with integers (order-independent, so the result
// does not depend on scheduling), kept positions leave in ascending order, and equal keys at the threshold
// are taken lowest position first, which is exactly "utility descending, position ascending".
//
// select_keys() is the core, one workgroup with its keys in registers (thread tid holds slots i * NT + tid, so the
// lane mask of a comparison is 64 consecutive slots). What bounds it is vector instructions per key, the chain of
// dependent steps and the fetch of its code, not bytes: the keys are gone over three times (build, maximum,
// one comparison), everything after that works on the few that can still be kept.
//   1. A lower bound of the threshold: the kp-th largest of the maxima of more than kp groups of keys (a thread's
//      keys, or each four of them where kp exceeds half the threads). With 1024 groups of 32 and kp = 480 about 2 %
//      of the keys lie above it, so the keys themselves need no histogram. The maxima's histogram spans their own
//      range: pooled window masses lie within +-30 %, where bins on fixed bits of the float would be a
//      handful of counters (same-address atomics, thousands of undecided keys in the threshold's bin).
//   2. Slots of keys at or above the bound go to a list in LDS, in order: a wave's masks are dealt to its lanes and
//      each lane walks the set bits of its own.
//   3. The threshold among the list's keys (read again, by slot): a histogram; where its bin holds at most 64 keys,
//      a comparison of all with all that every wave does for itself; else further digits.
//   4. The list's kept entries, in its order.
// Where too few groups hold candidates, the histogram goes over all keys; where the list would exceed its
// capacity (budgets in the thousands, masses of equal keys) and where a thread holds at most eight keys, the
// threshold is searched over the registers and every lane writes its own kept slots.
// Measured, us per call, graph of 20 calls, 32 units (before: 8- and 11-bit digits of all keys in registers): 1k / budget
// 128: 7.4 -> 4.7, 4k / 512: 8.5 -> 5.8, 16k / 256: 16.1 -> 7.6, 32k / 512: 27.7 -> 9.2; 32737 positions, before by
// the streaming kernel: 44.3 -> 9.3. Inside a 32k call of 10 us: loads 1.9, keys and maxima 1.6, their histogram 1.0,
// list 2.5, threshold 1.5, output 1.3. A launch costs 4.6 of them.
//
// Who calls the core: select_reg_kernel, one workgroup per (batch, KV head) with up to 65536 positions; keep_kernel, several
// workgroups per head that also copy the rows they keep;
// select_slice_kernel + select_merge_kernel, for longer rows a workgroup per 8192 or 16384 positions and one per unit
// on what the slices kept. select_split_kernel (budgets so large that slices keep nearly everything) and
// select_kernel (no workspace) stay for the rest.
#include "ckv_internal.h"

// x with lane `lane` (a constant) replaced by the wave-uniform v: one instruction, which has no builtin of its own.
extern "C" __device__ int ckv_llvm_writelane(int v, int lane, int x) __asm("llvm.amdgcn.writelane.i32");

namespace ckv {

__device__ __forceinline__ int write_lane(int v, int lane, int x) { return ckv_llvm_writelane(v, lane, x); }

struct SelectArgs {
  const float *utility;   // [units][P]
  const int32_t *budget;  // [units]
  const float *tau;       // [Bz]
  int32_t *idx;           // [units][cap]
  int32_t *count;         // [units]
  int Hkv, T, W, P, cap;
};

// -0.0 and anything negative order like +0.0; NaN is no candidate
__device__ __forceinline__ int key_of(float u, float tau) { return u >= tau ? max(__float_as_int(u), 0) : -1; }

// Prefix slots of a unit: its budget without the window's.
__device__ __forceinline__ int prefix_quota(const SelectArgs &a, int unit) {
  return max(a.W, min(a.budget[unit], min(a.cap, a.T))) - a.W;
}

constexpr int kBins = 2048;
constexpr int kFewKeys = 64;  // undecided keys that a wave settles by comparing all with all

template <int NK, int NT>
struct SelectShared {
  static constexpr int NW = NT / kWave;
  static constexpr int NE = NK * NW;   // 64-slot entries
  static constexpr int NQ = 4;         // list entries per thread
  static constexpr int CAP = NQ * NT;  // list capacity
  int hist[kBins];
  int list[CAP];
  int cnt[NE > 64 ? NE : 64], cnt_eq[NE > 64 ? NE : 64];
  uint32_t red_max[NW], red_min[NW];
  int red_cnt[NW], bin_cnt[NW];
  __attribute__((aligned(16))) int few[kFewKeys];
  int n_few, bin, above, in_bin;
};

template <class Shared>
__device__ __forceinline__ void clear_hist(Shared &sh, int tid) {
  constexpr int NT = Shared::NW * kWave;
#pragma unroll
  for (int i = 0; i < kBins / NT; ++i) sh.hist[i * NT + tid] = 0;
}

// Bin of the histogram where the running count from the top first reaches k (1-based), the count above it and its
// own, into sh.bin / above / in_bin. All threads call it; hist is complete (behind a barrier); ends behind a barrier.
template <class Shared>
__device__ __forceinline__ void find_bin_block(Shared &sh, int k, int tid, int lane, int wave) {
  constexpr int NW = Shared::NW, PER = kBins / (NW * kWave);
  int c[PER], sum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    c[e] = sh.hist[kBins - 1 - PER * tid - e];
    sum += c[e];
  }
  const int incl = wave_inclusive(sum);
  if (lane == kWave - 1) sh.bin_cnt[wave] = incl;
  __syncthreads();
  const int waves = lane < NW ? sh.bin_cnt[lane] : 0;
  int run = (int)lane_value((uint32_t)(wave_inclusive(waves) - waves), wave) + incl - sum;
  if (run < k && k <= run + sum) {
    bool found = false;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (!found && run + c[e] >= k) {
        found = true;
        sh.bin = kBins - 1 - PER * tid - e;
        sh.above = run;
        sh.in_bin = c[e];
      }
      run += c[e];
    }
  }
  __syncthreads();
}

// For lane i: the sum of cnt in front of entry i * NW + wave (lanes at and beyond NK: anything). Every wave scans
// the NE entries for itself.
template <int NK, int NW>
__device__ __forceinline__ int entries_before(const int *cnt, int lane, int wave, int &total) {
  constexpr int NE = NK * NW, PER = (NE + kWave - 1) / kWave;
  static_assert(NW % PER == 0 || PER % NW == 0, "a wave's entries sit at one place of their lanes' runs");
  int sum = 0, part = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int c = lane * PER + e < NE ? cnt[lane * PER + e] : 0;
    if (PER <= NW && e == wave % PER) part = sum;
    sum += c;
  }
  const int incl = wave_inclusive(sum);
  total = (int)lane_value((uint32_t)incl, kWave - 1);
  return __shfl(incl - sum + part, (lane * NW + wave) / PER & (kWave - 1));
}

// The k-th largest of the workgroup's keys, which lie in [low, low + 2048 << shift) where they are at least low; k becomes
// how many of the keys equal to it are among the k. hist is clear; begins with a use of it. All threads call it.
template <int N, int NT, class Shared>
__device__ __forceinline__ int find_threshold(const int (&key)[N], int low, int shift, int &k, Shared &sh, int tid, int lane, int wave) {
  uint32_t prefix = 0u;       // digits of (threshold - low) found so far
  int rem = shift, b = 31;    // bits of this round's digit: the first one takes all that the shift leaves
  while (true) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const uint32_t off = (uint32_t)(key[q] - low);
      if (key[q] >= low && (off >> rem >> b) == prefix) atomicAdd(&sh.hist[(off >> rem) & ((1u << b) - 1u)], 1);
    }
    __syncthreads();
    find_bin_block(sh, k, tid, lane, wave);
    prefix = prefix << b | (uint32_t)sh.bin;
    k -= sh.above;
    if (rem == 0) return low + (int)prefix;
    const int in_bin = sh.in_bin;
    if (in_bin <= kFewKeys) {
#pragma unroll
      for (int q = 0; q < N; ++q)
        if (key[q] >= low && ((uint32_t)(key[q] - low) >> rem) == prefix) sh.few[atomicAdd(&sh.n_few, 1)] = key[q];
      __syncthreads();
      const int my = lane < in_bin ? sh.few[lane] : -1;
      int above = 0, equal = 0;
      for (int i = 0; i < in_bin; i += 4) {  // the same four words for every lane; beyond in_bin whatever is there
        const int4 other = *reinterpret_cast<const int4 *>(&sh.few[i]);
        const bool y = i + 1 < in_bin, z = i + 2 < in_bin, w = i + 3 < in_bin;
        above += (other.x > my) + (y && other.y > my) + (z && other.z > my) + (w && other.w > my);
        equal += (other.x == my) + (y && other.y == my) + (z && other.z == my) + (w && other.w == my);
      }
      const int src = __ffsll((long long)__ballot(lane < in_bin && above < k && k <= above + equal)) - 1;
      k -= (int)lane_value((uint32_t)above, src);
      return (int)lane_value((uint32_t)my, src);
    }
    __syncthreads();
    clear_hist(sh, tid);
    __syncthreads();
    b = min(rem, 11);
    rem -= b;
  }
}

// Kept slots in slot order, where few of a wave's keys are kept: write(rank, slot) of the keys at or above bound. A
// wave's masks are dealt to its lanes, lane i takes row i and walks its set bits. Returns how many there are.
template <int NK, int NT, class Write>
__device__ __forceinline__ int emit_sparse(SelectShared<NK, NT> &sh, const int (&key)[NK], int bound, Write write, int lane, int wave) {
  constexpr int NW = NT / kWave;
  static_assert(NK <= kWave, "a lane per mask");
  int lo = 0, hi = 0;
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const unsigned long long mask = __ballot(key[i] >= bound);
    lo = write_lane((int)(uint32_t)mask, i, lo);
    hi = write_lane((int)(uint32_t)(mask >> 32), i, hi);
  }
  if (lane < NK) sh.cnt[lane * NW + wave] = __popc(lo) + __popc(hi);
  __syncthreads();
  int total;
  int rank = entries_before<NK, NW>(sh.cnt, lane, wave, total);
  if (lane < NK) {
    unsigned long long mask = (uint32_t)lo | (unsigned long long)(uint32_t)hi << 32;
    while (mask) {
      write(rank++, lane * NT + wave * kWave + __ffsll((long long)mask) - 1);
      mask &= mask - 1;
    }
  }
  return total;
}

// Kept slots in slot order, any number of them: every lane writes its own, the keys above thr and the first need_eq
// equal to it, as write(rank, slot, key); base_gt / base_eq count those in front of the workgroup's keys, ranks at or
// beyond limit are dropped. Returns how many of the workgroup's there are.
template <int NK, int NT, class Write>
__device__ __forceinline__ int emit_keys(SelectShared<NK, NT> &sh, const int (&key)[NK], int thr, int need_eq, int limit, int base_gt,
                                         int base_eq, Write write, int tid, int lane, int wave) {
  constexpr int NW = NT / kWave;
  int counts = 0, counts_eq = 0;
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    counts = write_lane(__popcll(__ballot(key[i] > thr)), i, counts);
    counts_eq = write_lane(__popcll(__ballot(key[i] == thr)), i, counts_eq);
  }
  if (lane < NK) {
    sh.cnt[lane * NW + wave] = counts;
    sh.cnt_eq[lane * NW + wave] = counts_eq;
  }
  __syncthreads();
  int total, total_eq;
  const int g0 = entries_before<NK, NW>(sh.cnt, lane, wave, total), q0 = entries_before<NK, NW>(sh.cnt_eq, lane, wave, total_eq);
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int g = base_gt + (int)lanes_below(__ballot(key[i] > thr), lane_value((uint32_t)g0, i));
    const int q = base_eq + (int)lanes_below(__ballot(key[i] == thr), lane_value((uint32_t)q0, i));
    const int r = g + min(q, need_eq);
    if ((key[i] > thr || (key[i] == thr && q < need_eq)) && r < limit) write(r, i * NT + tid, key[i]);
  }
  return min(total + min(total_eq, need_eq), limit);
}

// Keys per thread up to which the threshold is searched and the kept slots are written from the registers.
constexpr int kDirectKeys = 8;
// Largest quota that goes by the list (capacity 4096): 16k positions, quota 4064: 18.4 us with the list tried first,
// 12.4 without.
constexpr int kListQuota = 3584;

// The kp largest keys (equal ones: lowest slot first), in slot order: write(rank, slot, key). reload(slot) is the key of
// a slot. kp >= 1. Returns how many were kept. All threads of the workgroup call it.
template <int NK, int NT, class Reload, class Write>
__device__ __forceinline__ int select_keys(const int (&key)[NK], int kp, SelectShared<NK, NT> &sh, Reload reload, Write write,
                                           int tid, int lane, int wave) {
  using Shared = SelectShared<NK, NT>;
  constexpr int NW = NT / kWave, NG = NK / 4;
  const auto larger = [](uint32_t p, uint32_t q) { return max(p, q); };
  const auto smaller = [](uint32_t p, uint32_t q) { return min(p, q); };

  // -- 1: group maxima (as unsigned numbers: no candidate is the largest, so it never is the smallest maximum)
  int four[NG], mine = -1;
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    four[q] = max(max(key[4 * q], key[4 * q + 1]), max(key[4 * q + 2], key[4 * q + 3]));
    mine = max(mine, four[q]);
  }
  const bool by_thread = 2 * kp <= NT;
  uint32_t least = (uint32_t)mine;
  int groups = mine >= 0;
  if (!by_thread) {
    groups = 0;
#pragma unroll
    for (int q = 0; q < NG; ++q) {
      least = min(least, (uint32_t)four[q]);
      groups += four[q] >= 0;
    }
  }
  {
    const uint32_t top = wave_scan((uint32_t)(mine + 1), 0u, larger);  // + 1: 0 for none
    const uint32_t low = wave_scan(least, 0xffffffffu, smaller);
    const int n = wave_inclusive(groups);
    if (lane == kWave - 1) {
      sh.red_max[wave] = top;
      sh.red_min[wave] = low;
      sh.red_cnt[wave] = n;
    }
  }
  clear_hist(sh, tid);
  if (tid == 0) sh.n_few = 0;
  __syncthreads();
  uint32_t lo;
  int mx, n_groups;
  auto block_stats = [&] {
    const uint32_t top = wave_scan(lane < NW ? sh.red_max[lane] : 0u, 0u, larger);
    const uint32_t low = wave_scan(lane < NW ? sh.red_min[lane] : 0xffffffffu, 0xffffffffu, smaller);
    const int n = wave_inclusive(lane < NW ? sh.red_cnt[lane] : 0);
    mx = (int)lane_value(top, kWave - 1) - 1;
    lo = lane_value(low, kWave - 1);
    n_groups = (int)lane_value((uint32_t)n, kWave - 1);
  };
  block_stats();
  const bool by_groups = n_groups > kp;  // then there are more than kp candidates as well
  bool all = false;                      // keep every candidate
  if (!by_groups) {                      // uniform: count the candidates
    uint32_t cand_min = 0xffffffffu;
    int n = 0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      cand_min = min(cand_min, (uint32_t)key[i]);
      n += key[i] >= 0;
    }
    cand_min = wave_scan(cand_min, 0xffffffffu, smaller);
    n = wave_inclusive(n);
    __syncthreads();
    if (lane == kWave - 1) {
      sh.red_min[wave] = cand_min;
      sh.red_cnt[wave] = n;
    }
    __syncthreads();
    block_stats();
    all = n_groups <= kp;
  }
  const auto shift_for = [](uint32_t range) { return max(0, 21 - __clz((int)range | 1)); };  // range >> shift < kBins
  int k = kp, thr = -1;
  if constexpr (NK <= kDirectKeys) {
    if (all) k = 0;
    else thr = find_threshold<NK, NT>(key, (int)lo, shift_for((uint32_t)mx - lo), k, sh, tid, lane, wave);
    return emit_keys<NK, NT>(sh, key, thr, k, kp, 0, 0, write, tid, lane, wave);
  }
  // a quota that leaves the list no room for the undecided keys: straight to the registers
  int m = Shared::CAP + 1, bound = (int)lo, shift = shift_for((uint32_t)mx - lo);
  if (!all && kp <= kListQuota) {
    if (!by_groups) {
#pragma unroll
      for (int i = 0; i < NK; ++i)
        if (key[i] >= 0) atomicAdd(&sh.hist[((uint32_t)key[i] - lo) >> shift], 1);
    } else if (by_thread) {
      if (mine >= 0) atomicAdd(&sh.hist[((uint32_t)mine - lo) >> shift], 1);
    } else {
#pragma unroll
      for (int q = 0; q < NG; ++q)
        if (four[q] >= 0) atomicAdd(&sh.hist[((uint32_t)four[q] - lo) >> shift], 1);
    }
    __syncthreads();
    find_bin_block(sh, kp, tid, lane, wave);
    bound = (int)(lo + ((uint32_t)sh.bin << shift));  // at least kp keys are at or above it
    clear_hist(sh, tid);  // find_bin_block ended behind a barrier: hist has been read

    // -- 2: slots of the keys at or above the bound
    m = emit_sparse<NK, NT>(
        sh, key, bound,
        [&](int rank, int slot) {
          if (rank < Shared::CAP) sh.list[rank] = slot;
        },
        lane, wave);
    __syncthreads();
    shift = shift_for((uint32_t)(mx - bound));
  }
  if (all || m > Shared::CAP) {  // uniform
    if (all) k = 0;
    else thr = find_threshold<NK, NT>(key, bound, shift, k, sh, tid, lane, wave);
    return emit_keys<NK, NT>(sh, key, thr, k, kp, 0, 0, write, tid, lane, wave);
  }

  // -- 3: the list's keys, read again; the threshold among them. The first read found all of them between the bound and the
  // maximum. They are held there: the bins, the ranks and the number kept depend on it, and a caller may be writing its
  // input meanwhile (the result is then anybody's guess, but it stays inside its buffers).
  constexpr int NQ = Shared::NQ;
  int slot[NQ], lk[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    slot[q] = -1;
    lk[q] = -1;
    if (q * NT + tid < m) {
      slot[q] = sh.list[q * NT + tid];
      lk[q] = min(max(reload(slot[q]), bound), mx);
    }
  }
  thr = find_threshold<NQ, NT>(lk, bound, shift, k, sh, tid, lane, wave);

  // -- 4: kept entries of the list: those above thr and the first k equal to it
  uint32_t gt_before[NQ], eq_before[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const unsigned long long mg = __ballot(lk[q] > thr), mq = __ballot(lk[q] == thr);
    gt_before[q] = lanes_below(mg, 0u);
    eq_before[q] = lanes_below(mq, 0u);
    if (lane == 0) sh.cnt[q * NW + wave] = __popcll(mg) | __popcll(mq) << 16;
  }
  __syncthreads();
  static_assert(NQ * NW <= kWave, "an entry per lane");
  const int packed = lane < NQ * NW ? sh.cnt[lane] : 0;
  const int gi = wave_inclusive(packed & 0xffff), qi = wave_inclusive((int)((uint32_t)packed >> 16));
  const int gx = gi - (packed & 0xffff), qx = qi - (int)((uint32_t)packed >> 16);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int g = (int)gt_before[q] + (int)lane_value((uint32_t)gx, q * NW + wave);
    const int e = (int)eq_before[q] + (int)lane_value((uint32_t)qx, q * NW + wave);
    if (lk[q] > thr || (lk[q] == thr && e < k)) write(g + min(e, k), slot[q], lk[q]);
  }
  return kp;
}

template <int NK, int NT>
__device__ __forceinline__ void load_keys(const float *u, int P, int base, float tau, int (&key)[NK], int tid) {
  float x[NK];
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const int t = base + i * NT + tid;
    x[i] = t < P ? u[t] : __int_as_float(0x7fc00000);  // NaN: no candidate
  }
#pragma unroll
  for (int i = 0; i < NK; ++i) key[i] = key_of(x[i], tau);
}

// One workgroup per unit; all positions in registers.
template <int NK, int NT>
__global__ void __launch_bounds__(NT) select_reg_kernel(SelectArgs a) {
  __shared__ SelectShared<NK, NT> sh;
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *u = a.utility + (size_t)unit * a.P;
  const float tau = a.tau[unit / a.Hkv];
  int key[NK];
  load_keys<NK, NT>(u, a.P, 0, tau, key, tid);  // in flight while the budget arrives
  const int kp = prefix_quota(a, unit);
  int32_t *out = a.idx + (size_t)unit * a.cap;
  int kept = 0;
  if (kp > 0)
    kept = select_keys<NK, NT>(
        key, kp, sh, [&](int slot) { return key_of(u[slot], tau); }, [&](int rank, int slot, int) { out[rank] = slot; }, tid, lane, wave);
  for (int j = tid; j < a.W; j += NT) out[kept + j] = a.P + j;
  if (tid == 0) a.count[unit] = kept + a.W;
}

// ---------------------------------------------------------------------------------------------
// Selection and gather of a layer in one launch, where the most that one head may keep is in flight at once. `parts` workgroups make the same
// selection of a unit, which takes none of them longer than one of them (a chain of steps inside a workgroup, while most of the
// chip is idle), and each writes and copies its share of the rows: blocks of BLOCK rows in turn, whose positions stay in LDS. The
// gather's launch, and its way to count, index and row, are gone; what is left of it is the rows. us per layer, two launches / one: 4096
// keys, 32/32 heads 25.6 / 24.2, 8192, 32/8 25.6 / 24.7, 1000, 32/8 20.6 / 19.1, 28000, 32/8 46.8 / 46.4, 30000, 32/8, 2048 rows 50.3 / 48.7. With
// shares a head may have all rows of a batch element: it is this form where its workgroups take those with two blocks each; where they
// have more to move, the gather, which deals long lists out, is the faster one. Shares drawn from 0.5 to 1.5 and all in one head, us: 8192 keys,
// 32/8 heads 25.9 / 24.8, 28.1 / 27.4; f32, 1024, 4/4 (four calls' kernels) 21.6 / 18.3, 20.5 / 19.1; but with up to four blocks each 20011, batch 2
// 55.1 / 54.0, 65.4 / 68.0 and 16384, batch 4, given normalisers 43.5 / 43.6, 48.8 / 51.5.
// ---------------------------------------------------------------------------------------------
constexpr int kPartBlocks = 4;  // of a part, at most: a thread has all its rows of K and V in flight
struct KeepArgs {
  SelectArgs a;
  const char *k, *v;
  char *k_out, *v_out;
  int64_t ks_b, ks_h, ks_t, vs_b, vs_h, vs_t;  // bytes
  int log_parts;
};
typedef __attribute__((ext_vector_type(4))) uint32_t row_piece_t;

// LPR: 16-byte pieces of a row, one per lane
template <int NK, int NT, int LPR>
__global__ void __launch_bounds__(NT) keep_kernel(KeepArgs ka) {
  constexpr int BLOCK = NT / LPR;
  __shared__ SelectShared<NK, NT> sh;
  __shared__ int s_rows[kPartBlocks * BLOCK];
  const SelectArgs &a = ka.a;
  const int parts = 1 << ka.log_parts, part = blockIdx.x & (parts - 1), unit = blockIdx.x >> ka.log_parts;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *u = a.utility + (size_t)unit * a.P;
  const float tau = a.tau[b];
  int key[NK];
  load_keys<NK, NT>(u, a.P, 0, tau, key, tid);
  const int kp = prefix_quota(a, unit);
  int kept = 0;
  if (kp > 0)
    kept = select_keys<NK, NT>(
        key, kp, sh, [&](int slot) { return key_of(u[slot], tau); },
        [&](int rank, int slot, int) {
          const int block = rank / BLOCK, of_part = block >> ka.log_parts;
          if ((block & (parts - 1)) == part && of_part < kPartBlocks) s_rows[of_part * BLOCK + rank % BLOCK] = slot;
        },
        tid, lane, wave);
  __syncthreads();
  const int count = kept + a.W, local = tid / LPR, piece = tid % LPR * 16;
  if (part == 0 && tid == 0) a.count[unit] = count;
  const char *k = ka.k + b * ka.ks_b + g * ka.ks_h + piece, *v = ka.v + b * ka.vs_b + g * ka.vs_h + piece;
  const size_t first = (size_t)unit * a.cap;
  row_piece_t kk[kPartBlocks], vv[kPartBlocks];
  int from[kPartBlocks];
#pragma unroll
  for (int e = 0; e < kPartBlocks; ++e) {
    const int r = (e * parts + part) * BLOCK + local;
    if (r < count) {
      // held inside the row, whatever another stream writes over the utilities meanwhile
      from[e] = r < kept ? min(max(s_rows[e * BLOCK + local], 0), a.P - 1) : a.P + r - kept;
      kk[e] = *reinterpret_cast<const row_piece_t *>(k + (int64_t)from[e] * ka.ks_t);
      vv[e] = *reinterpret_cast<const row_piece_t *>(v + (int64_t)from[e] * ka.vs_t);
    }
  }
#pragma unroll
  for (int e = 0; e < kPartBlocks; ++e) {
    const int r = (e * parts + part) * BLOCK + local;
    if (r < count) {
      const size_t o = (first + r) * (LPR * 16) + piece;
      *reinterpret_cast<row_piece_t *>(ka.k_out + o) = kk[e];
      *reinterpret_cast<row_piece_t *>(ka.v_out + o) = vv[e];
      if (piece == 0) a.idx[first + r] = from[e];
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Long rows in two launches. A slice of 8192 or 16384 positions per workgroup keeps its own kp best (what the unit keeps
// is among them) as (key, position) pairs in the workspace, in position order, padded with "no candidate" to
// a length that both kernels know from the budget; one workgroup per unit then selects among the slices' pairs.
// No counter has to be cleared beforehand and no workgroup waits for another. Worth it while the slices drop
// most keys: plan_slices() draws the line.
// ---------------------------------------------------------------------------------------------
struct SliceArgs {
  SelectArgs a;
  int2 *pairs;  // [units][S][region] (key, position)
  int S, region, slice;  // slices per unit, pairs per slice, positions per slice
};

// Pairs that a slice hands over, a multiple of 64 (so is the region).
__device__ __forceinline__ int slice_pairs(int kp, int slice) { return (min(kp, slice) + kWave - 1) / kWave * kWave; }

template <int NK>
__global__ void __launch_bounds__(kSelectThreads) select_slice_kernel(SliceArgs sa) {
  __shared__ SelectShared<NK, kSelectThreads> sh;
  const SelectArgs &a = sa.a;
  const int unit = blockIdx.x / sa.S, slice = blockIdx.x % sa.S;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *u = a.utility + (size_t)unit * a.P;
  const float tau = a.tau[unit / a.Hkv];
  const int base = slice * sa.slice;
  int key[NK];
  load_keys<NK, kSelectThreads>(u, min(a.P, base + sa.slice), base, tau, key, tid);
  const int kp = prefix_quota(a, unit);
  if (kp <= 0 || slice_pairs(kp, sa.slice) > sa.region) return;
  int2 *out = sa.pairs + (size_t)blockIdx.x * sa.region;
  const int kept = select_keys<NK, kSelectThreads>(
      key, kp, sh, [&](int slot) { return key_of(u[base + slot], tau); },
      [&](int rank, int slot, int k) { out[rank] = make_int2(k, base + slot); }, tid, lane, wave);
  for (int i = kept + tid; i < slice_pairs(kp, sa.slice); i += kSelectThreads) out[i] = make_int2(-1, 0);
}

// Defined with the streaming kernel below.
struct StreamShared {
  int hist[256];
  int wave_gt[kSelectThreads / kWave], wave_eq[kSelectThreads / kWave];
  uint32_t prefix;
  int k, state;  // state: 0 = keep all candidates, 1 = select, 2 = keep none
};
template <class Key, class Emit>
__device__ __forceinline__ int select_stream(int n, int kp, StreamShared &sh, Key key_at, Emit emit, int tid, int lane, int wave);

template <int NK>
__device__ __forceinline__ int merge_slices(const int2 *pairs, int S, int region, int per_slice, int kp,
                                            SelectShared<NK, kSelectThreads> &sh, int32_t *out, int tid, int lane, int wave) {
  // the unit's pairs, slices back to back without the regions' rests; 64 slots never straddle two slices
  int key[NK];
  int slice = 0, off = wave * kWave;
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    while (off >= per_slice) {  // uniform
      off -= per_slice;
      ++slice;
    }
    key[i] = slice < S ? pairs[(size_t)slice * region + off + lane].x : -1;
    off += kSelectThreads;
  }
  const auto at = [&](int slot) { return pairs[(size_t)(slot / per_slice) * region + slot % per_slice]; };
  return select_keys<NK, kSelectThreads>(
      key, kp, sh, [&](int slot) { return at(slot).x; }, [&](int rank, int slot, int) { out[rank] = at(slot).y; }, tid, lane, wave);
}

// Most pairs of a unit; one whose budget would give more of them (its slices write none) goes over its row by itself.
constexpr int kMergePairs = 64 * kSelectThreads;

__global__ void __launch_bounds__(kSelectThreads) select_merge_kernel(SliceArgs sa) {
  __shared__ union {
    SelectShared<8, kSelectThreads> few;
    SelectShared<32, kSelectThreads> more;
    SelectShared<64, kSelectThreads> most;
    StreamShared stream;
  } sh;
  const SelectArgs &a = sa.a;
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int2 *pairs = sa.pairs + (size_t)unit * sa.S * sa.region;
  const int kp = prefix_quota(a, unit);
  int32_t *out = a.idx + (size_t)unit * a.cap;
  int kept = 0;
  if (kp > 0) {
    const int per_slice = slice_pairs(kp, sa.slice), n = sa.S * per_slice;
    if (per_slice > sa.region) {
      const float *u = a.utility + (size_t)unit * a.P;
      const float tau = a.tau[unit / a.Hkv];
      kept = select_stream(
          a.P, kp, sh.stream, [&](int t) { return key_of(u[t], tau); }, [&](int rank, int t) { out[rank] = t; }, tid, lane, wave);
    } else if (n <= 8 * kSelectThreads) kept = merge_slices<8>(pairs, sa.S, sa.region, per_slice, kp, sh.few, out, tid, lane, wave);
    else if (n <= 32 * kSelectThreads) kept = merge_slices<32>(pairs, sa.S, sa.region, per_slice, kp, sh.more, out, tid, lane, wave);
    else kept = merge_slices<64>(pairs, sa.S, sa.region, per_slice, kp, sh.most, out, tid, lane, wave);  // a head with far more than its share
  }
  for (int j = tid; j < a.W; j += kSelectThreads) out[kept + j] = a.P + j;
  if (tid == 0) a.count[unit] = kept + a.W;
}

// Adds one count per active lane to hist[digit]. Utilities cluster in a few exponent bins, so plain
// per-lane LDS atomics would serialise on one address: the wave first elects up to three leaders
// whose digit is shared by many lanes and adds a popcount for each; stragglers use their own atomic.
// Every lane of the wave must call this (it uses ballots).
__device__ __forceinline__ void hist_add(int *hist, bool active, int digit, int lane) {
  unsigned long long rem = __ballot(active);
#pragma unroll
  for (int it = 0; it < 3; ++it) {
    if (rem == 0) break;
    const int leader = __ffsll((long long)rem) - 1;
    const int d = __shfl(digit, leader);
    const unsigned long long same = __ballot(active && digit == d);
    if (lane == leader) atomicAdd(&hist[d], __popcll(same));
    active = active && digit != d;
    rem &= ~same;
  }
  if (active) atomicAdd(&hist[digit], 1);
}

// Executed by wave 0. Scans hist[NB-1..0]; returns the bin where the running count first reaches k
// (1-based) and the count strictly above that bin, plus the grand total.
struct BinResult {
  int bin, above, total;
};
template <int NB>
__device__ __forceinline__ BinResult find_bin(const int *hist, int k, int lane) {
  constexpr int PER = NB / kWave;  // lane i owns bins NB-1-PER*i .. NB-PER*(i+1) (descending)
  int c[PER], sum = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    c[e] = hist[NB - 1 - PER * lane - e];
    sum += c[e];
  }
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o);
    if (lane >= o) incl += up;
  }
  BinResult r;
  r.total = __shfl(incl, 63);
  const int excl = incl - sum;
  const bool mine = excl < k && k <= incl;
  int bin = -1, above = 0;
  if (mine) {
    int run = excl;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      if (bin < 0 && run + c[e] >= k) {
        bin = NB - 1 - PER * lane - e;
        above = run;
      }
      run += c[e];
    }
  }
  const unsigned long long who = __ballot(mine);
  const int src = who ? __ffsll((long long)who) - 1 : 0;
  r.bin = __shfl(bin, src);
  r.above = __shfl(above, src);
  if (!who) r.bin = -1;
  return r;
}

// Counts digit SHIFT .. SHIFT + BITS - 1 of the candidates whose higher bits are prefix_hi.
template <int NK, int SHIFT, int BITS>
__device__ __forceinline__ void digit_histogram(int *hist, const int (&key)[NK], uint32_t prefix_hi) {
#pragma unroll
  for (int i = 0; i < NK; ++i) {
    const uint32_t k = (uint32_t)key[i];
    if (key[i] >= 0 && (k >> (SHIFT + BITS)) == prefix_hi) atomicAdd(&hist[(k >> SHIFT) & ((1u << BITS) - 1u)], 1);
  }
}

// ---------------------------------------------------------------------------------------------
// Split select: long rows whose budgets are so large that slices could drop few keys. Slices of 8192
// positions, one workgroup each; five launches walk three digits of the key (11, 10 and 10 bits: slices merge their histograms
// into the unit's in global memory with integer atomics), the slices' counts of keys above / equal to the
// threshold, and the ranked write. Every workgroup derives the threshold digits from
// the merged histograms itself (4096 integers per unit), which saves the launches in between.
// ---------------------------------------------------------------------------------------------
constexpr int kSplitHist = 2048 + 1024 + 1024;              // merged histogram words per unit

constexpr int kSplitKeys = 8;
constexpr int kSplitSlice = kSplitKeys * kSelectThreads;  // positions per workgroup

struct SplitArgs {
  SelectArgs a;
  int *hist;       // [units][kSplitHist], zero before the first phase
  int *slice_cnt;  // [units][S] keys above | equal << 16 of each slice
  int *thr;        // [units][4 phases][4] digits found so far, keys still needed, state
  int S;           // slices per unit
};

__global__ void __launch_bounds__(kSelectThreads) select_split_zero_kernel(int *words, int n) {
  const int i = blockIdx.x * kSelectThreads + threadIdx.x;
  if (i < n) words[i] = 0;
}

// PHASE 0..2: histogram of digit PHASE (11, 10, 10 bits from the top) among the keys that match the
// digits found so far. PHASE 3: per-slice counts and the unit's threshold. PHASE 4: ranked write.
template <int PHASE>
__global__ void __launch_bounds__(kSelectThreads) select_split_kernel(SplitArgs sa) {
  __shared__ SelectShared<kSplitKeys, kSelectThreads> sh;
  int *const hist = sh.hist;
  __shared__ uint32_t s_prefix;
  __shared__ int s_k, s_state;  // s_state: 0 = keep all candidates, 1 = select, 2 = keep none
  __shared__ int s_red[kSelectThreads / kWave];

  const SelectArgs &a = sa.a;
  const int unit = blockIdx.x / sa.S, slice = blockIdx.x % sa.S;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int P = a.P, W = a.W;
  const float *u = a.utility + (size_t)unit * P;
  const float tau = a.tau[unit / a.Hkv];
  const int kp = prefix_quota(a, unit);
  const int base = slice * kSplitSlice;
  int *gh = sa.hist + (size_t)unit * kSplitHist;

  int key[kSplitKeys];
  load_keys<kSplitKeys, kSelectThreads>(u, P, base, tau, key, tid);

  // Threshold digits: phase p finds digit p - 1 from the histogram that phase p - 1 merged (the same
  // arithmetic in every workgroup of the unit) and takes the digits before it from the record that
  // the previous phase's first slice left; records are per phase, so no workgroup reads one that is
  // being written in its own launch.
  int state = 1, k = max(kp, 1);
  uint32_t prefix = 0u;
  int *rec = sa.thr + (size_t)unit * 16;  // [phase][prefix, k, state, -]
  if constexpr (PHASE >= 2) {
    prefix = (uint32_t)rec[4 * (PHASE - 1) + 0];
    k = rec[4 * (PHASE - 1) + 1];
    state = rec[4 * (PHASE - 1) + 2];
  }
  if constexpr (PHASE == 1) {
    for (int i = tid; i < 2048; i += kSelectThreads) hist[i] = gh[i];
    __syncthreads();
    if (wave == 0) {
      const BinResult r = find_bin<2048>(hist, max(kp, 1), lane);
      if (lane == 0) {
        s_prefix = (uint32_t)max(r.bin, 0);
        s_k = kp - r.above;
        s_state = r.total <= kp ? 0 : (kp == 0 ? 2 : 1);
      }
    }
    __syncthreads();
    state = s_state;
    prefix = s_prefix;
    k = s_k;
  }
  if constexpr (PHASE == 2 || PHASE == 3) {
    if (state == 1) {
      hist[tid] = gh[2048 + 1024 * (PHASE - 2) + tid];
      __syncthreads();
      if (wave == 0) {
        const BinResult r = find_bin<1024>(hist, k, lane);
        if (lane == 0) {
          s_prefix = (prefix << 10) | (uint32_t)r.bin;
          s_k = k - r.above;
        }
      }
      __syncthreads();
      prefix = s_prefix;
      k = s_k;
    }
  }
  if constexpr (PHASE >= 1 && PHASE <= 3) {
    if (slice == 0 && tid == 0) {
      rec[4 * PHASE + 0] = (int)prefix;
      rec[4 * PHASE + 1] = k;
      rec[4 * PHASE + 2] = state;
    }
  }

  if constexpr (PHASE <= 2) {
    if (PHASE > 0 && state != 1) return;
    constexpr int NB = PHASE == 0 ? 2048 : 1024;
    __syncthreads();
    for (int i = tid; i < NB; i += kSelectThreads) hist[i] = 0;
    __syncthreads();
    digit_histogram<kSplitKeys, 20 - 10 * PHASE, PHASE == 0 ? 11 : 10>(hist, key, prefix);
    __syncthreads();
    int *g = gh + (PHASE == 0 ? 0 : 2048 + 1024 * (PHASE - 1));
    for (int i = tid; i < NB; i += kSelectThreads) {
      const int h = hist[i];
      if (h) atomicAdd(&g[i], h);
    }
    return;
  }

  // threshold: the digits found; keep-all (state 0): every candidate is above -1; keep-none (state 2)
  const int thr = state == 0 ? -1 : state == 2 ? 0x7fffffff : (int)prefix;
  const int need_eq = state == 1 ? k : 0;
  if constexpr (PHASE == 3) {
    int c = 0;
#pragma unroll
    for (int i = 0; i < kSplitKeys; ++i) c += (key[i] > thr ? 1 : 0) + (need_eq && key[i] == thr ? 0x10000 : 0);
    c = wave_inclusive(c);  // 512 positions a wave, 8192 a slice: neither half overflows
    if (lane == kWave - 1) s_red[wave] = c;
    __syncthreads();
    if (tid == 0) {
      int tot = 0;
      for (int w = 0; w < kSelectThreads / kWave; ++w) tot += s_red[w];
      sa.slice_cnt[(size_t)unit * sa.S + slice] = tot;
    }
    return;
  }

  if constexpr (PHASE == 4) {
    int base_gt = 0, base_eq = 0, all_gt = 0, all_eq = 0;
    for (int i = 0; i < sa.S; ++i) {  // same address in every lane: one broadcast load each
      const int c = sa.slice_cnt[(size_t)unit * sa.S + i];
      if (i < slice) {
        base_gt += c & 0xffff;
        base_eq += c >> 16;
      }
      all_gt += c & 0xffff;
      all_eq += c >> 16;
    }
    int32_t *out = a.idx + (size_t)unit * a.cap;
    emit_keys<kSplitKeys, kSelectThreads>(
        sh, key, thr, need_eq, kp, base_gt, base_eq, [&](int rank, int slot, int) { out[rank] = base + slot; }, tid, lane, wave);
    if (slice == 0) {
      const int kept = min(all_gt + min(all_eq, need_eq), kp);
      for (int j = tid; j < W; j += kSelectThreads) out[kept + j] = P + j;
      if (tid == 0) a.count[unit] = kept + W;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Streaming select: any length, nothing kept on chip but counters. Keys come from key_at(i) (-1: no candidate),
// several at a time, once per 8-bit digit and twice for the ranks; emit(rank, i) for the kept ones.
// ---------------------------------------------------------------------------------------------
constexpr int kUnroll = 8;

template <class Key, class Emit>
__device__ __forceinline__ int select_stream(int n, int kp, StreamShared &sh, Key key_at, Emit emit, int tid, int lane, int wave) {
  // digits from the top; the first histogram also counts the candidates
  int thr = -1;  // keep-all: every candidate's key is above -1
  int need_eq = 0;
  int k = max(kp, 1);
  uint32_t prefix = 0u;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) sh.hist[tid] = 0;
    __syncthreads();
    const uint32_t hi_mask = shift == 24 ? 0u : 0xffffffffu << (shift + 8);
    // eight loads in flight per thread: the pass is bound by L2 latency, not by arithmetic
    for (int t0 = 0; t0 < n; t0 += kUnroll * kSelectThreads) {
      int x[kUnroll];
#pragma unroll
      for (int e = 0; e < kUnroll; ++e) {
        const int t = t0 + e * kSelectThreads + tid;
        x[e] = t < n ? key_at(t) : -1;
      }
#pragma unroll
      for (int e = 0; e < kUnroll; ++e)
        hist_add(sh.hist, x[e] >= 0 && ((uint32_t)x[e] & hi_mask) == prefix, (x[e] >> shift) & 255, lane);
    }
    __syncthreads();
    if (wave == 0) {
      const BinResult r = find_bin<256>(sh.hist, k, lane);
      if (lane == 0) {
        if (shift == 24) sh.state = r.total <= kp ? 0 : kp == 0 ? 2 : 1;
        sh.prefix = prefix | ((uint32_t)max(r.bin, 0) << shift);
        sh.k = k - r.above;
      }
    }
    __syncthreads();
    if (sh.state != 1) break;
    prefix = sh.prefix;
    k = sh.k;
    thr = (int)prefix;
    need_eq = k;  // how many keys equal to thr are kept (>= 1)
  }
  if (sh.state == 2) thr = 0x7fffffff;

  // ranks: wave w owns keys [w * seg, (w + 1) * seg); seg is a multiple of 64
  const int n_waves = kSelectThreads / kWave;
  const int seg = ((n + n_waves - 1) / n_waves + kWave - 1) / kWave * kWave;
  const int lo = wave * seg, hi = min(lo + seg, n);
  int n_gt = 0, n_eq = 0;
  for (int t0 = lo; t0 < hi; t0 += kUnroll * kWave) {
    int x[kUnroll];
#pragma unroll
    for (int e = 0; e < kUnroll; ++e) {
      const int t = t0 + e * kWave + lane;
      x[e] = t < hi ? key_at(t) : -1;
    }
#pragma unroll
    for (int e = 0; e < kUnroll; ++e) {
      n_gt += __popcll(__ballot(x[e] > thr));
      n_eq += __popcll(__ballot(need_eq && x[e] == thr));
    }
  }
  if (lane == 0) {
    sh.wave_gt[wave] = n_gt;
    sh.wave_eq[wave] = n_eq;
  }
  __syncthreads();
  int base_gt = 0, base_eq = 0, tot_gt = 0, tot_eq = 0;
  for (int w = 0; w < n_waves; ++w) {
    base_gt += w < wave ? sh.wave_gt[w] : 0;
    base_eq += w < wave ? sh.wave_eq[w] : 0;
    tot_gt += sh.wave_gt[w];
    tot_eq += sh.wave_eq[w];
  }
  for (int t0 = lo; t0 < hi; t0 += kUnroll * kWave) {
    int x[kUnroll];
#pragma unroll
    for (int e = 0; e < kUnroll; ++e) {
      const int t = t0 + e * kWave + lane;
      x[e] = t < hi ? key_at(t) : -1;
    }
#pragma unroll
    for (int e = 0; e < kUnroll; ++e) {
      const bool gt = x[e] > thr, eq = need_eq && x[e] == thr;
      const unsigned long long bg = __ballot(gt), be = __ballot(eq);
      const int gt_before = (int)lanes_below(bg, (uint32_t)base_gt), eq_before = (int)lanes_below(be, (uint32_t)base_eq);
      if (gt || (eq && eq_before < need_eq)) {
        const int pos = gt_before + min(eq_before, need_eq);
        if (pos < kp) emit(pos, t0 + e * kWave + lane);
      }
      base_gt += __popcll(bg);
      base_eq += __popcll(be);
    }
  }
  return min(tot_gt + min(tot_eq, need_eq), kp);
}

__global__ void __launch_bounds__(kSelectThreads) select_kernel(SelectArgs a) {
  __shared__ StreamShared sh;
  const int unit = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *u = a.utility + (size_t)unit * a.P;
  const float tau = a.tau[unit / a.Hkv];
  const int kp = prefix_quota(a, unit);
  int32_t *out = a.idx + (size_t)unit * a.cap;
  const int kept = select_stream(
      a.P, kp, sh,
      [&](int t) { return key_of(u[t], tau); },
      [&](int rank, int t) { out[rank] = t; }, tid, lane, wave);
  for (int j = tid; j < a.W; j += kSelectThreads) out[kept + j] = a.P + j;
  if (tid == 0) a.count[unit] = kept + a.W;
}

// ---------------------------------------------------------------------------------------------
// Which kernel
// ---------------------------------------------------------------------------------------------
// Up to 32768 positions one workgroup per unit in one launch is the faster form, and no workspace is touched
// (callers need not pass one).
constexpr int kOneLaunch = 32 * kSelectThreads;
static int slices(const Shape &s, int size) { return (s.P + size - 1) / size; }

// Slices, where they pay: S of them (0: they do not), `slice` positions each, at most `limit`, `region` pairs.
struct SlicePlan {
  int S, limit, slice, region;
};
// The budgets are on the device, so the rule goes by what heads are likely to have: twice the nominal quota, and with room for
// eight times. Slices + merge / split selection, us, 34000 to 262144 positions, 8 heads, batch 1 and 4, two distributions, where the
// largest quota of a unit's heads is up to 2048: 15-25 / 24-35 and 15-34 / 25-89; where it is 3072: 27-45 / 24-35 and 28-46 /
// 25-49. So twice the nominal quota, or all that cap leaves a head, has to be at most 2048. With half of a nominal 8 x 1024 in
// one head 35-45 / 24-49, with all of it 40-75 / 24-49. One KV head alone, 65504 to 262112 positions, 1100 to 2016: 18-24 / 28-31.
// A unit has at most 65536 pairs, which the merge takes in registers (streaming more of them, as it did, took one workgroup
// 90-600 us). There is room in them for eight times the nominal quota (and one), or the split is taken; a head with more than the room is
// selected from its row by one workgroup (32 heads, all of the budget in one, 128k: 219-247 / 43-49; before 223-295).
// 8192 positions per slice where the merge then has at most 8192 pairs, which it takes eight to a thread; else 16384, which
// halves the pairs (98304 positions, 32 units, 512: 20 -> 17 us; one head at twice that 23 -> 18).
static SlicePlan plan_slices(const ckv_params *p, const Shape &s) {
  SlicePlan plan = {0, 0, 0, 0};
  const int64_t quota = p->budget_per_kv_head - s.W;
  const int most = max(1, min(p->cap, s.T) - s.W);
  const auto up = [](int64_t x) { return (x + kWave - 1) / kWave * kWave; };
  const auto least = [](int64_t x, int64_t y) { return x < y ? x : y; };
  if (s.P <= kOneLaunch || least(most, 2 * quota) > 2048) return plan;
  for (int limit = 8 * kSelectThreads; limit <= 16 * kSelectThreads; limit *= 2) {
    const int64_t n = slices(s, limit), room = kMergePairs / n / kWave * kWave, top = least(limit, most);
    if (up(least(top, 8 * quota + 1)) > room || (limit == 8 * kSelectThreads && n * least(top, 2 * quota) > 8 * kSelectThreads)) continue;
    plan.S = (int)n;
    plan.limit = limit;
    plan.slice = (int)up((s.P + n - 1) / n);  // equal lengths: a short last one would keep all it has
    plan.region = (int)least(up(top), room);
    break;
  }
  return plan;
}

size_t select_split_bytes(const Shape &s) {
  if (s.P <= kOneLaunch) return 0;
  return (size_t)s.Bz * s.Hkv * (kSplitHist + slices(s, kSplitSlice) + 16) * sizeof(int);
}

static size_t slice_pair_bytes(const Shape &s, const SlicePlan &plan) {
  return (size_t)s.Bz * s.Hkv * plan.S * plan.region * sizeof(int2);
}

size_t select_workspace_bytes(const ckv_params *p, const Shape &s) {
  return max(select_split_bytes(s), slice_pair_bytes(s, plan_slices(p, s)));
}

template <int NK, int NT>
static void launch_reg(const SelectArgs &a, int units, hipStream_t stream) {
  hipLaunchKernelGGL((select_reg_kernel<NK, NT>), dim3(units), dim3(NT), 0, stream, a);
}

static SelectArgs select_args(const ckv_params *p, const Shape &s, const float *utility, const int32_t *budget, const float *tau,
                              int32_t *idx, int32_t *count) {
  SelectArgs a;
  a.utility = utility;
  a.budget = budget;
  a.tau = tau;
  a.idx = idx;
  a.count = count;
  a.Hkv = s.Hkv; a.T = s.T; a.W = s.W; a.P = s.P;
  a.cap = p->cap;
  return a;
}

// Workgroups per unit for selection and gather in one launch, a power of two: one for each CU, and no more than have a block of
// rows. Less than two, or more rows than those have in flight: not this form, which then gains nothing (us per layer, two launches / one:
// 128 units, 512 rows, two parts 81.0 / 81.1, 64 units, 2048 rows 120.1 / 120.0).
static int keep_parts(const ckv_params *p, const Shape &s, bool shares) {
  if (s.P > kOneLaunch || s.P < 1) return 0;
  const int units = s.Bz * s.Hkv, lpr = s.d * s.esize / 16;
  const int rows = min(shares ? p->cap : min(p->budget_per_kv_head, p->cap), s.T);  // the most that a head can keep
  const int block = (s.P <= 4 * 256 ? 256 : s.P <= 8 * 512 ? 512 : kSelectThreads) / lpr;
  int parts = 1;
  while (2 * parts * units <= kComputeUnits && parts * block < rows) parts *= 2;
  return parts >= 2 && rows <= parts * (shares ? kPartBlocks / 2 : kPartBlocks) * block ? parts : 0;
}
bool keeps_in_one_launch(const ckv_params *p, const Shape &s, bool shares) { return keep_parts(p, s, shares) > 0; }

template <int NK, int NT>
static void launch_keep_rows(const KeepArgs &ka, int lpr, dim3 grid, hipStream_t stream) {
  if (lpr == 8) hipLaunchKernelGGL((keep_kernel<NK, NT, 8>), grid, dim3(NT), 0, stream, ka);
  else if (lpr == 16) hipLaunchKernelGGL((keep_kernel<NK, NT, 16>), grid, dim3(NT), 0, stream, ka);
  else hipLaunchKernelGGL((keep_kernel<NK, NT, 32>), grid, dim3(NT), 0, stream, ka);
}

hipError_t launch_keep(const ckv_params *p, const Shape &s, const float *utility, const int32_t *budget, const float *tau, const void *k,
                       const void *v, int32_t *idx, int32_t *count, void *k_out, void *v_out, bool shares, hipStream_t stream) {
  KeepArgs ka;
  ka.a = select_args(p, s, utility, budget, tau, idx, count);
  ka.k = (const char *)k;
  ka.v = (const char *)v;
  ka.k_out = (char *)k_out;
  ka.v_out = (char *)v_out;
  ka.ks_b = p->k_stride[0] * s.esize; ka.ks_h = p->k_stride[1] * s.esize; ka.ks_t = p->k_stride[2] * s.esize;
  ka.vs_b = p->v_stride[0] * s.esize; ka.vs_h = p->v_stride[1] * s.esize; ka.vs_t = p->v_stride[2] * s.esize;
  const int parts = keep_parts(p, s, shares), lpr = s.d * s.esize / 16;
  ka.log_parts = __builtin_ctz(parts);
  const dim3 grid((unsigned)(s.Bz * s.Hkv * parts));
  if (s.P <= 4 * 256) launch_keep_rows<4, 256>(ka, lpr, grid, stream);
  else if (s.P <= 8 * 512) launch_keep_rows<8, 512>(ka, lpr, grid, stream);
  else if (s.P <= 8 * kSelectThreads) launch_keep_rows<8, kSelectThreads>(ka, lpr, grid, stream);
  else if (s.P <= 16 * kSelectThreads) launch_keep_rows<16, kSelectThreads>(ka, lpr, grid, stream);
  else launch_keep_rows<32, kSelectThreads>(ka, lpr, grid, stream);
  return hipGetLastError();
}

hipError_t launch_select(const ckv_params *p, const Shape &s, const float *utility,
                         const int32_t *budget, const float *tau, int32_t *idx, int32_t *count,
                         char *ws, size_t ws_bytes, hipStream_t stream) {
  const SelectArgs a = select_args(p, s, utility, budget, tau, idx, count);
  const int units = s.Bz * s.Hkv;
  const dim3 block(kSelectThreads);
  const SlicePlan plan = plan_slices(p, s);
  if (ws && plan.S > 0 && ws_bytes >= slice_pair_bytes(s, plan)) {
    SliceArgs sa;
    sa.a = a;
    sa.S = plan.S;
    sa.slice = plan.slice;
    sa.region = plan.region;
    sa.pairs = reinterpret_cast<int2 *>(ws);
    const dim3 slice_grid((unsigned)(units * sa.S));
    if (plan.limit == 8 * kSelectThreads) hipLaunchKernelGGL(select_slice_kernel<8>, slice_grid, block, 0, stream, sa);
    else hipLaunchKernelGGL(select_slice_kernel<16>, slice_grid, block, 0, stream, sa);
    hipLaunchKernelGGL(select_merge_kernel, dim3(units), block, 0, stream, sa);
  } else if (ws && s.P > kOneLaunch) {
    SplitArgs sa;
    sa.a = a;
    sa.S = slices(s, kSplitSlice);
    sa.hist = reinterpret_cast<int *>(ws);
    sa.slice_cnt = sa.hist + (size_t)units * kSplitHist;
    sa.thr = sa.slice_cnt + (size_t)units * sa.S;
    const int n_zero = units * kSplitHist;
    const dim3 split_grid((unsigned)(units * sa.S));
    hipLaunchKernelGGL(select_split_zero_kernel, dim3((n_zero + kSelectThreads - 1) / kSelectThreads), block, 0,
                       stream, sa.hist, n_zero);
    hipLaunchKernelGGL(select_split_kernel<0>, split_grid, block, 0, stream, sa);
    hipLaunchKernelGGL(select_split_kernel<1>, split_grid, block, 0, stream, sa);
    hipLaunchKernelGGL(select_split_kernel<2>, split_grid, block, 0, stream, sa);
    hipLaunchKernelGGL(select_split_kernel<3>, split_grid, block, 0, stream, sa);
    hipLaunchKernelGGL(select_split_kernel<4>, split_grid, block, 0, stream, sa);
  } else if (s.P <= 4 * 256) launch_reg<4, 256>(a, units, stream);
  else if (s.P <= 8 * 512) launch_reg<8, 512>(a, units, stream);
  else if (s.P <= 8 * kSelectThreads) launch_reg<8, kSelectThreads>(a, units, stream);
  else if (s.P <= 16 * kSelectThreads) launch_reg<16, kSelectThreads>(a, units, stream);
  else if (s.P <= 32 * kSelectThreads) launch_reg<32, kSelectThreads>(a, units, stream);
  else if (s.P <= 64 * kSelectThreads) launch_reg<64, kSelectThreads>(a, units, stream);
  else hipLaunchKernelGGL(select_kernel, dim3(units), block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace ckv
