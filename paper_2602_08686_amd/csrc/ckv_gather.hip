// Token-axis gather (paper Sec. 3: K~ = K[S], V~ = V[S]; Alg. 1 Gather_tok): bit copies of rows.
// A row of head_dim elements is moved as 16-byte pieces, one per lane, so a wave copies 64/LPR whole
// rows per instruction with 128-bit loads and stores; K and V rows travel in the same thread.
#include "ckv_internal.h"

namespace ckv {

typedef __attribute__((ext_vector_type(4))) uint32_t piece_t;

struct GatherArgs {
  const char *k, *v;
  char *k_out, *v_out;
  const int32_t *idx, *count;
  int64_t ks_b, ks_h, ks_t, vs_b, vs_h, vs_t;  // bytes
  int Hkv, T, cap;
  int shared;     // idx [Bz][cap] and count [Bz]: one index list for all KV heads of a batch element
};

constexpr int kGatherThreads = 256;

// LPR: lanes (16-byte pieces) per row. A workgroup copies one block of rows (kGatherThreads / LPR of them) of its own list. Blocks of
// lists that are longer than their workgroups take are dealt to the workgroups of the batch element, those without a block of their
// own first: a list that its own workgroups go over alone is bound by what few CUs can move (us, 32 heads, all that the budget
// allows in one of them: 15392 rows of 64 11.8, dealt out 3.3, 7200 rows of 128 11.2 and 3.3; shares drawn unevenly 4.6 and 3.3;
// two or four rows per thread in flight 13.3 and 15.4). What bounds a short list is the chain count -> index -> row: the
// first index is read beside the counts, the next block's beside a row (below cap it is the caller's memory, and it is used only below
// the count).
template <int LPR>
__global__ void __launch_bounds__(kGatherThreads) gather_kernel(GatherArgs a) {
  constexpr int STEP = kGatherThreads / LPR;  // rows of a block
  const int unit = blockIdx.y, x = blockIdx.x, per = gridDim.x;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int lane = threadIdx.x & 63, local = threadIdx.x / LPR, piece = (threadIdx.x % LPR) * 16;
  // the heads that share their workgroups: up to 64 neighbours, lane l has the count of head first + l
  const int first = g & ~(kWave - 1), heads = min(kWave, a.Hkv - first);
  const int mine = first + min(lane, heads - 1);
  const int counted = a.count[a.shared ? b : b * a.Hkv + mine];
  int head = g, r = x * STEP + local;
  int t = a.idx[(size_t)(a.shared ? b : unit) * a.cap + min(r, a.cap - 1)];
  const uint32_t rows = lane < heads ? (uint32_t)max(0, min(counted, a.cap)) : 0u;
  int n = (int)lane_value(rows, g - first);
  // blocks of each list beyond its own workgroups, and workgroups without a block of their own
  const uint32_t blocks = (rows + STEP - 1) / STEP, own = min(blocks, (uint32_t)per);
  const auto sum = [](uint32_t p, uint32_t q) { return p + q; };
  uint32_t job = ~0u, extra = 0, extra_end = 0;
  for (;;) {
    const char *k = a.k + b * a.ks_b + head * a.ks_h + piece, *v = a.v + b * a.vs_b + head * a.vs_h + piece;
    const bool take = r < n && t >= 0 && t < a.T;
    const size_t o = ((size_t)(b * a.Hkv + head) * a.cap + r) * (LPR * 16) + piece;
    piece_t kk, vv;
    if (take) {
      kk = *reinterpret_cast<const piece_t *>(k + (int64_t)t * a.ks_t);
      vv = *reinterpret_cast<const piece_t *>(v + (int64_t)t * a.vs_t);
    }
    if (job == ~0u) {  // the first time
      extra_end = wave_scan(blocks - own, 0u, sum);
      extra = lane_value(extra_end, kWave - 1);
      if (extra) {
        const uint32_t idle = lane < heads ? per - own : 0u, idle_end = wave_scan(idle, 0u, sum);
        const uint32_t all_idle = lane_value(idle_end, kWave - 1), mine_end = lane_value(idle_end, g - first);
        const uint32_t my_own = lane_value(own, g - first), before = mine_end - (per - my_own);  // idle ones of the heads in front
        job = (uint32_t)x >= my_own ? before + (x - my_own) : all_idle + (g - first) * per - before + x;
      }
    } else {
      job += heads * per;
    }
    const bool more = job < extra;  // uniform
    int next_head = head, next_r = r, next_t = t, next_n = n;
    if (more) {
      const int at = __popcll(__ballot(lane < heads && extra_end <= job));  // the list whose blocks these are
      const uint32_t behind = lane_value(extra_end, at) - lane_value(blocks - own, at);
      next_head = first + at;
      next_r = (int)(per + job - behind) * STEP + local;
      next_n = (int)lane_value(rows, at);
      next_t = a.idx[(size_t)(a.shared ? b : b * a.Hkv + next_head) * a.cap + min(next_r, a.cap - 1)];
    }
    if (take) {
      *reinterpret_cast<piece_t *>(a.k_out + o) = kk;
      *reinterpret_cast<piece_t *>(a.v_out + o) = vv;
    }
    if (!more) break;
    head = next_head;
    r = next_r;
    t = next_t;
    n = next_n;
  }
}

hipError_t launch_gather(const ckv_params *p, const Shape &s, const void *k, const void *v,
                         const int32_t *idx, const int32_t *count, void *k_out, void *v_out,
                         hipStream_t stream, bool shared_list) {
  GatherArgs a;
  a.k = (const char *)k;
  a.v = (const char *)v;
  a.k_out = (char *)k_out;
  a.v_out = (char *)v_out;
  a.idx = idx;
  a.count = count;
  a.ks_b = p->k_stride[0] * s.esize; a.ks_h = p->k_stride[1] * s.esize; a.ks_t = p->k_stride[2] * s.esize;
  a.vs_b = p->v_stride[0] * s.esize; a.vs_h = p->v_stride[1] * s.esize; a.vs_t = p->v_stride[2] * s.esize;
  a.Hkv = s.Hkv;
  a.T = s.T;
  a.cap = p->cap;
  a.shared = shared_list ? 1 : 0;
  // As many workgroups as the nominal budget has rows for (at least 512 where the cap has rows for them, at most 4096): together
  // they have room for what a batch element's heads keep, however it is shared out. The cap is several times the nominal budget;
  // sized by it, most of 4096 workgroups had nothing to do, and handing them out took longer than the copy. us, before and
  // now: 32 heads, 512 of 4096 rows 5.2 -> 3.8; 32 heads, 256 of 10006 4.8 -> 3.0; 16 heads, 1024 of 20011 5.3 -> 4.0, all of it
  // in one head of either batch element 5.0 -> 4.3; 128 heads, 512 of 32768 11.9 -> 11.6, in one of eight 18.0 -> 12.1.
  const int lpr = s.d * s.esize / 16, per_block = kGatherThreads / lpr;
  const int units = s.Bz * s.Hkv;
  const int nominal = (min(p->cap, p->budget_per_kv_head) + per_block - 1) / per_block, most = (p->cap + per_block - 1) / per_block;
  const int per_unit = max(1, min((4096 + units - 1) / units, max(nominal, min(most, 512 / units))));
  const dim3 grid(per_unit, units), block(kGatherThreads);
  if (lpr == 8) hipLaunchKernelGGL(gather_kernel<8>, grid, block, 0, stream, a);
  else if (lpr == 16) hipLaunchKernelGGL(gather_kernel<16>, grid, block, 0, stream, a);
  else hipLaunchKernelGGL(gather_kernel<32>, grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace ckv
