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

// LPR: lanes (16-byte pieces) per row. What bounds a short list is the chain count -> index -> row: the workgroup's first index
// is read beside the count, the next one beside a row (below cap it is the caller's memory, and it is used only below the count).
template <int LPR>
__global__ void __launch_bounds__(kGatherThreads) gather_kernel(GatherArgs a) {
  constexpr int STEP = kGatherThreads / LPR;  // rows of the workgroup side by side
  const int unit = blockIdx.y;
  const int b = unit / a.Hkv, g = unit % a.Hkv;
  const int list = a.shared ? b : unit;  // whose index list this unit follows
  const int32_t *idx = a.idx + (size_t)list * a.cap;
  const int stride = gridDim.x * STEP;
  int r = blockIdx.x * STEP + threadIdx.x / LPR;
  int t = idx[min(r, a.cap - 1)];
  const int n = min(a.count[list], a.cap);
  const int piece = (threadIdx.x % LPR) * 16;
  const char *kb = a.k + b * a.ks_b + g * a.ks_h + piece, *vb = a.v + b * a.vs_b + g * a.vs_h + piece;
  while (r < n) {
    const int next = idx[min(r + stride, a.cap - 1)];
    if (t >= 0 && t < a.T) {
      const piece_t kk = *reinterpret_cast<const piece_t *>(kb + (int64_t)t * a.ks_t);
      const piece_t vv = *reinterpret_cast<const piece_t *>(vb + (int64_t)t * a.vs_t);
      const size_t o = ((size_t)unit * a.cap + r) * (LPR * 16) + piece;
      *reinterpret_cast<piece_t *>(a.k_out + o) = kk;
      *reinterpret_cast<piece_t *>(a.v_out + o) = vv;
    }
    r += stride;
    t = next;
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
  // As many workgroups as the nominal budget has rows for (at least 512 where the cap has rows for them, at most 4096): a head
  // with more goes over its list in steps. The cap is several times the nominal budget; sized by it, most of 4096
  // workgroups had nothing to do, and handing them out took longer than the copy. us, before and now: 32 heads, 512 of 4096 rows
  // 5.8 -> 4.8; 32 heads, 256 of 10006 4.7 -> 3.4; 16 heads, 256 to 768 of 20011 4.7 -> 3.6; 8 heads, 512 of 131072 3.4 -> 2.8, all of
  // it in one of them 3.2 and 3.2 (of 32 heads of 4096 4.8 -> 5.4); 128 heads, 256 to 768 of 32768 13.6 -> 13.4: 7.3 TB/s, read and
  // written. Two and four rows per thread, 2048 workgroups at most: no faster anywhere.
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
