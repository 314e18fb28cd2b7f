// ckv_window_utility and ckv_window_scores with the scan's form chosen by the caller, for tests: both passes as two launches, or as one whose
// workgroups wait `wait` units of 10 ns for one another's row sums. Host code; the functions called are libckv.so's own.
#include "ckv_internal.h"

using namespace ckv;

namespace {
struct Plan {
  Shape s;
  Workspace w;
  Exchange exchange;
  ckv_status st;
  Plan(const ckv_params *p, void *workspace, int two_launches, uint32_t wait) {
    st = validate(p);
    if (st != CKV_OK) return;
    derive(p, &s);
    layout(p, s, &w);
    if (!two_launches) exchange = exchange_of(p, s, w, nullptr, workspace);
    exchange.wait = wait;
  }
};
}  // namespace

extern "C" ckv_status hook_window_utility(const ckv_params *p, const void *q, const void *k, const float *w_head, float *scratch,
                                          float *utility, int32_t *budget, float *tau, void *workspace, size_t bytes,
                                          int two_launches, uint32_t wait, void *stream) {
  const Plan c(p, workspace, two_launches, wait);
  if (c.st != CKV_OK) return c.st;
  return utility_of(p, c.s, c.w, q, k, nullptr, nullptr, w_head, nullptr, nullptr, 0, 0, nullptr, scratch, nullptr, utility, budget, tau,
                    workspace, bytes, (hipStream_t)stream, c.exchange);
}

extern "C" ckv_status hook_window_scores(const ckv_params *p, const void *q, const void *k, float *scores, void *workspace,
                                         size_t bytes, int two_launches, uint32_t wait, void *stream) {
  const Plan c(p, workspace, two_launches, wait);
  if (c.st != CKV_OK) return c.st;
  return scores_of(p, c.s, c.w, q, k, nullptr, nullptr, scores, nullptr, workspace, bytes, (hipStream_t)stream, c.exchange);
}

// Where the marks of a call in one launch lie in its workspace and how many there are (eight bytes each); 0: two launches.
extern "C" int64_t hook_marks(const ckv_params *p, int64_t *offset) {
  char *const base = (char *)4096;
  const Plan c(p, base, 0, 0);
  if (c.st != CKV_OK || !c.exchange.marks) return 0;
  *offset = (char *)c.exchange.marks - base;
  return (int64_t)c.s.Bz * c.s.Hkv * c.s.n_chunks;
}
