"""A layer as one call refuses on the host what its separate calls refuse, with their status."""
import ctypes

import pytest
import torch

from paper_2602_08686_amd import binding as B

D = ctypes.c_void_p(256)   # never dereferenced: every case is refused before a launch


def _params(**kw):
    base = dict(batch=2, n_q_heads=8, n_kv_heads=2, head_dim=128, seq_len=4096, window=32, dtype=torch.bfloat16,
                pool=B.POOL_AVG, pool_kernel=7, budget=256, cap=512)
    base.update(kw)
    return B.make_params(**base)


CASES = [dict(params=dict(window=0)), dict(params=dict(head_dim=96)), dict(params=dict(budget=16)), dict(q=None), dict(k=None), dict(scores=None),
         dict(ws=None), dict(ws=ctypes.c_void_p(8)), dict(ws_bytes=16), dict(params=dict(flags=B.FLAG_VALUE_NORM), v=None),
         dict(params=dict(flags=B.FLAG_VALUE_NORM), rho=None), dict(params=dict(flags=B.FLAG_GROUP_MASS, n_q_heads=16))]


@pytest.mark.parametrize("wanted", [0, 1])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, list(c) + list(c.get("params", {})))))
def test_one_call_refuses_what_the_separate_calls_refuse(case, wanted):
    lib = B.load()
    p = _params(**case.get("params", {}))
    a = {n: case.get(n, D) for n in ("q", "k", "v", "scores", "rho", "ws")}
    nbytes = case.get("ws_bytes", max(B.ckv_workspace_bytes(p), 256))
    ref = ctypes.byref(p)
    if wanted:
        want = lib.ckv_window_scores(ref, a["q"], a["k"], a["v"], None, a["scores"], a["rho"], a["ws"], nbytes, None)
    else:
        want = lib.ckv_window_utility(ref, a["q"], a["k"], a["v"], None, D, None, None, 0, 0, None, a["scores"], a["rho"], D, D, D,
                                      a["ws"], nbytes, None)
    assert want not in (B.CKV_OK, B.CKV_EHIP)
    got = lib.ckv_retention_layer(ref, a["q"], a["k"], a["v"], None, D, None, None, 0, 0, None, a["scores"], wanted, a["rho"], D, D, D, D, D,
                                  D, D, a["ws"], nbytes, None)
    assert got == want


# What a later step refuses, the layer refuses as well, and before its first launch: there is no device here, a launch gives CKV_EHIP.
LATER = [(dict(w_head=None), B.CKV_EINVAL), (dict(utility=None), B.CKV_EINVAL), (dict(budget=None), B.CKV_EINVAL), (dict(tau=None), B.CKV_EINVAL),
         (dict(gate=D), B.CKV_EINVAL), (dict(gate=D, bins=D, n_ent=0, n_ppl=2), B.CKV_EINVAL), (dict(idx=None), B.CKV_EINVAL),
         (dict(count=None), B.CKV_EINVAL), (dict(v=None), B.CKV_EINVAL), (dict(k_out=None), B.CKV_EINVAL), (dict(v_out=None), B.CKV_EINVAL),
         (dict(params=dict(flags=B.FLAG_GROUP_MASS)), B.CKV_EINVAL),
         # two faults: the first step's is the one that is told
         (dict(idx=None, ws=None), B.CKV_EWORKSPACE), (dict(v_out=None, params=dict(window=200, seq_len=4096)), B.CKV_EUNSUPPORTED)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers: only where nothing can be launched")
@pytest.mark.parametrize("wanted", [0, 1])
@pytest.mark.parametrize("case,want", LATER, ids=lambda c: "-".join(map(str, c)) if isinstance(c, dict) else str(c))
def test_one_call_refuses_before_its_first_launch(case, want, wanted):
    lib = B.load()
    p = _params(**dict(dict(budget=256), **case.get("params", {})))
    if case.get("params", {}).get("window", 0) > 128:
        p.cap = p.seq_len
    names = ("q", "k", "v", "w_head", "scores", "rho", "utility", "budget", "tau", "idx", "count", "k_out", "v_out", "ws")
    a = {n: case.get(n, D) for n in names}
    nbytes = max(B.ckv_workspace_bytes(p), 256)
    call = lambda a, n_ent, n_ppl: lib.ckv_retention_layer(  # noqa: E731
        ctypes.byref(p), a["q"], a["k"], a["v"], None, a["w_head"], None, case.get("gate"), n_ent, n_ppl, case.get("bins"),
        a["scores"], wanted, a["rho"], a["utility"], a["budget"], a["tau"], a["idx"], a["count"], a["k_out"], a["v_out"], a["ws"], nbytes, None)
    assert call(a, case.get("n_ent", 2), case.get("n_ppl", 2)) == want
