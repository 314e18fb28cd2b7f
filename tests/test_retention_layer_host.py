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
