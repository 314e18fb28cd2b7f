"""One workspace for layers of one shape with budgets of their own (the paper's B_l): sized for any of the budgets, it
serves every call of every other, and the results are those of a workspace sized for the call."""
import pytest
import torch

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import workloads as wl
from parity_util import params_of

pytestmark = pytest.mark.gpu
DEV = "cuda"
BUDGETS = (128, 700, 5000)


@pytest.mark.parametrize("fused", [False, True], ids=["separate", "one_call"])
@pytest.mark.parametrize("length", [40032, 70035], ids=["multiple_of_four", "ragged"])
def test_workspace_of_another_budget(length, fused):
    print(f"case {length} fused={fused}", flush=True)
    base = wl.Workload("budgets", "bf16", 2, 8, 2, 128, length, 32, wl.POOL_AVG, 7, 128, 1, seed=length, shares=True)
    t, tabs = wl.make_layer(base, 0, DEV), wl.make_tables(base, DEV)
    ps = {b: params_of(base.scaled(budget=b), t["q"], t["k"], t["v"]) for b in BUDGETS}
    ws = {b: torch.full((B.ckv_workspace_bytes(ps[b]),), 0x5A, dtype=torch.uint8, device=DEV) for b in BUDGETS}
    for b in BUDGETS:
        want = None
        for sized_for in (b, *BUDGETS):
            buf = B.LayerBuffers(ps[b], DEV)
            buf.workspace = ws[sized_for]
            B.retention_layer(ps[b], t["q"], t["k"], t["v"], tabs, buf, fused_utility=fused)
            lse = torch.empty(base.batch, base.n_q_heads, base.window, device=DEV)
            B.ckv_window_lse(ps[b], t["q"], t["k"], lse, buf.workspace)
            torch.cuda.synchronize()
            got = (buf.utility, buf.budget, buf.idx, buf.count, buf.k_out, buf.v_out, lse)
            want = want or got
            assert all(torch.equal(x, y) for x, y in zip(got, want)), (b, sized_for)
