"""Selection and gather of a layer in one launch against the two calls on the same utilities, bit by bit: without shares and with
all of the budget in one head; prefixes at the kernels' limits, quotas of nothing, of less than a block of rows and of several,
fewer candidates than the quota, strided rows, both head sizes and types."""
import pytest
import torch

from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("kind", ["plain", "gate", "one_head"])
@pytest.mark.parametrize("dtype,d", [(torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 64), (torch.float32, 128)], ids=str)
@pytest.mark.parametrize("P,batch,kv,budget", [
    (1, 1, 2, 9), (1024, 1, 4, 128), (1025, 2, 8, 8), (4064, 1, 32, 512), (4097, 1, 8, 77), (8192, 4, 8, 513), (8193, 1, 3, 2040),
    (16385, 2, 8, 257), (32768, 1, 8, 1000), (32769, 1, 4, 300), (700, 40, 4, 64), (600, 65, 2, 64),
])
def test_layer_keeps_what_the_two_calls_keep(P, batch, kv, budget, dtype, d, kind):
    print("case", P, batch, kv, budget, dtype, d, kind, flush=True)
    W, T = 8, P + 8
    g = torch.Generator(device=DEV)
    g.manual_seed(P + d)
    budget = min(max(budget, W), T)
    cap = min(T, budget * kv - (kv - 1) * W)
    draw = lambda rows, h: torch.randn(batch, h, rows, d, generator=g, device=DEV).to(dtype)  # noqa: E731
    q, k = draw(W, kv), draw(T, kv)
    v = draw(T, kv).transpose(1, 2).contiguous().transpose(1, 2)   # rows of all heads of a token side by side
    p = B.params_for(q, k, v, pool=B.POOL_AVG, pool_kernel=5, budget=budget, cap=cap)
    tables = {"w_head": 0.5 + torch.rand(1, kv, generator=g, device=DEV)}
    if kind == "one_head":
        tables["head_share"] = torch.zeros(1, kv, device=DEV)
        tables["head_share"][0, kv // 2] = 1.0
    if kind == "gate":   # masses have a mean of one: few positions reach the threshold
        tables.update(t_gate=torch.full((1, 1, 1), 1.3, device=DEV), n_ent=1, n_ppl=1, risk_bins=torch.zeros(batch, 2, dtype=torch.int32, device=DEV))
    buf, want = B.LayerBuffers(p, DEV), B.LayerBuffers(p, DEV)
    B.retention_layer(p, q, k, v, tables, buf, fused_utility=True)
    B.ckv_select_topk(p, buf.utility, buf.budget, buf.tau, want.idx, want.count, want.workspace)
    B.ckv_compact_kv(p, k, v, want.idx, want.count, want.k_out, want.v_out)
    torch.cuda.synchronize()
    for name in ("count", "idx", "k_out", "v_out"):
        assert torch.equal(getattr(buf, name), getattr(want, name)), name
