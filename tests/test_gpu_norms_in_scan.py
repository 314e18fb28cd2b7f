"""Value norms taken beside the scan's first pass against the separate kernel (which a call with given normalisers runs): the same
ratios to the last bit, and within fp32 rounding of 64 bits. Ranges that end inside a block of 512 rows, inside a step, in one row; one to four
query tiles; strided V; both head sizes; shapes that keep the separate kernel."""
import numpy as np
import pytest
import torch

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import workloads as wl
from parity_util import norms_beside_the_scan

pytestmark = pytest.mark.gpu
DEV = "cuda"
WIDTHS = (64, 128)
GROUPS = ((1, 32), (2, 32), (3, 20), (4, 32), (2, 64), (7, 32))
LENGTHS = ((8, 10006), (8, 16384), (2, 66049), (4, 33281), (1, 1500), (64, 2047))


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("group,window", GROUPS)
@pytest.mark.parametrize("d", WIDTHS)
def test_norms_beside_the_scan_are_the_separate_kernels(d, group, window, fused):
    for kv, T in LENGTHS:
        g = torch.Generator(device=DEV)
        g.manual_seed(T + d + group)
        q = torch.randn(1, kv * group, window, d, generator=g, device=DEV).bfloat16()
        k = torch.randn(1, kv, T, d, generator=g, device=DEV).bfloat16()
        v = torch.randn(1, T, kv, d, generator=g, device=DEV).bfloat16().transpose(1, 2)  # rows of all heads side by side
        v[:, :, T // 3] *= 1e4
        v[:, :, -1] = 0
        p = B.params_for(q, k, v, pool=wl.POOL_AVG, pool_kernel=7, budget=window + 8, cap=T, n_layers=1, flags=B.FLAG_VALUE_NORM)
        w_head = torch.ones(1, kv * group, device=DEV)
        got = []
        for given in (False, True):
            buf = B.LayerBuffers(p, DEV)
            for t in (buf.vnorm_ratio, buf.utility, buf.scores):
                t.fill_(float("nan"))
            lse = torch.empty(1, kv * group, window, device=DEV) if given else None
            if given:
                B.ckv_window_lse(p, q, k, lse, buf.workspace)
            B.retention_layer(p, q, k, v, {"w_head": w_head}, buf, lse=lse, fused_utility=fused)
            got.append((buf.vnorm_ratio.clone(), buf.utility.clone()))
        assert torch.equal(got[0][0], got[1][0]), (kv, T)
        assert torch.equal(got[0][1], got[1][1]), (kv, T)
        r = v.double().norm(dim=-1)
        ref = (r / (r.mean(-1, keepdim=True) + 1e-6)).cpu().numpy()
        # 128 squares added in fp32 and the mean of T norms: a few ulp
        np.testing.assert_allclose(got[0][0].cpu().numpy(), ref, rtol=2e-6)


@pytest.mark.parametrize("flags", [B.FLAG_VALUE_NORM, B.FLAG_VALUE_NORM | B.FLAG_GROUP_MASS], ids=["heads", "group_mass"])
@pytest.mark.parametrize("d,group", [(64, 4), (128, 1), (128, 3), (128, 4)])
def test_norms_of_a_batch_and_with_group_sums(d, group, flags):
    """Two batch elements whose V rows lie side by side for all heads of both, per-head and group-sum second passes."""
    kv, window, batch = 4, 32, 2
    for T in (16384, 21001, 33000):
        g = torch.Generator(device=DEV)
        g.manual_seed(T + d + group)
        q = torch.randn(batch, kv * group, window, d, generator=g, device=DEV).bfloat16()
        k = torch.randn(batch, kv, T, d, generator=g, device=DEV).bfloat16()
        v = torch.randn(T, batch, kv, d, generator=g, device=DEV).bfloat16().permute(1, 2, 0, 3)
        p = B.params_for(q, k, v, pool=wl.POOL_AVG, pool_kernel=7, budget=window + 8, cap=T, n_layers=1, flags=flags)
        assert norms_beside_the_scan(p) and not norms_beside_the_scan(p, lse_given=True)
        rows = kv if flags & B.FLAG_GROUP_MASS else kv * group
        ws = torch.empty(B.ckv_workspace_bytes(p), dtype=torch.uint8, device=DEV)
        lse = torch.empty(batch, kv * group, window, device=DEV)
        B.ckv_window_lse(p, q, k, lse, ws)
        got = []
        for given in (None, lse):
            scores, ratio = (torch.full((batch, n, T), float("nan"), device=DEV) for n in (rows, kv))
            B.ckv_window_scores(p, q, k, v, given, scores, ratio, ws)
            got.append((scores, ratio))
        assert torch.equal(got[0][1], got[1][1]), T
        # the normalisers merged by the second pass and those of ckv_window_lse: the same partials in the same order
        assert torch.equal(got[0][0], got[1][0]), T
        r = v.double().norm(dim=-1)
        np.testing.assert_allclose(got[0][1].cpu().numpy(), (r / (r.mean(-1, keepdim=True) + 1e-6)).cpu().numpy(), rtol=2e-6)


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), 3e38])
@pytest.mark.parametrize("kv,group,d,T,given", [(8, 4, 128, 16384, False), (8, 1, 64, 16384, False), (8, 4, 128, 16384, True), (4, 7, 128, 9000, False)])
def test_rows_of_v_that_are_not_finite(kv, group, d, T, given, bad):
    """A row with an infinite norm makes its head's mean infinite: every ratio of the head is 0, that row's own no number; a row that is no
    number makes all of them none. Other heads are what they were, and the utilities are the utilities without the factor times the ratio."""
    window = 32
    g = torch.Generator(device=DEV)
    g.manual_seed(T + d)
    q = torch.randn(1, kv * group, window, d, generator=g, device=DEV).bfloat16()
    k = torch.randn(1, kv, T, d, generator=g, device=DEV).bfloat16()
    v = torch.randn(1, kv, T, d, generator=g, device=DEV).bfloat16()
    with_norms, plain = (B.params_for(q, k, v, pool=wl.POOL_AVG, pool_kernel=7, budget=window + 8, cap=T, n_layers=1, flags=f)
                         for f in (B.FLAG_VALUE_NORM, 0))
    w_head = torch.ones(1, kv * group, device=DEV)
    ws = torch.empty(B.ckv_workspace_bytes(with_norms), dtype=torch.uint8, device=DEV)
    lse = torch.empty(1, kv * group, window, device=DEV) if given else None
    if given:
        B.ckv_window_lse(plain, q, k, lse, ws)
    new = lambda *s, dtype=torch.float32: torch.empty(*s, dtype=dtype, device=DEV)  # noqa: E731
    scratch, budget, tau = new(1, kv * group, T), new(1, kv, dtype=torch.int32), new(1)

    def utility(p, values):
        u, ratio = new(1, kv, T - window), new(1, kv, T)
        B.ckv_window_utility(p, q, k, values, lse, w_head, None, None, 0, 0, None, scratch, ratio, u, budget, tau, ws)
        return u, ratio

    u0, _ = utility(plain, None)
    before = utility(with_norms, v)[1]
    broken = v.clone()
    broken[0, 1, 777, 3] = bad
    u, ratio = utility(with_norms, broken)
    norm = broken.double().norm(dim=-1).float()  # a square beyond the range of 32 bits is infinite there as well
    norm = torch.where(broken.float().square().sum(-1).isinf(), torch.full_like(norm, float("inf")), norm)
    want = norm[0, 1] / (norm[0, 1].mean() + 1e-6)
    assert torch.equal(ratio[0, 1].isnan(), want.isnan()) and (ratio[0, 1][~want.isnan()] == 0).all()
    others = [h for h in range(kv) if h != 1]
    assert torch.equal(ratio[0, others], before[0, others])
    torch.testing.assert_close(u, u0 * ratio[..., :T - window], rtol=0, atol=0, equal_nan=True)
