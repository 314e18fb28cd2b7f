"""Value norms taken beside the scan's first pass against the separate kernel (which a call with given normalisers runs): the same
ratios to the last bit, and within fp32 rounding of 64 bits. Ranges that end inside a block of 512 rows, inside a step, in one row; one to four
query tiles; strided V; both head sizes; shapes that keep the separate kernel."""
import numpy as np
import pytest
import torch

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("group,window", [(1, 32), (2, 32), (3, 20), (4, 32), (2, 64), (7, 32)])
@pytest.mark.parametrize("d", [64, 128])
def test_norms_beside_the_scan_are_the_separate_kernels(d, group, window, fused):
    for kv, T in ((8, 10006), (8, 16384), (2, 66049), (4, 33281), (1, 1500), (64, 2047)):
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
