"""ckv_window_utility where ranges meet: the ends of waves' and workgroups' key ranges and of the prefix at every offset of a tile
and of a group of four, ranges without pipeline rounds, lengths below a tile. The two unfused calls are the reference: the same
sums, the same taps in the same order, the quotient to the last bit in both, hence equal bits."""
import pytest
import torch

from paper_2602_08686_amd import binding as B
from paper_2602_08686_amd import workloads as wl
from parity_util import params_of

pytestmark = pytest.mark.gpu
DEV = "cuda"

# (batch, query heads, KV heads, head size, lengths, windows): 64, 96 and 128 keys per wave, one and several rounds with and without
# keys behind them, one to eight query tiles
SHAPES = [
    (1, 4, 1, 128, (33, 36, 63, 64, 65, 130), (29, 30, 31, 32)),
    (1, 8, 8, 128, (4096, 8191, 8195, 12289), (31, 32, 33, 34)),
    (2, 14, 2, 64, (1023, 1056, 16387, 66000), (32, 33, 40)),
    (2, 8, 4, 128, (20011, 20012, 33001, 49157), (20, 32, 61, 64)),
    (1, 16, 2, 128, (40000, 70003), (30, 32)),
]


@pytest.mark.parametrize("pool,kernel", [(wl.POOL_AVG, 7), (wl.POOL_MAX, 5), (wl.POOL_AVG, 3), (wl.POOL_NONE, 1)])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(x) for x in s[:4]))
def test_fused_utilities_equal_the_unfused_ones(shape, pool, kernel):
    batch, hq, hkv, d, lengths, windows = shape
    for T in lengths:
        for W in windows:
            if W >= T:
                continue
            w = wl.Workload("edges", "bf16", batch, hq, hkv, d, T, W, pool, kernel, min(T, W + 16), 1, seed=T + W, shares=True, gate=True)
            t, tabs = wl.make_layer(w, 0, DEV), wl.make_tables(w, DEV)
            p = params_of(w, t["q"], t["k"], t["v"], layer=0)
            fused, plain = B.LayerBuffers(p, DEV), B.LayerBuffers(p, DEV)
            fused.utility.fill_(float("nan"))
            fused.budget.fill_(-1)
            B.retention_layer(p, t["q"], t["k"], t["v"], tabs, fused, fused_utility=True)
            B.retention_layer(p, t["q"], t["k"], t["v"], tabs, plain)
            for name in ("utility", "tau", "budget", "idx", "count"):
                assert torch.equal(getattr(fused, name), getattr(plain, name)), (name, T, W)


def test_a_share_that_is_no_number_gives_the_window():
    w = wl.Workload("nan_share", "bf16", 1, 4, 4, 128, 2000, 32, wl.POOL_AVG, 7, 100, 1, seed=3, shares=True)
    t, tabs = wl.make_layer(w, 0, DEV), wl.make_tables(w, DEV)
    tabs["head_share"][0, 1] = float("nan")
    p = params_of(w, t["q"], t["k"], t["v"], layer=0)
    fused, plain = B.LayerBuffers(p, DEV), B.LayerBuffers(p, DEV)
    B.retention_layer(p, t["q"], t["k"], t["v"], tabs, fused, fused_utility=True)
    B.retention_layer(p, t["q"], t["k"], t["v"], tabs, plain)
    assert torch.equal(fused.budget, plain.budget) and int(fused.budget[0, 1]) == w.window
