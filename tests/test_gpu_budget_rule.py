"""The budget rule of the tables kernels, by one wave: fewer heads than lanes, exactly as many, more (several per lane), shares that
make the heads drop a level at a time, all at once, or not at all; the copies of the rule in the long-pool kernel and in the fused
pass, and shares that are no numbers of tokens; batches that fill several rows of workgroups, or more than a launch's second dimension
holds beside the tiles. Integers, and tau's bits: equal to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["none", "even", "skewed", "ties", "over"])
@pytest.mark.parametrize("heads", [1, 2, 7, 63, 64, 65, 128, 200])
def test_budgets_of_any_number_of_heads(heads, kind):
    T, W, budget = 300, 9, 50
    rng = np.random.default_rng(heads)
    share = {"none": None, "even": np.full(heads, 1.0 / heads), "skewed": rng.dirichlet(np.full(heads, 0.2)),
             "ties": rng.integers(1, 4, heads) / (1.5 * heads), "over": rng.uniform(0.0, 6.0, heads) / heads}[kind]
    cap = min(T, budget * heads - (heads - 1) * W)
    p = B.make_params(batch=2, n_q_heads=heads, n_kv_heads=heads, head_dim=64, seq_len=T, window=W, dtype="bf16", pool=B.POOL_NONE,
                      pool_kernel=1, budget=budget, cap=cap)
    new = lambda *s, dtype=torch.float32: torch.zeros(*s, dtype=dtype, device="cuda")  # noqa: E731
    out = torch.full((2, heads), -1, dtype=torch.int32, device="cuda")
    shares = None if share is None else torch.from_numpy(share.astype(np.float32))[None].cuda()
    B.ckv_apply_tables(p, new(2, heads, T), None, new(1, heads) + 1, shares, None, 0, 0, None, new(2, heads, T - W), out, new(2))
    want = oracle.budgets(heads, T, W, budget, None if share is None else share.astype(np.float32))
    for b in range(2):
        np.testing.assert_array_equal(out[b].cpu().numpy(), want)


def _shares(kind, heads, rng):
    if kind == "none":
        return None
    share = {"even": np.full(heads, 1.0 / heads), "ties": rng.integers(1, 4, heads) / (1.5 * heads),
             "over": rng.uniform(0.0, 6.0, heads) / heads}.get(kind, rng.uniform(0.0, 2.0, heads) / heads).astype(np.float32)
    if kind in ("inf", "-inf", "nan", "-1"):
        share[heads // 2] = float(kind)
    return share


@pytest.mark.parametrize("kind", ["none", "even", "ties", "over", "inf", "-inf", "nan", "-1"])
@pytest.mark.parametrize("entry", ["short_pool", "long_pool", "fused", "no_prefix"])
@pytest.mark.parametrize("heads", [1, 4, 63, 64, 65, 200])
def test_every_copy_of_the_rule(entry, heads, kind):
    T, W, budget, batch = (24, 24, 30, 3) if entry == "no_prefix" else (300, 9, 50, 3)
    rng = np.random.default_rng(heads)
    share = _shares(kind, heads, rng)
    cap = min(T, budget * heads - (heads - 1) * W)
    kernel = 21 if entry == "long_pool" else 7
    g = torch.Generator(device="cuda")
    g.manual_seed(heads)
    q = torch.randn(batch, heads, W, 64, generator=g, device="cuda").bfloat16()
    k = torch.randn(batch, heads, T, 64, generator=g, device="cuda").bfloat16()
    p = B.params_for(q, k, None, pool=B.POOL_AVG, pool_kernel=kernel, budget=budget, cap=cap, n_layers=1)
    new = lambda *s, dtype=torch.float32: torch.zeros(*s, dtype=dtype, device="cuda")  # noqa: E731
    out, tau, utility = torch.full((batch, heads), -1, dtype=torch.int32, device="cuda"), new(batch) - 1, new(batch, heads, max(T - W, 1))
    shares = None if share is None else torch.from_numpy(share)[None].cuda()
    gate = torch.rand(1, 3, 5, generator=g, device="cuda")
    bins = torch.tensor([[0, 4], [2, 0], [9, -3]], dtype=torch.int32, device="cuda")  # the last one outside the table: its nearest cell
    w_head = new(1, heads) + 1
    if entry == "fused":
        ws = torch.empty(max(B.ckv_workspace_bytes(p), 256), dtype=torch.uint8, device="cuda")
        B.ckv_window_utility(p, q, k, None, None, w_head, shares, gate, 3, 5, bins, new(batch, heads, T), None, utility, out, tau, ws)
    else:
        B.ckv_apply_tables(p, new(batch, heads, T), None, w_head, shares, gate, 3, 5, bins, utility, out, tau)
    want = oracle.budgets(heads, T, W, budget, share)
    for b in range(batch):
        np.testing.assert_array_equal(out[b].cpu().numpy(), want)
    assert torch.equal(tau, torch.stack([gate[0, 0, 4], gate[0, 2, 0], gate[0, 2, 0]]))


@pytest.mark.parametrize("batch,heads,T,kernel", [
    (3, 1, 3100, 1), (4, 2, 3100, 7), (7, 2, 3100, 21), (300, 1, 1100, 1),  # a row of four or two tiles: one row in front, more, with a rest
    (32767, 1, 5, 1), (32768, 1, 5, 1), (65535, 1, 2, 1), (257, 255, 8, 3),  # one launch and two
])
@pytest.mark.parametrize("shares", [False, True])
def test_rows_in_front_of_the_tiles(batch, heads, T, kernel, shares):
    W, budget = 1, 2
    cap = min(T, budget * heads - (heads - 1) * W)
    g = torch.Generator(device="cuda")
    g.manual_seed(batch)
    p = B.make_params(batch=batch, n_q_heads=heads, n_kv_heads=heads, head_dim=64, seq_len=T, window=W, dtype="bf16", pool=B.POOL_MAX,
                      pool_kernel=kernel, budget=budget, cap=cap)
    scores = torch.rand(batch, heads, T, generator=g, device="cuda")
    share = np.random.default_rng(heads).uniform(0.0, 3.0, heads).astype(np.float32) / heads if shares else None
    gate = torch.rand(1, 7, 11, generator=g, device="cuda")
    bins = torch.stack([torch.randint(0, n, (batch,), generator=g, device="cuda", dtype=torch.int32) for n in (7, 11)], 1)
    utility = torch.full((batch, heads, T - W), float("nan"), device="cuda")
    out, tau = torch.full((batch, heads), -1, dtype=torch.int32, device="cuda"), torch.full((batch,), -1.0, device="cuda")
    w_head = torch.ones(1, heads, device="cuda")
    B.ckv_apply_tables(p, scores, None, w_head, None if share is None else torch.from_numpy(share)[None].cuda(), gate, 7, 11, bins, utility,
                       out, tau)
    want = torch.from_numpy(oracle.budgets(heads, T, W, budget, share)).cuda()
    assert (out == want).all() and torch.equal(tau, gate[0, bins[:, 0].long(), bins[:, 1].long()])
    pooled = scores[..., : T - W]  # maxima: the same bits
    if kernel > 1:
        pooled = torch.nn.functional.max_pool1d(pooled, kernel, 1, kernel // 2)
    assert torch.equal(utility, pooled)
