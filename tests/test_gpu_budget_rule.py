"""The budget rule of the tables kernels, by one wave: fewer heads than lanes, exactly as many, more (several per lane), shares that
make the heads drop a level at a time, all at once, or not at all. Integers: equal to the oracle's."""
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
