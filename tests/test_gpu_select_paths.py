"""Selection at the sizes where its kernels change: positions per thread, one launch against slices and merge, quotas at the
list's capacity, rows that start at any multiple of four bytes; values with ties, outliers and few candidates. Exact
against the oracle: the result is unique."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
SIZES = (1, 63, 1024, 1025, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 49157, 65536, 65537, 131071)
QUOTAS = (0, 1, 63, 512, 513, 3072, 3584, 3585)


def _values(rng, kind, shape):
    if kind == "ties":
        return rng.choice(np.linspace(0.0, 2.0, 9).astype(np.float32), size=shape)
    if kind == "outliers":
        u = np.exp(0.5 * rng.standard_normal(shape))
        u[..., : min(3, shape[-1])] *= 1e4
        return u.astype(np.float32)
    return (1.0 + 0.08 * np.abs(rng.standard_normal(shape))).astype(np.float32)   # pooled masses: all close together


@pytest.mark.parametrize("workspace", [False, True], ids=["plain", "workspace"])
@pytest.mark.parametrize("kind", ["close", "ties", "outliers"])
@pytest.mark.parametrize("P", SIZES)
def test_select_matches_oracle_at_the_borders(P, kind, workspace):
    print(f"case P={P} {kind} workspace={workspace}", flush=True)
    rng = np.random.default_rng(P + len(kind))
    W, Hkv, T = 4, 2, P + 4
    u = np.repeat(_values(rng, kind, (1, Hkv, P)), 2, axis=0)
    flat = torch.empty(u.size + 1, device=DEV)
    ut = flat[1:].view(u.shape)       # one float past an aligned address
    ut.copy_(torch.from_numpy(u))
    for quota in sorted({min(q, P) for q in QUOTAS}):
        for tau in (0.0, 1.3):
            cap = W + quota
            # one head at its nominal budget, one at the smallest, and the other way round
            budget = np.array([[W + quota, W + min(quota, 1)], [W + min(quota, 1), W + quota]], np.int32)
            p = B.make_params(batch=2, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=T, window=W, dtype="bf16",
                              pool=B.POOL_NONE, pool_kernel=1, budget=W + quota // 2, cap=cap)
            ws = None
            if workspace:   # contents on entry are ignored: ones
                ws = torch.full((max(256, B.ckv_workspace_bytes(p)),), 255, dtype=torch.uint8, device=DEV)
            idx = torch.full((2, Hkv, cap), -1, dtype=torch.int32, device=DEV)
            count = torch.empty(2, Hkv, dtype=torch.int32, device=DEV)
            B.ckv_select_topk(p, ut, torch.from_numpy(budget).to(DEV), torch.full((2,), tau, device=DEV), idx, count, ws)
            torch.cuda.synchronize()
            oi, oc = oracle.select(u, np.array([tau, tau], np.float32), budget, W, cap)
            np.testing.assert_array_equal(count.cpu().numpy(), oc)
            np.testing.assert_array_equal(idx.cpu().numpy(), oi)


def _bytes(units, P, W, budget, cap, Hkv):
    return B.ckv_workspace_bytes(B.make_params(batch=units // Hkv, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W,
                                               dtype="bf16", pool=B.POOL_NONE, pool_kernel=1, budget=budget, cap=cap))


@pytest.mark.parametrize("form", ["slices", "split"])
@pytest.mark.parametrize("kind", ["close", "ties", "outliers", "equal", "mantissa", "few"])
@pytest.mark.parametrize("P,top", [(32769, 8192), (65540, 15000), (70001, 12000), (131040, 9000), (200000, 7000)])
def test_select_over_long_rows_by_both_forms(P, top, kind, form):
    """Slices and merge, and the split selection, on the same rows: budgets from nothing to `top` for one head (beyond 32768
    pairs for the merge, and beyond the room for pairs), heads with fewer candidates than their budget, candidates that only
    position or the last bits of the mantissa tell apart. The nominal budget decides the form; the size of the workspace
    tells which one it is."""
    print(f"case P={P} top={top} {kind} {form}", flush=True)
    rng = np.random.default_rng(P + len(kind))
    W, Hkv, bz = 4, 5, 2
    cap = W + top
    nominal = W + (600 if form == "slices" else 3500)
    u = _values(rng, kind, (bz, Hkv, P))
    if kind == "equal":
        u = np.full((bz, Hkv, P), 0.75, np.float32)
    elif kind == "mantissa":
        u = (np.float32(1.0) + (np.arange(P, dtype=np.float32) % 97 * np.float32(1.2e-7))) * np.ones((bz, Hkv, 1), np.float32)
    tau = np.array([0.0, float(np.partition(u[1, 0], -200)[-200]) if kind == "few" else 0.0], np.float32)
    budget = np.array([[W + top, W, W + 1, W + 777, W + 2048], [W + 63, W + top, W + top // 2, W + 64, W]], np.int32)
    p = B.make_params(batch=bz, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W, dtype="bf16",
                      pool=B.POOL_NONE, pool_kernel=1, budget=nominal, cap=max(cap, Hkv * nominal - (Hkv - 1) * W))
    assert (B.ckv_workspace_bytes(p) > _bytes(bz * Hkv, P, W, W + 3500, Hkv * (W + 3500), Hkv)) == (form == "slices")
    ws = torch.full((B.ckv_workspace_bytes(p),), 255, dtype=torch.uint8, device=DEV)
    idx = torch.full((bz, Hkv, p.cap), -1, dtype=torch.int32, device=DEV)
    count = torch.empty(bz, Hkv, dtype=torch.int32, device=DEV)
    B.ckv_select_topk(p, torch.from_numpy(u).to(DEV), torch.from_numpy(budget).to(DEV), torch.from_numpy(tau).to(DEV), idx, count, ws)
    torch.cuda.synchronize()
    oi, oc = oracle.select(u, tau, budget, W, p.cap)
    np.testing.assert_array_equal(count.cpu().numpy(), oc)
    np.testing.assert_array_equal(idx.cpu().numpy(), oi)


@pytest.mark.parametrize("P", [32769, 65540, 262145])
@pytest.mark.parametrize("top", [1025, 1468, 2048])
def test_select_over_long_rows_of_one_head(P, top):
    """One KV head: the nominal budget is all that it can have, so slices and their merge serve it up to a list of 2048 entries
    (half of that where other heads can leave it theirs); the size of the workspace tells."""
    print(f"case P={P} top={top}", flush=True)
    W, bz = 4, 2
    u = _values(np.random.default_rng(P + top), "ties", (bz, 1, P))
    tau, budget = np.zeros(bz, np.float32), np.array([[W + top], [W + 1]], np.int32)
    cap = W + top
    assert _bytes(bz, P, W, cap, cap, 1) > _bytes(bz, P, W, W + 2049, W + 2049, 1)
    p = B.make_params(batch=bz, n_q_heads=1, n_kv_heads=1, head_dim=64, seq_len=P + W, window=W, dtype="bf16", pool=B.POOL_NONE,
                      pool_kernel=1, budget=cap, cap=cap)
    ws = torch.full((B.ckv_workspace_bytes(p),), 255, dtype=torch.uint8, device=DEV)
    idx = torch.full((bz, 1, cap), -1, dtype=torch.int32, device=DEV)
    count = torch.empty(bz, 1, dtype=torch.int32, device=DEV)
    B.ckv_select_topk(p, torch.from_numpy(u).to(DEV), torch.from_numpy(budget).to(DEV), torch.from_numpy(tau).to(DEV), idx, count, ws)
    torch.cuda.synchronize()
    oi, oc = oracle.select(u, tau, budget, W, cap)
    np.testing.assert_array_equal(count.cpu().numpy(), oc)
    np.testing.assert_array_equal(idx.cpu().numpy(), oi)
