"""Decode attention over values with infinite components: a weight above zero times an infinite component is infinite, with
the component's sign, in both element types (a component is NaN only where infinities of both signs meet or V holds NaN); the
other components, queries and KV heads stay what they are."""
import pytest
import torch

from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"
INF = float("inf")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [64, 128])
# one launch with V split over four, two and one workgroups; chunks and their merge; one chunk over long rows
@pytest.mark.parametrize("Bz,Hq,Hkv,rows,n_q", [(1, 4, 1, 1, 1), (2, 8, 2, 300, 1), (40, 8, 2, 100, 1), (40, 32, 8, 33, 1),
                                                (2, 8, 2, 5000, 2), (9, 128, 1, 4200, 4)])
def test_infinite_value_components(dtype, d, Bz, Hq, Hkv, rows, n_q):
    print(f"case {dtype} d={d} {Bz}x{Hq}/{Hkv} rows={rows} n_q={n_q}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(rows + d)
    q = torch.randn(Bz, Hq, n_q, d, generator=g).to(dt)
    k, v = (torch.randn(Bz, Hkv, rows, d, generator=g).to(dt) for _ in range(2))
    count = torch.randint(max(1, rows // 2), rows + 1, (Bz, Hkv), generator=g, dtype=torch.int32)
    count[0, 0] = rows
    clean = v.clone()
    # +inf in one row's component 3; -inf in two rows' component 17; both signs in d - 2; NaN in d - 1; +inf behind the count
    v[0, 0, rows // 2, 3] = INF
    v[0, 0, 0, 17] = v[0, 0, rows - 1, 17] = -INF
    v[0, 0, 0, d - 2] = INF
    v[0, 0, rows - 1, d - 2] = -INF
    v[0, 0, rows // 3, d - 1] = float("nan")
    if int(count[-1, -1]) < rows:
        v[-1, -1, int(count[-1, -1]):] = INF
    p = B.make_params(batch=Bz, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=rows, window=1, dtype=dtype, pool=B.POOL_NONE,
                      pool_kernel=1, budget=rows, cap=rows)

    def decode(values):
        out = torch.full((Bz, Hq, n_q, d), 7.0, device=DEV)
        lse = torch.full((Bz, Hq, n_q), float("nan"), device=DEV)
        ws = torch.full((max(256, B.ckv_decode_workspace_bytes(p, n_q, rows)),), 255, dtype=torch.uint8, device=DEV)
        B.ckv_decode_attention(p, q.to(DEV), k.to(DEV), values.to(DEV), count.to(DEV), out, lse, ws)
        torch.cuda.synchronize()
        return out.cpu(), lse.cpu()

    out, lse = decode(v)
    want, want_lse = decode(clean)
    heads = Hq // Hkv
    want[0, :heads, :, 3] = INF
    want[0, :heads, :, 17] = -INF
    want[0, :heads, :, d - 2] = -INF if rows == 1 else float("nan")
    want[0, :heads, :, d - 1] = float("nan")
    assert torch.isfinite(want_lse).all() and torch.equal(lse, want_lse)
    # what no infinity reaches is the same number (a component of one row's other sums may not move)
    assert torch.equal(torch.nan_to_num(out, 1e30, 2e30, -2e30), torch.nan_to_num(want, 1e30, 2e30, -2e30))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_infinite_component_at_a_small_weight(dtype):
    """Weights of e^-97 (below the smallest normal number, above zero) and e^-200 (zero): infinite and NaN."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rows, d = 8, 64
    q, k, v = (torch.zeros(1, 1, n, d, device=DEV, dtype=dt) for n in (1, rows, rows))
    q[..., 0] = 1.0
    k[0, 0, 5, 0], k[0, 0, 6, 0] = -97.0, -200.0
    v[0, 0, 5, 3], v[0, 0, 6, 9] = INF, INF
    p = B.make_params(batch=1, n_q_heads=1, n_kv_heads=1, head_dim=d, seq_len=rows, window=1, dtype=dtype, pool=B.POOL_NONE,
                      pool_kernel=1, budget=rows, cap=rows, softmax_scale=1.0)
    out, lse = torch.zeros(1, 1, 1, d, device=DEV), torch.zeros(1, 1, 1, device=DEV)
    B.ckv_decode_attention(p, q, k, v, None, out, lse, torch.empty(256, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    want = torch.zeros(d)
    want[3], want[9] = INF, float("nan")
    assert torch.equal(torch.nan_to_num(out.cpu().view(d), 1e30, 2e30, -2e30), torch.nan_to_num(want, 1e30, 2e30, -2e30))
