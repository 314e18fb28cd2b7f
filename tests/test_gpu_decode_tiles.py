"""Decode attention at the borders of its tiles: rows around the 32 a wave takes, around one workgroup's step and around the
size where rows are cut into chunks; query columns (heads of a group times decoding queries) around the 16 of a
tile; counts of zero, one and all; memory behind the count that holds NaN. Against the oracle with the tolerances of
test_gpu_decode.py."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_08686_amd import binding as B
from parity_util import f32
from test_gpu_decode import _close_rows

pytestmark = pytest.mark.gpu
DEV = "cuda"
# dtype, batch, query heads, KV heads, head_dim, rows, queries
CASES = [
    ("bf16", 1, 2, 2, 128, 1, 1), ("bf16", 2, 8, 2, 128, 31, 1), ("bf16", 1, 16, 1, 64, 33, 1), ("bf16", 2, 17, 1, 128, 257, 1),
    ("bf16", 1, 10, 2, 128, 300, 4), ("bf16", 1, 8, 1, 64, 255, 5), ("bf16", 9, 64, 16, 128, 96, 1), ("bf16", 20, 32, 16, 64, 130, 2),
    ("bf16", 40, 32, 8, 128, 65, 1), ("bf16", 1, 4, 1, 128, 4096, 1), ("bf16", 1, 4, 1, 128, 4097, 1), ("bf16", 2, 6, 2, 64, 4225, 3),
    ("bf16", 1, 20, 1, 128, 8191, 1), ("f32", 1, 4, 2, 128, 4097, 2), ("f32", 2, 8, 1, 64, 5000, 1),
]


@pytest.mark.parametrize("dtype,Bz,Hq,Hkv,d,rows,n_q", CASES)
def test_decode_at_the_borders_of_its_tiles(dtype, Bz, Hq, Hkv, d, rows, n_q):
    print(f"case {dtype} {Bz}x{Hq}/{Hkv}x{d} rows={rows} n_q={n_q}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(rows + 100 * n_q + Hq)
    q = torch.randn(Bz, Hq, n_q, d, generator=g).to(dt)
    k, v = (torch.randn(Bz, Hkv, rows, d, generator=g).to(dt) for _ in range(2))
    count = torch.randint(0, rows + 1, (Bz, Hkv), generator=g, dtype=torch.int32)
    count.view(-1)[0] = rows
    if Bz * Hkv > 1:
        count.view(-1)[-1] = 0
    kd, vd = k.clone(), v.clone()
    for b in range(Bz):
        for h in range(Hkv):
            kd[b, h, int(count[b, h]):] = float("nan")
            vd[b, h, int(count[b, h]):] = float("nan")
    p = B.make_params(batch=Bz, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=rows, window=1, dtype=dtype, pool=B.POOL_NONE,
                      pool_kernel=1, budget=rows, cap=rows)
    out = torch.full((Bz, Hq, n_q, d), float("nan"), device=DEV)
    lse = torch.full((Bz, Hq, n_q), float("nan"), device=DEV)
    ws = torch.full((max(256, B.ckv_decode_workspace_bytes(p, n_q, rows)),), 255, dtype=torch.uint8, device=DEV)
    B.ckv_decode_attention(p, q.to(DEV), kd.to(DEV), vd.to(DEV), count.to(DEV), out, lse, ws)
    torch.cuda.synchronize()
    ref_out, ref_lse = oracle.decode_attention(f32(q), f32(k), f32(v), np.maximum(count.numpy(), 1))
    empty = np.repeat(count.numpy() == 0, Hq // Hkv, axis=1)
    got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
    assert (got[empty] == 0).all() and np.isneginf(got_lse[empty]).all()
    _close_rows(got[~empty], np.asarray(ref_out)[~empty], "out")
    np.testing.assert_allclose(got_lse[~empty], np.asarray(ref_lse)[~empty], rtol=0, atol=1e-4)
