"""Decode attention over long KV sets of many units: so many (unit, query) workgroups that the rows are not cut (one chunk per
workgroup, which writes the result itself; no merge follows), or few chunks each. f32 with every count of heads a workgroup
takes, bf16 with one column (on the vector ALUs), and one and several column tiles, unit counts that are no multiple of
eight; counts of zero, one and all. All units read the same rows
(strides of zero), which keeps the memory small. Against the oracle with the tolerances of test_gpu_decode.py; every output is
prefilled with NaN, so one that nobody writes shows up."""
import numpy as np
import pytest
import torch

import oracle
from paper_2602_08686_amd import binding as B
from parity_util import f32
from test_gpu_decode import _close_rows

pytestmark = pytest.mark.gpu
DEV = "cuda"
# dtype, batch, query heads, KV heads, head_dim, rows, queries, partial rows of the workspace per unit and chunk: one chunk or more
CASES = [
    ("f32", 64, 32, 8, 64, 20000, 8, 32, True),      # 4096 workgroups of four heads
    ("f32", 513, 64, 8, 128, 16385, 1, 8, True),     # 4104 of eight
    ("f32", 4097, 2, 1, 64, 16400, 1, 2, True),      # two heads
    ("f32", 4097, 1, 1, 64, 16400, 1, 1, True),      # one
    ("bf16", 64, 32, 8, 128, 4200, 1, 4, True),      # 512 workgroups
    ("bf16", 127, 16, 4, 64, 4161, 2, 8, True),      # 508
    ("bf16", 85, 60, 3, 128, 4200, 1, 32, True),     # 255 units of 20 columns: two tiles
    ("bf16", 67, 68, 4, 64, 4161, 1, 32, False),     # 268 units of 17
    ("bf16", 27, 20, 5, 128, 4200, 5, 32, False),    # 135 units of 20 columns
    ("bf16", 33, 16, 8, 128, 5000, 1, 2, False),     # 264 units
    ("bf16", 263, 16, 4, 128, 16420, 1, 4, False),   # 1052
    ("bf16", 40, 8, 8, 128, 5000, 1, 1, False),      # one column: the vector kernel, chunks
    ("bf16", 4099, 1, 1, 128, 16400, 1, 1, True),    # and one chunk
]


@pytest.mark.parametrize("dtype,Bz,Hq,Hkv,d,rows,n_q,part_rows,one", CASES)
def test_decode_with_few_chunks_over_long_rows(dtype, Bz, Hq, Hkv, d, rows, n_q, part_rows, one):
    print(f"case {dtype} {Bz}x{Hq}/{Hkv}x{d} rows={rows} n_q={n_q}", flush=True)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(rows + Bz)
    q = torch.randn(Bz, Hq, n_q, d, generator=g).to(dt)
    k, v = (torch.randn(1, 1, rows, d, generator=g).to(dt) for _ in range(2))
    count = torch.randint(0, rows + 1, (Bz, Hkv), generator=g, dtype=torch.int32)
    count.view(-1)[:4] = torch.tensor([rows, 0, 1, rows - 1], dtype=torch.int32)
    count.view(-1)[-1] = rows
    p = B.make_params(batch=Bz, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=rows, window=1, dtype=dtype, pool=B.POOL_NONE,
                      pool_kernel=1, budget=rows, cap=rows)
    out = torch.full((Bz, Hq, n_q, d), float("nan"), device=DEV)
    lse = torch.full((Bz, Hq, n_q), float("nan"), device=DEV)
    need, one_chunk = B.ckv_decode_workspace_bytes(p, n_q, rows), Bz * Hkv * part_rows * (d + 2) * 4
    assert need - need % 256 in (one_chunk - one_chunk % 256, (one_chunk + 255) // 256 * 256) if one else need >= 2 * one_chunk
    ws = torch.full((need,), 255, dtype=torch.uint8, device=DEV)
    kd, vd = (x.to(DEV).expand(Bz, Hkv, rows, d) for x in (k, v))
    B.ckv_decode_attention(p, q.to(DEV), kd, vd, count.to(DEV), out, lse, ws)
    torch.cuda.synchronize()
    got, got_lse = out.cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(got).all() and not np.isnan(got_lse).any()
    G, flat = Hq // Hkv, count.view(-1)
    units = sorted({0, 1, 2, 3, 8, 9, Bz * Hkv // 2, Bz * Hkv - 2, Bz * Hkv - 1})
    for u in units:
        b, h, n = u // Hkv, u % Hkv, int(flat[u])
        heads = slice(h * G, (h + 1) * G)
        if n == 0:
            assert (got[b, heads] == 0).all() and np.isneginf(got_lse[b, heads]).all()
            continue
        ref_out, ref_lse = oracle.decode_attention(f32(q[b:b + 1, heads]), f32(k[:, :, :n]), f32(v[:, :, :n]))
        _close_rows(got[b, heads], np.asarray(ref_out)[0], f"unit {u}")
        np.testing.assert_allclose(got_lse[b, heads], np.asarray(ref_lse)[0], rtol=0, atol=1e-4)
