"""Kernels on the host CPU, where an access out of bounds ends a child process instead of a GPU: decode attention reads no
row behind the count (the memory there has no access)."""
import ctypes
import multiprocessing

import numpy as np
import pytest

import cpu_build as cpu
from paper_2602_08686_amd import binding as B

pytestmark = pytest.mark.skipif(cpu.CXX is None, reason="no clang++ for the host")


@pytest.fixture(scope="module")
def lib_path(tmp_path_factory):
    return cpu.build(tmp_path_factory.mktemp("cpu_build"))


def in_child(fn, *args):
    p = multiprocessing.get_context("fork").Process(target=fn, args=args)
    p.start()
    p.join(300)
    assert p.exitcode == 0, f"exit code {p.exitcode}"


def _decode_before_a_fence(path, dtype, d, heads, n_q, n_rows, counts):
    lib = cpu.load(path)
    rng = np.random.default_rng(n_rows + d)
    Hkv, size = len(counts), 4 if dtype == "f32" else 2
    bf16 = lambda x: (x.view(np.uint32) & 0xffff0000).view(np.float32)  # noqa: E731  (cut off: exact in bf16)
    # a unit's rows end where the next one's begin, the last one's at the fence: the head stride is the first count
    assert all(c == counts[0] for c in counts[:-1])
    kv = []
    for _ in range(2):
        x = bf16(rng.standard_normal((sum(counts), d)).astype(np.float32))
        mem = cpu.fenced(x.size * size)
        mem[:] = (x if dtype == "f32" else (x.view(np.uint32) >> 16).astype(np.uint16)).view(np.uint8).ravel()
        kv.append((x, mem))
    q = bf16(rng.standard_normal((Hkv * heads, n_q, d)).astype(np.float32))
    qm = cpu.aligned(q.size * size)
    qm[:] = (q if dtype == "f32" else (q.view(np.uint32) >> 16).astype(np.uint16)).view(np.uint8).ravel()
    p = B.make_params(batch=1, n_q_heads=Hkv * heads, n_kv_heads=Hkv, head_dim=d, seq_len=n_rows, window=1, dtype=dtype,
                      pool=B.POOL_NONE, pool_kernel=1, budget=n_rows, cap=n_rows)
    need = lib.ckv_decode_workspace_bytes(ctypes.byref(p), n_q, n_rows)
    ws, count = cpu.aligned(max(need, 256)), np.array(counts, np.int32)
    out = np.full((Hkv * heads, n_q, d), np.nan, np.float32)
    lse = np.full((Hkv * heads, n_q), np.nan, np.float32)
    stride = (ctypes.c_int64 * 3)(0, counts[0] * d, d)
    st = lib.ckv_decode_attention(ctypes.byref(p), cpu.ptr(qm), n_q, cpu.ptr(kv[0][1]), cpu.ptr(kv[1][1]), stride, stride, n_rows,
                                  cpu.ptr(count), cpu.ptr(out), cpu.ptr(lse), cpu.ptr(ws), ctypes.c_size_t(need), None)
    assert st == B.CKV_OK
    first = 0
    for g, c in enumerate(counts):
        k, v = (x[first:first + c].astype(np.float64) for x, _ in kv)
        first += c
        for h in range(g * heads, (g + 1) * heads):
            if c == 0:
                assert (out[h] == 0).all() and np.isneginf(lse[h]).all()
                continue
            z = q[h].astype(np.float64) @ k.T / np.sqrt(d)
            top = z.max(1, keepdims=True)
            w = np.exp(z - top)
            np.testing.assert_allclose(lse[h], top[:, 0] + np.log(w.sum(1)), rtol=0, atol=1e-4)
            np.testing.assert_allclose(out[h], (w / w.sum(1, keepdims=True)) @ v, rtol=0, atol=1e-4)


@pytest.mark.parametrize("dtype,d,heads,n_q,n_rows,counts", [
    ("bf16", 128, 4, 1, 544, [33, 70]), ("bf16", 64, 2, 2, 300, [0, 1]), ("bf16", 128, 1, 1, 4096, [64]), ("bf16", 128, 17, 1, 96, [95]),
    ("bf16", 128, 4, 1, 4500, [130, 257]), ("bf16", 64, 3, 1, 8000, [0, 0]), ("bf16", 128, 2, 1, 4200, [4200]),
    ("f32", 64, 2, 1, 544, [33, 70]), ("f32", 128, 4, 1, 4500, [1, 100]),
])
def test_decode_reads_no_row_behind_the_count(lib_path, dtype, d, heads, n_q, n_rows, counts):
    in_child(_decode_before_a_fence, lib_path, dtype, d, heads, n_q, n_rows, counts)
