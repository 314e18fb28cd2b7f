"""Kernels on the host CPU, where an access out of bounds ends a child process instead of a GPU: decode attention reads no
row behind the count (the memory there has no access), the selection stays inside its buffers whatever another stream
writes over its input meanwhile, and with a workspace that was sized for another budget, and the gather copies every row of lists
of any length, each once."""
import ctypes
import multiprocessing

import numpy as np
import pytest

import cpu_build as cpu
import oracle
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
    ("bf16", 128, 1, 1, 300, [40] * 128 + [17]), ("bf16", 128, 1, 1, 4100, [3] * 132 + [70]),   # one column: the vector kernel
    ("f32", 64, 2, 1, 544, [33, 70]), ("f32", 128, 4, 1, 4500, [1, 100]),
])
def test_decode_reads_no_row_behind_the_count(lib_path, dtype, d, heads, n_q, n_rows, counts):
    in_child(_decode_before_a_fence, lib_path, dtype, d, heads, n_q, n_rows, counts)


def _select_while_the_input_changes(path, P, nominal, budgets, with_workspace, one_read):
    lib = cpu.load(path)
    W, Hkv, guard = 4, 2, 4096
    rng = np.random.default_rng(P)
    before = (1.0 + 0.08 * np.abs(rng.standard_normal((1, Hkv, P)))).astype(np.float32)
    u = before.copy()
    cap = min(P + W, max(nominal * Hkv - W, max(budgets)))
    p = B.make_params(batch=1, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W, dtype="bf16",
                      pool=B.POOL_NONE, pool_kernel=1, budget=nominal, cap=cap)
    need = lib.ckv_workspace_bytes(ctypes.byref(p))
    ws = cpu.aligned(need) if with_workspace else None
    budget, tau = np.array([budgets], np.int32), np.zeros(1, np.float32)
    changes = {"zeros": np.zeros_like(u), "large": np.full_like(u, 3e38), "nan": np.full_like(u, np.nan),
               "mixed": np.where(rng.random(u.shape) < 0.5, u, 1e30 * u).astype(np.float32)}
    for name, after in changes.items():
        for at in (0, 3):  # barriers: behind the first read, and inside the search on one of the forms that read several times
            def write(block, barrier):
                if barrier in (-1, at):
                    u[:] = before if barrier < 0 else after

            hook = cpu.HOOK(write)
            lib.emu_set_hook(hook)
            idx, count = np.full(2 * guard + Hkv * cap, -1, np.int32), np.full(2 * guard + Hkv, -1, np.int32)
            st = lib.ckv_select_topk(ctypes.byref(p), cpu.ptr(u), cpu.ptr(budget), cpu.ptr(tau), cpu.ptr(idx[guard:]), cpu.ptr(count[guard:]),
                                     cpu.ptr(ws), ctypes.c_size_t(need), None)
            lib.emu_set_hook(ctypes.cast(None, cpu.HOOK))
            assert st == B.CKV_OK
            for a in (idx, count):
                assert (a[:guard] == -1).all() and (a[-guard:] == -1).all(), (name, at)
            lists, counts = idx[guard:-guard].reshape(Hkv, cap), count[guard:-guard]
            assert ((lists >= -1) & (lists < P + W)).all(), (name, at)
            for h in range(Hkv):
                assert W <= counts[h] <= min(cap, budgets[h]) and (lists[h, counts[h]:] == -1).all(), (name, at)
                if one_read:  # the decisions rest on one read: whatever it saw, every entry that is counted was written
                    assert (lists[h, :counts[h]] >= 0).all() and counts[h] == budgets[h], (name, at)


@pytest.mark.parametrize("P,nominal,budgets,with_workspace,one_read", [
    (8200, 200, [200, 380], False, True),       # 16 positions per thread, the list
    (20001, 500, [500, 900], False, True),      # 32
    (33000, 1600, [1600, 700], False, True),    # 64
    (35001, 1600, [1600, 700], True, True),     # slices of 16 per thread, merge
    (35001, 4000, [4004, 700], True, False),    # split: several reads
    (66001, 300, [300, 80], False, False),      # streaming: several reads
])
def test_selection_stays_inside_its_buffers_while_the_input_changes(lib_path, P, nominal, budgets, with_workspace, one_read):
    in_child(_select_while_the_input_changes, lib_path, P, nominal, budgets, with_workspace, one_read)


def _select_with_the_workspace_of_another_budget(path, P, budgets):
    lib = cpu.load(path)
    W, Hkv = 4, 2
    rng = np.random.default_rng(P)
    u = np.exp(0.6 * rng.standard_normal((1, Hkv, P))).astype(np.float32)
    tau = np.zeros(1, np.float32)

    def params(b):
        return B.make_params(batch=1, n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W, dtype="bf16",
                             pool=B.POOL_NONE, pool_kernel=1, budget=b, cap=min(P + W, b * Hkv - (Hkv - 1) * W))

    for sized_for in budgets:
        need = lib.ckv_workspace_bytes(ctypes.byref(params(sized_for)))
        for b in budgets:
            p = params(b)
            ws = cpu.fenced(need)   # a multiple of 256 before a page's end: aligned
            idx, count = np.full((1, Hkv, p.cap), -1, np.int32), np.zeros((1, Hkv), np.int32)
            budget = np.array([[b, min(p.cap, b + 7)]], np.int32)
            st = lib.ckv_select_topk(ctypes.byref(p), cpu.ptr(u), cpu.ptr(budget), cpu.ptr(tau), cpu.ptr(idx), cpu.ptr(count),
                                     cpu.ptr(ws), ctypes.c_size_t(need), None)
            assert st == B.CKV_OK, (sized_for, b, st)
            oi, oc = oracle.select(u, tau, budget, W, p.cap)
            np.testing.assert_array_equal(count, oc)
            np.testing.assert_array_equal(idx, oi)


def test_one_workspace_serves_every_budget_of_its_shape(lib_path):
    in_child(_select_with_the_workspace_of_another_budget, lib_path, 40000, (20, 600, 5000))


def _gather_lists(path, dtype, d, batch, kv, T, budget, cap, kind, shared):
    lib = cpu.load(path)
    rng = np.random.default_rng(T + d)
    size, lists = d * (4 if dtype == "f32" else 2), (batch, 1 if shared else kv)
    total = budget * lists[1]
    count = {"even": np.full(lists, min(budget, cap)), "one": np.where(np.arange(lists[1]) == lists[1] - 1, cap, rng.integers(0, 3, lists)),
             "first": np.where(np.arange(lists[1]) == 0, cap, np.zeros(lists)), "all_full": np.full(lists, cap), "beyond_cap": np.full(lists, cap + 9),
             "skewed": np.minimum(cap, (rng.dirichlet(np.full(lists[1], 0.3), batch) * total).astype(int)), "empty": np.zeros(lists),
             "negative": np.full(lists, -5)}[kind].astype(np.int32)
    idx = rng.integers(0, T, lists + (cap,)).astype(np.int32)
    idx[..., ::7] = np.where(rng.random(idx[..., ::7].shape) < 0.2, rng.choice([-1, T, 1 << 30], idx[..., ::7].shape), idx[..., ::7])
    src = [rng.integers(0, 256, (batch, kv, T, size)).astype(np.uint8) for _ in range(2)]
    mem, outs = [], []
    for x in src:
        m, o = cpu.fenced(x.size), cpu.fenced(batch * kv * cap * size)
        m[:], o[:] = x.ravel(), 7
        mem.append(m)
        outs.append(o)
    im = cpu.fenced(idx.nbytes)
    im[:] = idx.view(np.uint8).ravel()
    cm = cpu.fenced(count.nbytes)
    cm[:] = count.view(np.uint8).ravel()
    p = B.make_params(batch=batch, n_q_heads=kv, n_kv_heads=kv, head_dim=d, seq_len=T, window=1, dtype=dtype, pool=B.POOL_NONE,
                      pool_kernel=1, budget=budget, cap=cap)
    call = lib.ckv_compact_kv_shared if shared else lib.ckv_compact_kv
    assert call(ctypes.byref(p), cpu.ptr(mem[0]), cpu.ptr(mem[1]), cpu.ptr(im), cpu.ptr(cm), cpu.ptr(outs[0]), cpu.ptr(outs[1]), None) == B.CKV_OK
    for x, o in zip(src, outs):
        got = o.reshape(batch, kv, cap, size)
        for b in range(batch):
            for g in range(kv):
                lst = (b, 0) if shared else (b, g)
                want = np.full((cap, size), 7, np.uint8)
                n = max(0, min(int(count[lst]), cap))
                ok = np.flatnonzero((idx[lst][:n] >= 0) & (idx[lst][:n] < T))
                want[ok] = x[b, g][idx[lst][ok]]
                np.testing.assert_array_equal(got[b, g], want)


@pytest.mark.parametrize("kind", ["even", "one", "first", "all_full", "beyond_cap", "skewed", "empty", "negative"])
@pytest.mark.parametrize("dtype,d,batch,kv,T,budget,shared", [
    ("bf16", 128, 2, 8, 700, 40, False), ("bf16", 64, 1, 32, 900, 33, False), ("f32", 128, 1, 3, 2100, 9, False),
    ("bf16", 64, 1, 70, 300, 5, False),     # more heads than lanes
    ("f32", 64, 3, 4, 500, 20, True), ("bf16", 128, 1, 1, 400, 16, False),
])
def test_gather_copies_lists_of_any_length(lib_path, dtype, d, batch, kv, T, budget, shared, kind):
    cap = T if kind in ("all_full", "beyond_cap") else min(T, budget * kv)
    in_child(_gather_lists, lib_path, dtype, d, batch, kv, T, budget, cap, kind, shared)
