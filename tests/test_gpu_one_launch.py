"""Both scan passes of a short call in one launch: ranges of one to four key tiles per wave, with and without keys that fill them,
against two launches, bit by bit, and against normalisers by a call of their own and a call that is given them; workgroups that make the missing row sums themselves give
the same bits as workgroups that wait for them; marks of an earlier call, or anything else, in the workspace do no harm."""
import ctypes

import pytest
import torch

import hooks
import oracle
from paper_2602_08686_amd import binding as B
from parity_util import assert_scores_close, f32

pytestmark = pytest.mark.gpu
DEV = "cuda"
NO_ROOM = (1, 4, 4, 128, 16384, 32, B.POOL_AVG, 7)   # more workgroups per unit than the normalisers' place has room for: two launches, by the rule
SHAPES = [  # batch, query heads, KV heads, d, T, W, pooling, kernel
    (1, 32, 32, 128, 4096, 32, B.POOL_MAX, 7), (1, 32, 8, 128, 4097, 32, B.POOL_AVG, 7), (2, 32, 8, 64, 1000, 17, B.POOL_AVG, 5),
    (1, 8, 8, 128, 33, 1, B.POOL_NONE, 1), (1, 4, 1, 128, 20, 4, B.POOL_MAX, 3), (3, 6, 2, 128, 511, 32, B.POOL_AVG, 3), (1, 4, 2, 64, 3001, 64, B.POOL_MAX, 7),
    NO_ROOM, (4, 4, 4, 128, 4096, 32, B.POOL_AVG, 7), (1, 2, 1, 128, 16383, 40, B.POOL_AVG, 7), (16, 8, 8, 128, 777, 32, B.POOL_MAX, 5),
    (1, 4, 1, 128, 10000, 32, B.POOL_AVG, 7), (1, 3, 1, 64, 11111, 32, B.POOL_MAX, 3),   # 40 workgroups and more of a unit
    (2, 8, 1, 128, 65536, 32, B.POOL_AVG, 7), (3, 8, 1, 64, 43001, 32, B.POOL_MAX, 5),   # more than a wave has lanes
    (2, 28, 4, 128, 2600, 32, B.POOL_AVG, 7), (1, 16, 2, 128, 9001, 32, B.POOL_MAX, 5), (1, 10, 2, 64, 3100, 32, B.POOL_AVG, 3),   # 7, 8, 5 tiles
    (1, 32, 8, 128, 1999, 64, B.POOL_AVG, 7), (1, 12, 4, 128, 777, 50, B.POOL_MAX, 7),                                            # 8, 6: two per head
]


def _call(shape, seed):
    batch, hq, kv, d, T, W, pool, kernel = shape
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    q = torch.randn(batch, hq, W, d, generator=g, device=DEV).bfloat16()
    k = (torch.randn(batch, kv, T, d, generator=g, device=DEV) * (1 + 3 * torch.rand(batch, kv, T, 1, generator=g, device=DEV))).bfloat16()
    w_head = 0.5 + torch.rand(1, hq, generator=g, device=DEV)
    p = B.make_params(batch=batch, n_q_heads=hq, n_kv_heads=kv, head_dim=d, seq_len=T, window=W, dtype=torch.bfloat16, pool=pool,
                      pool_kernel=kernel, budget=W, cap=T)
    return p, q, k, w_head


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


def _lse(p, q, k, ws):
    lse = torch.empty(p.batch, p.n_q_heads, p.window, device=DEV)
    B.ckv_window_lse(p, q, k, lse, ws)
    return lse


def _run(p, q, k, w_head, ws, nbytes, lse=None, **form):
    """form: the hooks' two_launches or wait; without it the call that a program makes."""
    lib = B.load()
    n = p.batch * p.n_kv_heads
    u = torch.full((n, max(p.seq_len - p.window, 1)), float("nan"), device=DEV)
    scratch = torch.empty(p.batch, p.n_q_heads, p.seq_len, device=DEV)
    budget, tau = torch.empty(n, dtype=torch.int32, device=DEV), torch.full((p.batch,), float("nan"), device=DEV)
    if form:
        hooks.window_utility(p, q, k, w_head, scratch, u, budget, tau, ws[:nbytes], torch.cuda.current_stream(), **form)
    else:
        st = lib.ckv_window_utility(ctypes.byref(p), _ptr(q), _ptr(k), None, None if lse is None else _ptr(lse), _ptr(w_head), None, None, 0, 0, None, _ptr(scratch),
                                    None, _ptr(u), _ptr(budget), _ptr(tau), _ptr(ws), nbytes, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == B.CKV_OK
    torch.cuda.synchronize()
    assert (tau == 0).all() and (budget == min(p.budget_per_kv_head, p.seq_len)).all()
    return u


def _no_marks(p, ws):
    """The call took its marks back."""
    at, n = hooks.marks(p)
    assert (n > 0) == (p.seq_len != NO_ROOM[4]) and (ws[at:at + 8 * n].view(torch.int64) == 0).all()


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_one_launch_matches_two(shape):
    print("case", shape, flush=True)
    p, q, k, w_head = _call(shape, 1)
    whole = B.ckv_workspace_bytes(p)
    ws = torch.full((whole,), 0x5A, dtype=torch.uint8, device=DEV)
    two = _run(p, q, k, w_head, ws, whole, lse=_lse(p, q, k, ws))
    one = _run(p, q, k, w_head, ws, whole)
    assert torch.equal(_run(p, q, k, w_head, ws, whole, two_launches=True), one)
    # given normalisers: the same sums in the same order but for what is finished behind the rounds: roundings of exponents of a few tens
    torch.testing.assert_close(one, two, rtol=1e-5, atol=0)
    for wait in (0, 1, 3000):
        ws.random_(0, 256)
        assert torch.equal(_run(p, q, k, w_head, ws, whole, wait=wait), one), wait
        _no_marks(p, ws)


@pytest.mark.parametrize("shape", SHAPES + [(1, 1, 1, 128, 2000, 100, B.POOL_NONE, 1), (1, 2, 2, 64, 5000, 128, B.POOL_NONE, 1)],
                         ids=lambda s: "-".join(map(str, s)))
def test_scores_in_one_launch_match_two(shape):
    print("case", shape, flush=True)
    p, q, k, _ = _call(shape, 3)
    ws = torch.full((B.ckv_workspace_bytes(p),), 0xA5, dtype=torch.uint8, device=DEV)
    outs = []
    for lse in (_lse(p, q, k, ws), None, None):
        scores = torch.full((p.batch, p.n_q_heads, p.seq_len), float("nan"), device=DEV)
        B.ckv_window_scores(p, q, k, None, lse, scores, None, ws)
        outs.append(scores)
    torch.testing.assert_close(outs[1], outs[0], rtol=1e-5, atol=1e-30)
    assert torch.equal(outs[1], outs[2])
    for form in ({"two_launches": True}, {"wait": 0}, {"wait": 1}):
        scores = torch.full((p.batch, p.n_q_heads, p.seq_len), float("nan"), device=DEV)
        ws.random_(0, 256)
        hooks.window_scores(p, q, k, scores, ws, torch.cuda.current_stream(), **form)
        assert torch.equal(scores, outs[1]), form
        if "wait" in form:
            _no_marks(p, ws)
    torch.testing.assert_close(outs[1].double().sum(-1), torch.full((p.batch, p.n_q_heads), float(p.seq_len), dtype=torch.float64, device=DEV),
                               rtol=1e-4, atol=0)


def _graph_us(p, q, k, w_head, **form):
    """us per call of 20 in a graph, the least of five replays."""
    n, stream = p.batch * p.n_kv_heads, torch.cuda.Stream()
    out = dict(scratch=torch.empty(p.batch, p.n_q_heads, p.seq_len, device=DEV), utility=torch.empty(n, p.seq_len - p.window, device=DEV),
               budget=torch.empty(n, dtype=torch.int32, device=DEV), tau=torch.empty(p.batch, device=DEV),
               ws=torch.zeros(B.ckv_workspace_bytes(p), dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    hooks.window_utility(p, q, k, w_head, stream=stream, **out, **form)
    torch.cuda.synchronize()
    graph, times = torch.cuda.CUDAGraph(), []
    with torch.cuda.graph(graph, stream=stream):
        for _ in range(20):
            hooks.window_utility(p, q, k, w_head, stream=stream, **out, **form)
    for _ in range(5):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        graph.replay()
        end.record()
        torch.cuda.synchronize()
        times.append(begin.elapsed_time(end) * 1e3 / 20)
    return min(times), out["utility"]


@pytest.mark.parametrize("shape", [(2, 8, 1, 128, 65536, 32, B.POOL_AVG, 7), (1, 32, 8, 128, 8192, 32, B.POOL_AVG, 7)], ids=lambda s: "-".join(map(str, s)))
def test_workgroups_that_do_not_wait_share_the_missing_ranges(shape):
    """Nobody waits: what a launch beside a busy stream comes to. With every missing range made by every workgroup it took 31 and 8 times as long as
    two launches."""
    print("case", shape, flush=True)
    p, q, k, w_head = _call(shape, 11)
    two, want = _graph_us(p, q, k, w_head, two_launches=True)
    none, got = _graph_us(p, q, k, w_head, wait=0)
    assert torch.equal(got, want)
    assert none < 4 * two, (none, two)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("T,W", [(1, 1), (9, 4), (20, 4), (31, 9), (32, 9), (33, 33)])
def test_sequences_of_a_tile_or_less(T, W, heads, d):
    """The only key tile's loads are the last that a wave waits for, however many images they fill: with five and more query tiles fewer than
    for a longer sequence. The ring holds another call's keys before."""
    print("case", T, W, heads, d, flush=True)
    batch, kv = 3, 2
    p, q, k, w_head = _call((batch, heads * kv, kv, d, T, W, B.POOL_MAX, 3), 7 * T + heads)
    other, oq, ok, ow = _call((64, heads, 1, d, 512, 32, B.POOL_NONE, 1), 5)
    ws = torch.zeros(max(B.ckv_workspace_bytes(p), B.ckv_workspace_bytes(other)), dtype=torch.uint8, device=DEV)
    outs = []
    for lse in (_lse(p, q, k, ws), None, None):
        _run(other, oq, ok, ow, ws, ws.numel())
        scores = torch.full((batch, heads * kv, T), float("nan"), device=DEV)
        B.ckv_window_scores(p, q, k, None, lse, scores, None, ws)
        outs.append(scores)
    torch.testing.assert_close(outs[1], outs[0], rtol=1e-5, atol=1e-30)
    assert torch.equal(outs[1], outs[2])
    want = oracle.window_scores(f32(q), f32(k))
    assert_scores_close(outs[1].cpu().numpy(), want)
    if T > W:
        two = _run(p, q, k, w_head, ws, ws.numel(), lse=_lse(p, q, k, ws))
        for form in ({}, {"wait": 0}):
            _run(other, oq, ok, ow, ws, ws.numel())
            one = _run(p, q, k, w_head, ws, ws.numel(), **form)
            torch.testing.assert_close(one, two, rtol=1e-5, atol=0)
            ref = oracle.utility(want, W, kv, B.POOL_MAX, 3, f32(w_head[0]))
            assert_scores_close(one.cpu().numpy().reshape(ref.shape), ref, "utility")


@pytest.mark.parametrize("wait", [hooks.RULE, 0])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[1], SHAPES[5], (2, 8, 1, 128, 65536, 32, B.POOL_AVG, 7)], ids=lambda s: "-".join(map(str, s)))
def test_replays_with_other_inputs(shape, wait):
    """A replayed launch has the marks' tag of the first one: none of them may be left. One call in the graph, so that no other one's tag
    lies over its marks before it comes again."""
    print("case", shape, wait, flush=True)
    p, q, k, w_head = _call(shape, 1)
    ws = torch.zeros(B.ckv_workspace_bytes(p), dtype=torch.uint8, device=DEV)
    n, stream = p.batch * p.n_kv_heads, torch.cuda.Stream()
    u = torch.empty(n, p.seq_len - p.window, device=DEV)
    scratch = torch.empty(p.batch, p.n_q_heads, p.seq_len, device=DEV)
    budget, tau = torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(p.batch, device=DEV)
    torch.cuda.synchronize()
    hooks.window_utility(p, q, k, w_head, scratch, u, budget, tau, ws, stream, wait=wait)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        hooks.window_utility(p, q, k, w_head, scratch, u, budget, tau, ws, stream, wait=wait)
    for seed in range(2, 7):
        _, q2, k2, _ = _call(shape, seed)
        q.copy_(q2)
        k.copy_(k2)
        u.zero_()
        graph.replay()
        torch.cuda.synchronize()
        _no_marks(p, ws)
        got = u.clone()
        assert torch.equal(got, _run(p, q, k, w_head, torch.zeros_like(ws), ws.numel(), two_launches=True).view_as(got)), seed


def test_streams_and_a_kernel_that_holds_the_chip():
    """Short calls on four streams, each with buffers of its own, beside matrix products that fill the chip: workgroups of a launch start far
    apart, some wait in vain and make the missing sums themselves; all results are those of a call by itself."""
    shape = SHAPES[0]
    calls = [_call(shape, 20 + i) for i in range(4)]
    nbytes = B.ckv_workspace_bytes(calls[0][0])
    want = [_run(*c, torch.zeros(nbytes, dtype=torch.uint8, device=DEV), nbytes) for c in calls]
    big = torch.randn(8192, 8192, device=DEV).bfloat16()
    streams = [torch.cuda.Stream() for _ in calls]
    state = []
    for p, q, k, w_head in calls:
        n = p.batch * p.n_kv_heads
        state.append((torch.zeros(nbytes, dtype=torch.uint8, device=DEV), torch.empty(p.batch, p.n_q_heads, p.seq_len, device=DEV),
                      torch.zeros(30, n, p.seq_len - p.window, device=DEV), torch.empty(n, dtype=torch.int32, device=DEV),
                      torch.empty(p.batch, device=DEV)))
    torch.cuda.synchronize()
    for r in range(30):
        if r % 10 == 0:
            big @ big
        for (p, q, k, w_head), (ws, scratch, u, budget, tau), stream in zip(calls, state, streams):
            B.ckv_window_utility(p, q, k, None, None, w_head, None, None, 0, 0, None, scratch, None, u[r], budget, tau, ws, stream)
    torch.cuda.synchronize()
    for w, (ws, _, u, _, _) in zip(want, state):
        _no_marks(calls[0][0], ws)
        for r in range(30):
            assert torch.equal(u[r], w.view_as(u[r])), r
