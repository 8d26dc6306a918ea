"""The attention call in one launch (workgroups exchange their partials and merge them) against the same call in two: the
same partials are folded in the same order, so every output has the same bits."""
import ctypes
import time

import pytest
import torch

from paper_2502_20330_amd import binding
from paper_2502_20330_amd.binding import OPT_ATTN_WAIT_US, Rapid

pytestmark = pytest.mark.gpu


def _case(B, Q, Hq, Hkv, d, lens, gammas, page=0, layout="head", seed=0, max_ctx=None):
    g = torch.Generator(device="cuda").manual_seed(seed)
    max_ctx = max_ctx or max(max(lens), Q)
    q = torch.randn(B, Q, Hq, d, device="cuda", generator=g).bfloat16()
    table = None
    if page:
        per = -(-max_ctx // page)
        table = torch.randperm(B * per, device="cuda", generator=g).to(torch.int32).view(B, per)
        shape = (B * per, page, Hkv, d)
    else:
        shape = (B, max_ctx, Hkv, d)
    if layout == "head":
        k, v = (torch.randn(shape[0], shape[2], shape[1], d, device="cuda", generator=g).bfloat16().permute(0, 2, 1, 3) for _ in "kv")
    else:
        k, v = (torch.randn(shape, device="cuda", generator=g).bfloat16() for _ in "kv")
    return dict(q=q, k=k, v=v, lens=torch.tensor(lens, dtype=torch.int32, device="cuda"),
                gammas=None if gammas is None else torch.tensor(gammas, dtype=torch.int32, device="cuda"), table=table, max_ctx=max_ctx)


def _two(r, c, chunk=0):
    s = r.attn_shape(c["q"], c["k"], c["max_ctx"], page_table=c["table"], chunk_tokens=chunk)
    out = torch.full_like(c["q"], float("nan"))
    lse = torch.full((s.batch, s.n_q_heads, s.q_max), float("nan"), device="cuda")
    ws = torch.empty(r.lib.rapid_verify_attn_workspace_bytes(r._ctx, ctypes.byref(s)), dtype=torch.uint8, device="cuda")
    p = lambda t: None if t is None else t.data_ptr()
    rc = r.lib.rapid_verify_attn(r._ctx, ctypes.byref(s), p(c["q"]), p(c["k"]), p(c["v"]), p(c["lens"]), p(c["gammas"]), p(c["table"]),
                                 p(out), p(lse), p(ws), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    return out, lse


def _one(r, c, chunk=0):
    out = torch.full_like(c["q"], float("nan"))
    lse = torch.full((c["q"].shape[0], c["q"].shape[2], c["q"].shape[1]), float("nan"), device="cuda")
    r.rapid_verify_attn(c["q"], c["k"], c["v"], c["lens"], gammas=c["gammas"], page_table=c["table"], max_ctx=c["max_ctx"], out=out,
                        lse_out=lse, chunk_tokens=chunk)
    return out, lse


def _same(x, y):
    for a, b in zip(x, y):
        assert torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                           b.view(torch.int16 if b.dtype == torch.bfloat16 else torch.int32))


# B, Q, Hq, Hkv, d, lens, gammas, page, layout: one split and several, up to the 32 that run in one launch; shares of less than a
# row and of several rows, up to the 256 elements that they may have, more shares than elements to share; splits and whole sequences without tokens, nearly
# all of a sequence's splits among them; one and two row blocks; grids of up to 64 workgroups with heads of 128, 128 with heads of 64
SHAPES = [
    (1, 1, 4, 4, 64, [1], None, 0, "head"),
    (1, 1, 1, 1, 64, [8192], None, 0, "head"),
    (1, 5, 4, 1, 64, [2048], None, 0, "token"),
    (1, 4, 1, 1, 64, [200], None, 0, "head"),
    (1, 2, 4, 1, 128, [1000], None, 0, "head"),
    (1, 1, 32, 8, 128, [2048], None, 0, "head"),
    (1, 4, 8, 2, 128, [8192], None, 0, "head"),
    (1, 3, 32, 8, 128, [1900], [1], 16, "head"),
    (1, 2, 28, 4, 128, [4065], None, 0, "token"),
    (1, 5, 3, 1, 128, [7300], None, 0, "token"),
    (1, 4, 8, 1, 64, [8192], [2], 64, "head"),
    (2, 2, 32, 4, 128, [2000, 700], [1, 0], 0, "head"),
    (3, 4, 16, 4, 64, [2500, 0, 4], [3, 3, 3], 16, "head"),
    (8, 8, 8, 4, 64, [1024] * 8, None, 0, "head"),
    (8, 3, 8, 4, 64, [513] * 8, [0, 1, 2, 2] * 2, 0, "token"),
    (32, 2, 8, 4, 64, [33] * 32, [0, 1, 1, 1] * 8, 0, "token"),
    (2, 4, 8, 1, 64, [8192, 100], None, 0, "head"),
    (2, 2, 8, 1, 128, [4096, 0], [1, 0], 0, "token"),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_shapes_run_in_one_launch(shape):
    r = Rapid(0)
    c = _case(*shape)
    s = r.attn_shape(c["q"], c["k"], c["max_ctx"], page_table=c["table"])
    assert r.lib.rapid_verify_attn_exchange_bytes(r._ctx, ctypes.byref(s)) > 0
    _one(r, c)
    assert r._ws is None                               # no workspace for a second launch


@pytest.mark.parametrize("shape", SHAPES)
def test_one_launch_has_the_bits_of_two(shape):
    r = Rapid(0)
    c = _case(*shape)
    for chunk in (0, 384):
        want = _two(r, c, chunk)
        for wait in (100, 100, 0, 1, 3, 100):          # (short bounds: shares that are not there yet are left to the last workgroup of their head)
            r.set_option(OPT_ATTN_WAIT_US, wait)
            _same(_one(r, c, chunk), want)


def test_calls_of_many_shapes_and_replays_share_one_exchange():
    r = Rapid(0)
    cases = [_case(*s, seed=i) for i, s in enumerate(SHAPES)]
    want = [_two(r, c) for c in cases]
    for c in cases:
        _one(r, c)                                     # the exchange has its size from here on
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        got = [_one(r, c) for c in cases[:6]]
    order = torch.Generator().manual_seed(1)
    for _ in range(6):
        for o, l in got:
            o.fill_(float("nan")), l.fill_(float("nan"))
        graph.replay()
        for i in torch.randint(len(cases), (8,), generator=order).tolist():
            _same(_one(r, cases[i]), want[i])
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            _same(g, w)


def test_every_copy_of_the_calls_number_moves_by_one():
    r = Rapid(0)
    cases = [_case(*s) for s in SHAPES]
    for c in cases:
        _one(r, c)
    n = int(r._ws_exchange[:4].view(torch.int32))
    for i, c in enumerate(cases * 2):
        r.set_option(OPT_ATTN_WAIT_US, 100 if i % 3 else 0)
        _one(r, c)
        n += 1
        assert r._ws_exchange[:1024].view(torch.int32).unique().tolist() == [n]


# 4 kv heads in 8 splits, and as many words of one head in 32: the words of the second shape's later splits are those of other heads of the first
ACROSS = [(1, 1, 4, 4, 64, [2048], None, 0, "head"), (1, 1, 1, 1, 64, [8192], None, 0, "head")]


def _set_calls(r, values):
    r._ws_exchange[:1024].view(torch.int32).copy_(torch.as_tensor(values, dtype=torch.int64).to(torch.int32))


def test_the_number_of_the_call_skips_0():
    """0 is the tag of words that nobody has written: a call under it would take them for its partners'.  The third call after the
    copies were set is the one that would have it, the first on most of its part of the memory; its last split holds 8 tokens and looks for
    the words of the others long before they are there."""
    for seed in range(3):
        r = Rapid(0)
        short, long = _case(1, 1, 1, 1, 64, [64], None, seed=seed), _case(1, 1, 4, 1, 64, [8200], None, seed=seed)
        want = {False: _two(r, short, 4096), True: _two(r, long, 4096)}
        _one(r, short, 4096)
        _set_calls(r, [0xfffffffd - (1 << 32)] * 256)
        for now in (False, False, True, False, True):
            _same(_one(r, long if now else short, 4096), want[now])
        assert r._ws_exchange[:1024].view(torch.int32).unique().tolist() == [3]


def test_clearing_mends_what_overlapping_calls_leave():
    """Unequal copies of the number, and words of other heads under the tags that the next calls have."""
    r = Rapid(0)
    cases = [_case(*s, seed=i) for i, s in enumerate(ACROSS)]
    want = [_two(r, c) for c in cases]
    for trial in range(8):
        _one(r, cases[0])
        n = int(r._ws_exchange[:4].view(torch.int32))
        _set_calls(r, [n + (t + trial) % 5 for t in range(256)])
        _one(r, cases[0])
        r.clear_exchange()
        for _ in range(3):
            for c, w in zip(cases[::-1], want[::-1]):
                _same(_one(r, c), w)
        assert r._ws_exchange[:1024].view(torch.int32).unique().tolist() == [6]


@pytest.mark.parametrize("d,hkv", [(64, 8), (128, 4)])
def test_sequences_without_tokens_many_times(d, hkv):
    """Workgroups without tokens publish at once, so that their team's number moves as early as it ever does: it still moves by one a call,
    and every share is merged."""
    r = Rapid(0)
    c = _case(4, 2, hkv, hkv, d, [0, 3, 0, 0], None, max_ctx=1024)
    want = _two(r, c)
    _one(r, c)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        got = [_one(r, c) for _ in range(32)]
    for _ in range(20):
        graph.replay()
        torch.cuda.synchronize()
        for g in got:
            _same(g, want)
    assert r._ws_exchange[:1024].view(torch.int32).unique().tolist() == [1 + 32 * 20]


def test_missing_or_small_exchange_is_refused_and_none_takes_two_launches():
    r = Rapid(0)
    c = _case(*SHAPES[2])
    s = r.attn_shape(c["q"], c["k"], c["max_ctx"])
    need = r.lib.rapid_verify_attn_exchange_bytes(r._ctx, ctypes.byref(s))
    out = torch.empty_like(c["q"])
    x = torch.zeros(need + 256, dtype=torch.uint8, device="cuda")
    ws = torch.empty(r.lib.rapid_verify_attn_workspace_bytes(r._ctx, ctypes.byref(s)), dtype=torch.uint8, device="cuda")

    def call(xp, xn, wp, wn):
        return r.lib.rapid_verify_attn_exchange(r._ctx, ctypes.byref(s), c["q"].data_ptr(), c["k"].data_ptr(), c["v"].data_ptr(),
                                                c["lens"].data_ptr(), None, None, out.data_ptr(), None, xp, xn, wp, wn,
                                                torch.cuda.current_stream().cuda_stream)
    assert call(x.data_ptr(), need - 1, ws.data_ptr(), ws.numel()) == binding.RAPID_EWORKSPACE
    assert call(x.data_ptr() + 16, need, ws.data_ptr(), ws.numel()) == binding.RAPID_EWORKSPACE
    assert call(None, 0, None, 0) == binding.RAPID_EWORKSPACE
    assert call(x.data_ptr(), need, None, 0) == 0
    _same((out,), (_two(r, c)[0],))
    assert call(None, 0, ws.data_ptr(), ws.numel()) == 0
    _same((out,), (_two(r, c)[0],))


@pytest.mark.parametrize("shape", [(1, 5, 4, 1, 128, [2048], None), (1, 9, 4, 1, 64, [2048], None), (1, 1, 4, 1, 64, [65536], None),
                                   (1, 1, 32, 8, 128, [2049], None), (1, 1, 32, 8, 128, [8192], None), (33, 1, 8, 4, 64, [64] * 33, None),
                                   (1, 4, 8, 1, 64, [200], None), (1, 2, 8, 1, 128, [1700], None)])
def test_shapes_that_stay_at_two_launches(shape):
    """More rows, more than 32 splits, more than a quarter of the workgroups that the chip holds, more than 256 elements a share: no exchange memory is asked for, and none is
    needed."""
    r = Rapid(0)
    c = _case(*shape)
    s = r.attn_shape(c["q"], c["k"], c["max_ctx"])
    assert r.lib.rapid_verify_attn_exchange_bytes(r._ctx, ctypes.byref(s)) == 0
    got = _one(r, c)
    assert r._ws is not None and bool(got[0].float().isfinite().all())


def _launches(r, call):
    """Kernels that a call enqueues: nodes of its recorded graph."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        call()
    n = ctypes.c_size_t(0)
    assert r.lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


def test_launches_of_the_entries():
    """One launch with exchange memory, two without; the static entry has none, as nobody could clear it after a race."""
    r = Rapid(0)
    c = _case(*SHAPES[5])
    out = torch.empty_like(c["q"])
    call = dict(max_ctx=c["max_ctx"], out=out)
    eager = lambda: r.rapid_verify_attn(c["q"], c["k"], c["v"], c["lens"], **call)
    assert _launches(r, eager) == 2                    # an object's first call, inside a capture: no exchange memory yet
    eager()
    assert _launches(r, eager) == 1
    assert _launches(r, lambda: r.rapid_verify_attn_static(c["q"], c["k"], c["v"], c["lens"], **call)) == 2


@pytest.mark.parametrize("shape", [SHAPES[2], SHAPES[5], SHAPES[6]])
def test_first_call_of_an_object_inside_a_capture(shape):
    """Nothing can be cleared there, so the call takes two launches; the next eager one makes the exchange memory and takes one.  The
    splits are the same."""
    r = Rapid(0)
    c = _case(*shape)
    want = _two(r, c)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        got = _one(r, c)
    assert r._ws_exchange is None
    for _ in range(3):
        _same(_one(r, c), want)
        graph.replay()
        _same(got, want)


@pytest.mark.parametrize("shape", [(1, 4, 32, 8, 128, [2048], None), (1, 4, 32, 8, 128, [8192], None), (4, 2, 16, 8, 64, [1024] * 4, None),
                                   (1, 4, 16, 8, 64, [8192], None)])
def test_chains_on_four_streams_do_not_wait_for_one_another(shape):
    """Four objects, a recorded chain of calls each, replayed side by side, with a bound of the waits that is far longer than all of them
    take: no workgroup may keep another one's partner off the chip."""
    objects, graphs, outs, want = [Rapid(0) for _ in range(4)], [], [], []
    cases = [_case(*shape, seed=i) for i in range(4)]  # (kept: the graphs read them)
    for r, c in zip(objects, cases):
        want.append(_one(r, c))
        r.set_option(OPT_ATTN_WAIT_US, 100000)
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            outs.append([_one(r, c) for _ in range(8)])
        graphs.append(graph)
        graph.replay()
    streams = [torch.cuda.Stream() for _ in objects]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(3):
        for s, graph in zip(streams, graphs):
            with torch.cuda.stream(s):
                graph.replay()
    torch.cuda.synchronize()
    took = time.perf_counter() - t0
    for got, w in zip(outs, want):
        for g in got:
            _same(g, w)
    assert took < 0.1, took


@pytest.mark.parametrize("d,hq,L", [(64, 4, 8200), (128, 4, 8200), (64, 32, 7 * 4096 + 8)])
def test_shares_are_left_to_the_last_workgroup(d, hq, L):
    """Splits of 4096 tokens and a last one of 8: with one look the workgroup of the last one leaves its share, marked with the call's number, and
    others merge it.  With a bound of 100 ms it waits, and no share is marked."""
    r = Rapid(0)
    c = _case(1, 1, hq, 1, d, [L], None)
    want = _two(r, c, 4096)
    for wait in (0, 100000, 1, 100000, 0):
        r.set_option(OPT_ATTN_WAIT_US, wait)
        _same(_one(r, c, 4096), want)
        words = r._ws_exchange[:1024 + 128].view(torch.int32).tolist()
        tag, marks = words[0], words[256:256 + -(-L // 4096)]
        assert marks[-1] == tag if wait < 100000 else tag not in marks, (wait, tag, marks)


def test_two_objects_on_two_streams():
    """Each has exchange memory of its own.  Recorded chains of calls, replayed side by side so that their kernels run back to back, and
    one with workgroups that leave their shares to others."""
    cases = [_case(*SHAPES[5]), _case(*SHAPES[6], seed=1)]
    objects = [Rapid(0), Rapid(0)]
    want = [_one(r, c) for r, c in zip(objects, cases)]
    for wait in (100, 0):
        objects[1].set_option(OPT_ATTN_WAIT_US, wait)
        graphs, got = [torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()], []
        for graph, r, c in zip(graphs, objects, cases):
            torch.cuda.synchronize()
            with torch.cuda.graph(graph):
                got.append([_one(r, c) for _ in range(20)])
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        torch.cuda.synchronize()
        for _ in range(4):
            for o, l in got[0] + got[1]:
                o.fill_(float("nan")), l.fill_(float("nan"))
            torch.cuda.synchronize()
            for s, graph in zip(streams, graphs):
                with torch.cuda.stream(s):
                    graph.replay()
            torch.cuda.synchronize()
            for i in range(2):
                for g in got[i]:
                    _same(g, want[i])
