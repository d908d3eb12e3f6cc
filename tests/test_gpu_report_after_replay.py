"""Reports after the replay of a captured call, where the last call made outside the graph had another tile
shape (a fault list selects the injecting one) or was still to be overtaken by the replay.  The report is that of
the launch that ran last: its events, all of them, and none of an earlier call's."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn, ftdecoupled, ftgemm

pytestmark = pytest.mark.gpu


def _capture(forward):
    """forward(stream) recorded into a graph on a stream of its own, after one eager call there."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        forward(side.cuda_stream)
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        forward(torch.cuda.current_stream().cuda_stream)
    return g


# (m, n, k): tile shape and shares of K without a fault list, report slots without one and with one; test_launch_plans.py
# holds the plan to it
PLANS = {(37, 1000, 1024): ("strip", 1, 8, 4), (700, 1000, 1024): ("strip", 1, 88, 44),      # 32-token tiles against 64-token ones
         (40, 601, 2056): ("strip", 16, 9, 3), (4097, 2050, 264): ("wide", 1, 153, 585)}     # K split; 256-token tiles


@pytest.mark.parametrize("m,n,k", PLANS)
def test_linear(m, n, k):
    print(f"[report after replay] linear {m} x {n} x {k}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    x = torch.randn((m, k), generator=g, device="cuda").half()
    x[:, 3] = 1.0
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).half()
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    ctx = ftgemm.FtGemm(m, n, k)
    ctx.encode_weights(w, stream)
    graph = _capture(lambda st: ctx.forward(x, w, y, None, st))
    ctx.forward(x, w, y, None, stream)
    clean = ctx.report()
    assert clean.n_events == 0
    faults = np.array([(m - 1, n - 1, 30), (m // 2, 0, 30), (0, n // 2, 30)], np.int32)
    for _ in range(3):
        ctx.forward(x, w, y, faults, stream)
        assert ctx.report().n_events == 3
        graph.replay()
        torch.cuda.synchronize()
        rep = ctx.report()
        assert (rep.n_events, rep.n_events_dropped) == (0, 0) and rep.residual_max == clean.residual_max
    # a weight changed after its checksums were taken shows in every token of the replay
    ctx.forward(x, w, y, faults, stream)
    was = w[n // 2, 3].clone()
    w[n // 2, 3] = was + 8.0
    graph.replay()
    torch.cuda.synchronize()
    rep = ctx.report()
    assert rep.n_events_dropped == 0 and rep.event_list() == [(r, n // 2, 1) for r in range(m)]
    w[n // 2, 3] = was
    graph.replay()
    torch.cuda.synchronize()
    assert ctx.report().n_events == 0
    ctx.close()


@pytest.mark.parametrize("seq,head_dim", [(700, 64), (300, 128)])
def test_decoupled(seq, head_dim):
    print(f"[report after replay] decoupled {seq} x {head_dim}", flush=True)
    shape = (1, 3, seq, head_dim)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    o = torch.empty(shape, dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    faults = np.array([(0, 0, 0, seq - 1, 5, 30), (0, 2, 3, seq - 1, 7, 30), (0, 1, 1, 9, 9, 31)], np.int32)
    ctx = ftdecoupled.FtDecoupled(*shape, 0, False)
    graph = _capture(lambda st: ctx.forward(q, k, v, o, None, st))
    for _ in range(3):
        ctx.forward(q, k, v, o, faults, stream)
        rep = ctx.report()
        assert rep.event_set() == {tuple(f[:5]) for f in faults.tolist()} and rep.retried_rows == 1
        graph.replay()
        torch.cuda.synchronize()
        rep = ctx.report()
        assert (rep.n_events, rep.n_events_dropped, rep.retried_rows) == (0, 0, 0)
    ctx.close()
    # with a threshold below the rounding of the products nearly every class is an event: the replay's are those
    # of an eager call on the same inputs, whatever tile shape ran in between
    ctx = ftdecoupled.FtDecoupled(*shape, 0, False, tau_rel=1e-12, max_events=1 << 16)
    graph = _capture(lambda st: ctx.forward(q, k, v, o, None, st))
    ctx.forward(q, k, v, o, None, stream)
    want = ctx.report()
    assert want.n_events_dropped == 0 and want.n_events > 3 * seq
    ctx.forward(q, k, v, o, faults, stream)
    graph.replay()
    torch.cuda.synchronize()
    rep = ctx.report()
    ctx.close()
    assert rep.n_events_dropped == 0 and rep.event_set() == want.event_set() and rep.n_events == want.n_events


def test_captured_and_not_run():
    """Before any launch has run the report is empty."""
    m, n, k = 300, 520, 128
    x, w = (torch.randn((r, k), device="cuda").half() for r in (m, n))
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    q = torch.randn((1, 2, 128, 64), device="cuda").half()
    o = torch.empty((1, 2, 128, 64), dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    for warm in (True, False):                     # (the first use of a kernel is not captured)
        a, b = ftgemm.FtGemm(m, n, k), ftdecoupled.FtDecoupled(1, 2, 128, 64, 0, True)
        a.encode_weights(w, stream)
        if warm:
            a.forward(x, w, y, None, stream)
            b.forward(q, q, q, o, None, stream)
        torch.cuda.synchronize()
        if not warm:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                st = torch.cuda.current_stream().cuda_stream
                a.forward(x, w, y, None, st)
                b.forward(q, q, q, o, None, st)
        rep = a.report()
        assert rep.n_events == 0 and rep.n_events_dropped == 0 and (rep.residual_max > 0) == warm
        rep = b.report()
        assert rep.n_events == 0 and rep.n_events_dropped == 0 and rep.retried_rows == 0
        a.close(), b.close()


@pytest.mark.parametrize("path", ["attention", "linear", "decoupled"])
def test_replay_on_the_default_stream(path):
    """A graph captured on one stream and replayed on the default stream, behind enough work there that the
    replay has not begun when the report is asked for: it waits for the replay and shows it, not the call with
    a fault that was made before."""
    print(f"[report after replay] default stream, {path}", flush=True)
    q, k, v = (torch.randn((1, 2, 200, 64), device="cuda").half() for _ in range(3))
    o = torch.empty((1, 2, 200, 64), dtype=torch.float32, device="cuda")
    x, w = (torch.randn((200, 64), device="cuda").half() for _ in range(2))
    y = torch.empty((200, 200), dtype=torch.float32, device="cuda")
    if path == "attention":
        ctx, operands = ftattn.FtAttn(1, 2, 200, 64, 0, False), (q, k, v, o)
        faults = [(0, 0, ftattn.ST_OACC, 1, 7, 5, 30)]
    elif path == "linear":
        ctx, operands, faults = ftgemm.FtGemm(200, 200, 64), (x, w, y), [(7, 5, 30)]
        ctx.encode_weights(w, torch.cuda.current_stream().cuda_stream)
    else:
        ctx, operands, faults = ftdecoupled.FtDecoupled(1, 2, 200, 64, 0, False), (q, k, v, o), [(0, 0, 3, 7, 5, 30)]
    big = torch.randn((8192, 8192), device="cuda")
    big @ big
    graph = _capture(lambda st: ctx.forward(*operands, None, st))
    side = torch.cuda.Stream()
    for _ in range(2):
        torch.cuda.synchronize()
        ctx.forward(*operands, np.array(faults, np.int32), side.cuda_stream)
        assert ctx.report().n_events == 1
        for _ in range(6):
            big @ big                              # 6.6 TFLOP in fp32: some tens of milliseconds
        graph.replay()
        assert ctx.report().n_events == 0
    ctx.close()
