"""Calls in one launch: heads of one row tile whose key and value tiles fit the ring of the fused kernel (128 keys at head_dim 64,
192 at head_dim 128) are encoded by its workgroups.  At the edges of tiles and of that rule: the output, bit for bit, and the
report are those of a timed call, which keeps the launch that encodes; a report is of its own call, whatever the one before counted."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import efta_oracle as eorc
from paper_2504_02211_amd import ftattn, synth
import ft_harness as H

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1, 64), (2, 3, 63, 64), (1, 5, 64, 64), (3, 7, 65, 64), (1, 2, 127, 64), (16, 20, 128, 64), (1, 2, 129, 64),
          (1, 1, 1, 128), (2, 3, 64, 128), (1, 4, 130, 128), (2, 2, 191, 128), (9, 31, 192, 128), (1, 2, 193, 128)]


def _tensors(shape, dtype, seed, scale=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return [(scale * torch.randn(shape, generator=g, device="cuda")).to((torch.float16, torch.bfloat16)[dtype]) for _ in range(3)]


def _call(ctx, q, k, v, out, timed):
    ctx.set_timing(timed)
    o = torch.full(q.shape, float("nan"), dtype=out, device="cuda")
    ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    return o, ctx.report()


def _same(a, b, ra, rb):
    assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))
    assert (ra.n_events, ra.n_events_dropped, ra.range_flags, ra.recheck_entries) == (rb.n_events, rb.n_events_dropped, rb.range_flags, rb.recheck_entries)
    assert np.array_equal(ra.residual_max, rb.residual_max) and np.array_equal(ra.tile_flags, rb.tile_flags)
    assert np.array_equal(ra.rowtile_flags, rb.rowtile_flags)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("causal", [False, True])
def test_one_launch_gives_what_two_give(shape, causal):
    for dtype, mode, fold, out in [(synth.F16, ftattn.FT_CORRECT, False, torch.float32), (synth.BF16, ftattn.FT_CORRECT, True, torch.bfloat16),
                                   (synth.BF16, ftattn.FT_OFF, False, torch.float32), (synth.F16, ftattn.FT_DETECT, False, torch.float16)]:
        print(f"[one launch] {shape} causal {causal} dtype {dtype} mode {mode} fold {fold}", flush=True)
        out_code = ftattn.F32 if out == torch.float32 else dtype
        ctx = ftattn.FtAttn(*shape, dtype, causal, out_dtype=out_code, ft_mode=mode, rowsum_fold=fold)
        q, k, v = _tensors(shape, dtype, shape[2])
        one, r1 = _call(ctx, q, k, v, out, False)
        two, r2 = _call(ctx, q, k, v, out, True)
        _same(one, two, r1, r2)
        assert r1.n_events == 0
        if out == torch.float32:
            # (bars of the fused path: fp16 weights and tiles)
            Q, K, V = (H.head_f64(x.view(torch.int16).cpu().numpy().view(np.uint16), dtype, 0, shape[1] - 1) for x in (q, k, v))
            ma, rf = H.tolerance_ok(one[0, -1].double().cpu().numpy(), eorc.attention_clean(Q, K, V, float(ctx.config.softmax_scale), causal))
            assert ma <= 2e-3 and rf <= 1e-3
        ctx.close()


@pytest.mark.parametrize("shape", [(1, 6, 128, 64), (1, 6, 90, 64), (1, 6, 192, 128), (1, 6, 70, 128)])
@pytest.mark.parametrize("dtype", [synth.F16, synth.BF16])
@pytest.mark.parametrize("causal", [False, True])
def test_infinities_and_nan(shape, dtype, causal):
    """One head each with an infinity or NaN in an operand, with the type's lowest value, and with keys whose scores are all -inf (in bf16
    by the conversion to fp16): outputs and reports of one launch and of two."""
    print(f"[one launch, not finite] {shape} dtype {dtype} causal {causal}", flush=True)
    q, k, v = _tensors(shape, dtype, shape[2])
    n = shape[2]
    q[0, 0, n // 2, 3] = float("inf")
    k[0, 1, n - 1, 5] = float("-inf")
    v[0, 2, 0, 7] = float("nan")
    k[0, 3, n // 3] = torch.finfo(k.dtype).min
    q[0, 4, :, 0], q[0, 4, :, 1:], k[0, 4, :, 0] = 1.0, 0.0, float("-inf")
    v[0, 5, n // 2, 1] = float("inf")
    for mode in (ftattn.FT_CORRECT, ftattn.FT_DETECT, ftattn.FT_OFF):
        ctx = ftattn.FtAttn(*shape, dtype, causal, ft_mode=mode, max_events=1 << 20)
        one, r1 = _call(ctx, q, k, v, torch.float32, False)
        two, r2 = _call(ctx, q, k, v, torch.float32, True)
        _same(one, two, r1, r2)
        assert not r1.event_set() ^ r2.event_set() and (mode == ftattn.FT_OFF or r1.n_events > 0)
        assert bool(torch.isnan(one[0, 0, n // 2]).all()) and bool(torch.isnan(one[0, 2, n - 1, 7])) and bool(torch.isfinite(one[0, 2, :, 8:]).all())
        ctx.close()


@pytest.mark.parametrize("shape", [(2, 3, 127, 64), (1, 300, 70, 64), (2, 5, 192, 128)])
def test_reports_are_of_their_own_call(shape):
    """Thresholds far below rounding make every check fire; values that fp16 cannot hold set range flags.  Calls in one and
    in two launches, with and without such inputs, in turn: each report is that of a context that made no other call."""
    print(f"[one launch reports] {shape}", flush=True)
    options = dict(eps1=1e-7, tau_o=1e-9, max_events=1 << 20)
    clean = _tensors(shape, synth.BF16, 5)
    large = [x.clone() for x in clean]
    large[1][0, 0, 0, 0] = 1e6
    large[2][-1, -1, -1, -1] = 1e-9
    def report(ctx, data, timed):
        return _call(ctx, *data, torch.float32, timed)[1]
    def fresh(data, timed):
        ctx = ftattn.FtAttn(*shape, synth.BF16, True, **options)
        r = report(ctx, data, timed)
        ctx.close()
        return r
    want = {("clean", t): fresh(clean, t) for t in (False, True)} | {("large", t): fresh(large, t) for t in (False, True)}
    assert want["clean", False].n_events > 100 and want["large", False].range_flags & 3 == 3 and want["clean", False].range_flags == 0
    ctx = ftattn.FtAttn(*shape, synth.BF16, True, **options)
    for name, timed in [("clean", False), ("large", False), ("large", False), ("clean", False), ("clean", True), ("large", False),
                        ("clean", True), ("large", True), ("clean", False), ("clean", False)]:
        got, ref = report(ctx, {"clean": clean, "large": large}[name], timed), want[name, timed]
        assert got.n_events == ref.n_events and got.n_events_dropped == 0 and not got.event_set() ^ ref.event_set()
        assert got.range_flags == ref.range_flags and got.recheck_entries == ref.recheck_entries
        assert np.array_equal(got.residual_max, ref.residual_max)
    # both ways of a call flag the same
    assert not want["clean", False].event_set() ^ want["clean", True].event_set()
    ctx.close()


def test_one_launch_in_a_captured_graph():
    shape = (3, 4, 100, 64)
    q, k, v = _tensors(shape, synth.F16, 9)
    ctx = ftattn.FtAttn(*shape, synth.F16, True)
    o = torch.empty(shape, dtype=torch.float32, device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        ctx.forward(q, k, v, o, None, side.cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    eager = ftattn.FtAttn(*shape, synth.F16, True)
    for seed in range(4):
        for x, y in zip((q, k, v), _tensors(shape, synth.F16, 20 + seed)):
            x.copy_(y)
        o.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        want, ref = _call(eager, q, k, v, torch.float32, False)
        rep = ctx.report()
        assert torch.equal(o, want) and rep.n_events == 0 and np.array_equal(rep.residual_max, ref.residual_max)
    ctx.close(); eager.close()


def test_static_entry_point_in_one_launch():
    """Counts of the entry point without a context: one launch, two launches and one launch again."""
    events = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for shape in [(2, 3, 128, 64), (1, 2, 400, 64), (2, 2, 192, 128), (2, 3, 128, 64)]:
        q, k, v = _tensors(shape, synth.F16, 3)
        o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
        events.fill_(-1)
        ftattn.forward_static(q, k, v, o, *shape, synth.F16, True, n_events=events, stream=torch.cuda.current_stream().cuda_stream)
        ctx = ftattn.FtAttn(*shape, synth.F16, True)
        want, _ = _call(ctx, q, k, v, torch.float32, True)
        ctx.close()
        assert torch.equal(o, want) and int(events) == 0


def test_static_calls_that_overlap_leave_nothing_behind():
    """Calls of different numbers of heads that overlap in time, on three streams, may spoil their own counts: those of every call after
    them are its own.  (All checks fire, so that each workgroup has something to count.)"""
    lib = ftattn.load_library()
    def call(x, n_events, stream):
        cfg = ftattn.Config(struct_size=C.sizeof(ftattn.Config), batch=x.shape[0], heads=x.shape[1], seq=x.shape[2], head_dim=x.shape[3], in_dtype=synth.F16,
                            out_dtype=ftattn.F32, causal=1, ft_mode=ftattn.FT_DETECT, eps1=1e-7, tau_o=1e-9, max_events=4096)
        o = outs[tuple(x.shape)]
        assert lib.ftattn_forward_static(C.byref(cfg), x.data_ptr(), x.data_ptr(), x.data_ptr(), o.data_ptr(), n_events.data_ptr(), C.c_void_p(stream)) == 0
    shapes = [(1, 3, 64, 64), (20, 16, 128, 64), (2, 35, 70, 64), (3, 100, 150, 128)]
    data = {s: _tensors(s, synth.F16, s[1])[0] for s in shapes}
    outs = {s: torch.empty(s, dtype=torch.float32, device="cuda") for s in shapes}
    want = {}
    for s, x in data.items():
        ctx = ftattn.FtAttn(*s, synth.F16, True, ft_mode=ftattn.FT_DETECT, eps1=1e-7, tau_o=1e-9)
        ctx.forward(x, x, x, outs[s], None, torch.cuda.current_stream().cuda_stream)
        rep = ctx.report()
        want[s] = rep.n_events + rep.n_events_dropped
        ctx.close()
        assert want[s] > s[0] * s[1]
    streams = [torch.cuda.Stream() for _ in range(3)]
    spoilt = torch.zeros(3, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for turn in range(20):
        for i, st in enumerate(streams):
            call(data[shapes[(turn + i) % len(shapes)]], spoilt[i:i + 1], st.cuda_stream)
    torch.cuda.synchronize()
    n = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for s in shapes * 3:
        print(f"[one launch after an overlap] {s}", flush=True)
        n.fill_(-1)
        call(data[s], n, torch.cuda.current_stream().cuda_stream)
        assert int(n) == want[s]
