"""Every tile shape and the split of the K dimension of the linear layer's kernel, at sizes with
remainders in tokens, features and K.  Verification is exercised without the injector: one element of
one weight row is changed after its checksums were taken, which shifts one output of every token by a
known amount; every token must be reported at that column and restored from the checksum of the
unchanged weights.  Reference: the product in fp64 on the device.  Tolerance as in test_gpu_gemm.py:
fp32 accumulation over k <= 6136 terms of outputs of order one, 1e-4; a value restored from bf16 words
(16 bits) 4e-3."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftgemm

pytestmark = pytest.mark.gpu

# (m, n, k): tile shape and shares of K with the checksums over the features, and over the tokens (the same kernel with m
# and n exchanged); test_launch_plans.py holds the plan to it.  Matrices of 128 features or fewer are in
# test_gpu_gemm_narrow.py, those here are too small for their tiles.
PLANS = {(1, 70, 72): (("strip", 1), ("strip", 1)), (130, 33, 200): (("strip", 1), ("strip", 1)),
         (37, 1000, 1024): (("strip", 1), ("slim2", 1)), (40, 601, 2056): (("strip", 16), ("strip", 8)),
         (700, 1000, 1024): (("strip", 1), ("strip", 1)), (31, 300, 64): (("strip", 1), ("strip", 1)),
         (2049, 1030, 72): (("quarter", 1), ("quarter", 1)), (2000, 1999, 512): (("quarter", 1), ("quarter", 1)),
         (1000, 8000, 136): (("half", 1), ("half", 1)),
         (4097, 2050, 264): (("wide", 1), ("wide", 1)), (3000, 3000, 72): (("wide", 1), ("wide", 1)),
         (701, 1499, 4040): (("quarter", 2), ("strip", 1)), (5001, 299, 6136): (("half", 2), ("quarter", 2))}
SHAPES = list(PLANS)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype,fold", [(ftgemm.F16, False), (ftgemm.BF16, True)])
def test_tile_shapes(m, n, k, dtype, fold):
    print(f"[gemm tiles] m={m} n={n} k={k} dtype={dtype} fold_tokens={fold}", flush=True)
    tt = torch.float16 if dtype == ftgemm.F16 else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(m + 3 * n + 7 * k)
    x = torch.randn((m, k), generator=g, device="cuda").to(tt)
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).to(tt)
    for out in (ftgemm.F32, dtype):
        y = torch.full((m, n), float("nan"), dtype=torch.float32 if out == ftgemm.F32 else tt, device="cuda")
        ctx = ftgemm.FtGemm(m, n, k, out_dtype=out, in_dtype=dtype, fold_tokens=fold)
        ctx.encode_weights(w)
        ctx.forward(x, w, y)
        rep = ctx.report()
        ctx.close()
        want = x.double() @ w.double().t()
        tol = 1e-4 if out == ftgemm.F32 else (2.0 ** -10 if dtype == ftgemm.F16 else 2.0 ** -7)
        assert rep.n_events == 0 and rep.n_events_dropped == 0
        assert bool(((y.double() - want).abs() <= tol * want.abs().clamp(min=1.0)).all())


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype,correct", [(ftgemm.F16, True), (ftgemm.BF16, True), (ftgemm.F16, False)])
def test_location_and_repair_in_every_tile_shape(m, n, k, dtype, correct):
    print(f"[gemm tiles repair] m={m} n={n} k={k} dtype={dtype} correct={correct}", flush=True)
    tt = torch.float16 if dtype == ftgemm.F16 else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(m + 5 * n + 11 * k)
    x = torch.randn((m, k), generator=g, device="cuda").to(tt)
    x[:, 3] = 1.0
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).to(tt)
    want = x.double() @ w.double().t()
    y = torch.full((m, n), float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftgemm.FtGemm(m, n, k, in_dtype=dtype, ft_mode=ftgemm.FT_CORRECT if correct else ftgemm.FT_DETECT)
    ctx.encode_weights(w)
    cols = sorted({0, n // 2, n - 1})
    for col in cols:
        was = w[col, 3].clone()
        w[col, 3] = was + 8.0                                  # every output of this feature moves by 8 (exact to the type's rounding)
        shift = float(w[col, 3].double() - was.double())
        ctx.forward(x, w, y)
        rep = ctx.report()
        w[col, 3] = was
        assert rep.n_events_dropped == 0
        assert rep.event_list() == [(r, col, int(correct)) for r in range(m)]
        expect = want.clone()
        if not correct:
            expect[:, col] += shift
        err = (y.double() - expect).abs()
        assert float(err.max()) <= (1e-4 if dtype == ftgemm.F16 else 4e-3)
    # the same context without a fault: nothing of the earlier calls is left in its report
    ctx.forward(x, w, y)
    rep = ctx.report()
    ctx.close()
    assert rep.n_events == 0 and float((y.double() - want).abs().max()) <= 1e-4
    assert np.isfinite(rep.residual_max)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype", [ftgemm.F16, ftgemm.BF16])
def test_restore_of_16_bit_results_and_of_infinities(m, n, k, dtype):
    """As above with results in the input type, and with a weight that becomes infinite: then the residuals leave
    the fp32 range, the fold of overwhelming size is the located one, and the restored value is finite.  Tolerance: the
    rounding of the result type, and of the checksum words (2^-22 of their value in fp16, 2^-16 in bf16; a value
    is restored from a sum of at most 32 of order one)."""
    print(f"[gemm tiles 16-bit] m={m} n={n} k={k} dtype={dtype}", flush=True)
    tt = torch.float16 if dtype == ftgemm.F16 else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(m + 13 * n + 17 * k)
    x = torch.randn((m, k), generator=g, device="cuda").to(tt)
    x[:, 3] = 1.0
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).to(tt)
    want = x.double() @ w.double().t()
    for out in (dtype, ftgemm.F32):
        y = torch.full((m, n), float("nan"), dtype=torch.float32 if out == ftgemm.F32 else tt, device="cuda")
        ctx = ftgemm.FtGemm(m, n, k, in_dtype=dtype, out_dtype=out)
        ctx.encode_weights(w)
        for col, value in ((n // 3, 8.0), (n - 1, float("inf")), (0, float("-inf"))):
            was = w[col, 3].clone()
            w[col, 3] = was + value
            ctx.forward(x, w, y)
            rep = ctx.report()
            w[col, 3] = was
            assert rep.n_events_dropped == 0
            assert rep.event_list() == [(r, col, 1) for r in range(m)]
            ulp = 0.0 if out == ftgemm.F32 else (2.0 ** -11 if dtype == ftgemm.F16 else 2.0 ** -8)
            err = (y.double() - want).abs()
            assert bool((err <= (1e-4 if dtype == ftgemm.F16 else 4e-3) + ulp * want.abs()).all())
        ctx.close()


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("out", [ftgemm.F32, ftgemm.F16])
def test_every_class_flagged_is_restored_in_place(m, n, k, fold, out):
    """With a threshold far below rounding nearly every class is flagged and some element of it, wherever the
    ratio of two rounding residuals points, is replaced by what the checksum implies for it.  That differs from the
    element by the residual, which a clean call keeps below 2^-15 of the class's sum of at most 32 magnitudes:
    the output moves by no more than that, in both orientations, and an element written to another place would be off
    by its own size.  (With checksums over the token rows they are taken inside the call, so nothing can
    be changed behind them.)"""
    print(f"[gemm tiles restore] m={m} n={n} k={k} fold_tokens={fold} out={out}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m + 19 * n + 23 * k)
    x = torch.randn((m, k), generator=g, device="cuda").half()
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).half()
    y = []
    for tau_rel in (0.0, 1e-12):
        ctx = ftgemm.FtGemm(m, n, k, out_dtype=out, fold_tokens=fold, tau_rel=tau_rel)
        ctx.encode_weights(w)
        y.append(torch.full((m, n), float("nan"), dtype=torch.float32 if out == ftgemm.F32 else torch.float16, device="cuda"))
        ctx.forward(x, w, y[-1])
        rep = ctx.report()
        ctx.close()
        if tau_rel == 0.0:
            assert rep.n_events == 0
    kept, lanes = (n, m) if fold else (m, n)                 # rows of the folded product, and what a row folds
    classes = kept * sum(min(8, min(256, lanes - at)) for at in range(0, lanes, 256))
    total = rep.n_events + rep.n_events_dropped
    if lanes <= 8:                                           # one result per class, accumulated as its checksum is
        assert total == 0
        return
    assert classes // 4 < total <= classes
    ev = rep.events
    assert ((ev["row"] >= -1) & (ev["row"] < m) & (ev["col"] >= -1) & (ev["col"] < n)).all()
    assert (ev["row" if not fold else "col"] >= 0).all() and (ev["action"] == 1).any()
    top = float(y[0].double().abs().max())
    ulp = 0.0 if out == ftgemm.F32 else 2.0 ** -10 * top
    moved = float((y[1].double() - y[0].double()).abs().max())
    assert moved <= 2.0 ** -15 * 32 * top + ulp


@pytest.mark.parametrize("max_events", [1, 3, 4, 8, 64])
@pytest.mark.parametrize("m,n,k", [(5, 300, 64), (70, 1000, 1024), (300, 40, 72)])
def test_event_log_wraps_and_overflows(m, n, k, max_events):
    """Calls that each log m or 2 m events, one or two per token: the log wraps from call to call, and holds only a
    part of a call's events where they are more than max_events.  Every event reported is one of its own call's, none
    is reported twice, and the rest is counted."""
    print(f"[gemm event log] m={m} n={n} k={k} max_events={max_events}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(m)
    x = torch.randn((m, k), generator=g, device="cuda").half()
    x[:, 3] = 1.0
    w = (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).half()
    y = torch.empty((m, n), dtype=torch.float32, device="cuda")
    ctx = ftgemm.FtGemm(m, n, k, max_events=max_events)
    ctx.encode_weights(w)
    for call in range(7):
        cols = [(8 * call) % n] + ([(8 * call + 3) % n] if call % 3 == 1 else [])      # (other columns in every call, two classes)
        was = w[cols, 3].clone()
        w[cols, 3] = was + 8.0
        ctx.forward(x, w, y)
        rep = ctx.report()
        w[cols, 3] = was
        total = m * len(cols)
        assert (rep.n_events, rep.n_events_dropped) == (min(total, max_events), total - min(total, max_events))
        events = rep.event_list()
        assert len(set(events)) == len(events) and set(events) <= {(r, c, 1) for r in range(m) for c in cols}
    ctx.forward(x, w, y)
    rep = ctx.report()
    assert (rep.n_events, rep.n_events_dropped) == (0, 0)
    ctx.close()
