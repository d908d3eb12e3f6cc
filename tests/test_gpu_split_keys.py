"""Calls with few or unevenly many row tiles, whose keys are split over several workgroups: every row of every head,
against attention in fp64 on the device from the inputs as the kernel takes them.  Tolerance as in
test_gpu_parity.py (fp16 weights): 2e-3 absolute, 1e-3 relative Frobenius; a 16-bit result adds half a unit of its last
place (2^-11 / 2^-8 relative)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn

pytestmark = pytest.mark.gpu

# shape: (row tiles that are not split, shares of the longest row tile that is); test_launch_plans.py holds the plan to it.
# Row tiles of one share beside others of many (causal), a ragged last row tile and key tile, sixteen shares, the row tiles
# left over by one and by three whole rounds of 256 at both head sizes, heads that the 8 XCDs do not divide
PLANS = {(1, 1, 1024, 128, False): (0, 4), (1, 1, 8200, 128, True): (0, 10), (2, 3, 733, 128, True): (0, 3), (1, 5, 3001, 64, True): (0, 3),
         (1, 1, 2047, 64, False): (0, 4), (1, 2, 6000, 64, True): (0, 4), (3, 16, 1531, 128, False): (256, 3), (1, 20, 2048, 128, True): (0, 2),
         (1, 22, 8900, 128, False): (768, 16), (3, 5, 2244, 64, False): (256, 6)}
SHAPES = list(PLANS)


def reference(q, k, v, causal):
    """fp64, head by head and in blocks of rows; yields (b, h, first row, rows)."""
    n = q.shape[2]
    cols = torch.arange(n, device="cuda")
    for b in range(q.shape[0]):
        for h in range(q.shape[1]):
            kt, vv = k[b, h].double().t().contiguous(), v[b, h].double()
            for r0 in range(0, n, 2048):
                s = (q[b, h, r0:r0 + 2048].double() @ kt) * q.shape[3] ** -0.5
                if causal:
                    s.masked_fill_(cols[None, :] > (r0 + torch.arange(s.shape[0], device="cuda"))[:, None], float("-inf"))
                yield b, h, r0, torch.softmax(s, -1) @ vv


@pytest.mark.parametrize("batch,heads,seq,head_dim,causal", SHAPES)
@pytest.mark.parametrize("option", ["correct", "off", "fold", "outliers"])
def test_shares_add_up(batch, heads, seq, head_dim, causal, option):
    print(f"[split keys] {batch} x {heads} x {seq} x {head_dim} causal {causal} {option}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + 31 * heads + head_dim)
    shape = (batch, heads, seq, head_dim)
    bf16 = option != "fold"
    q, k, v = (torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16 if bf16 else torch.float16) for _ in range(3))
    if option == "outliers":            # maxima of the shares far apart
        k *= torch.where(torch.rand(shape[:3], generator=g, device="cuda") < 0.01, 8.0, 1.0).unsqueeze(-1).to(k.dtype)
    o = torch.full(shape, float("nan"), dtype=torch.float16 if option == "fold" else torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, 1 if bf16 else 0, causal, out_dtype=0 if option == "fold" else 2,
                        ft_mode=ftattn.FT_OFF if option == "off" else ftattn.FT_CORRECT, rowsum_fold=option == "fold")
    st = torch.cuda.current_stream().cuda_stream
    for _ in range(2):
        ctx.forward(q, k, v, o, None, st)
        rep = ctx.report()
        assert rep.n_events == 0 and rep.n_events_dropped == 0
        if option != "off":
            assert (rep.residual_max[..., 1] > 0).all() and (rep.residual_max[..., 1] <= ctx.config.tau_o).all()
            assert (rep.residual_max[..., 2] > 0).all()
    ctx.close()
    unit = 2.0 ** -11 if option == "fold" else 0.0
    num = den = 0.0
    for b, h, r0, want in reference(q, k, v, causal):
        diff = o[b, h, r0:r0 + want.shape[0]].double() - want
        assert bool((diff.abs() <= 2e-3 + unit * want.abs()).all())
        num += float((diff ** 2).sum())
        den += float((want ** 2).sum())
    assert (num / den) ** 0.5 <= 1e-3 + unit


def test_split_call_in_a_graph_and_from_static_scratch():
    """Replays, and the entry point without a context, give what the eager call gives, bit for bit."""
    shape = (1, 2, 2500, 128)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    ctx = ftattn.FtAttn(*shape, 0, True)
    want, o = (torch.full(shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    ctx.forward(q, k, v, want, None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        o.fill_(float("nan"))
        junk = (torch.rand(1 << 20, device="cuda") * 2).sum()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.isfinite(junk) and torch.equal(o, want)
    ctx.close()
    o.fill_(float("nan"))
    ftattn.forward_static(q, k, v, o, *shape, 0, True, stream=torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(o, want)


TOO_LARGE_FOR_STATIC_STATE = (1, 4, 16384, 128, True)       # 46 MB of encoded tiles and 87 MB of state; the array holds 67 MB


def test_static_call_whose_state_does_not_fit_runs_unsplit():
    """The tiles fit the library's array, the state of the shares does not: same result to within rounding, not bit for bit."""
    *shape, causal = TOO_LARGE_FOR_STATIC_STATE
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    nev = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    ftattn.forward_static(q, k, v, o, *shape, 0, causal, n_events=nev, stream=torch.cuda.current_stream().cuda_stream)
    assert int(nev.item()) == 0
    num = den = 0.0
    for b, h, r0, want in reference(q, k, v, causal):
        diff = o[b, h, r0:r0 + want.shape[0]].double() - want
        assert bool((diff.abs() <= 2e-3).all())
        num += float((diff ** 2).sum())
        den += float((want ** 2).sum())
    assert (num / den) ** 0.5 <= 1e-3


def test_faults_in_a_call_that_would_be_split():
    """A call with a fault list runs unsplit on the same context: the fault is found and repaired, and the result is that of
    the split call to within the two tolerances, the row with the fault by itself as well."""
    shape = (1, 1, 4096, 128)
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    ctx = ftattn.FtAttn(*shape, 0, True)
    a, b = (torch.full(shape, float("nan"), dtype=torch.float32, device="cuda") for _ in range(2))
    st = torch.cuda.current_stream().cuda_stream
    ctx.forward(q, k, v, a, None, st)
    ctx.forward(q, k, v, b, [[0, 0, 0, 7, 3000, 450, 27]], st)
    rep = ctx.report()
    assert [(e[2], e[3], e[4], e[5]) for e in sorted(rep.event_set())] == [(0, 7, 3000, 450)]
    for rows in (slice(None), slice(3000, 3001)):
        diff = (b - a)[0, 0, rows].double()
        assert float(diff.abs().max()) <= 4e-3 and float(diff.norm() / a[0, 0, rows].double().norm()) <= 2e-3
    ctx.forward(q, k, v, b, None, st)
    assert ctx.report().n_events == 0 and torch.equal(a, b)
    ctx.close()


FIRING = [(1, 1, 1024, 128, False), (2, 3, 733, 128, True), (1, 5, 3001, 64, True), (1, 1, 2047, 64, False)]


@pytest.mark.parametrize("batch,heads,seq,head_dim,causal", FIRING)
@pytest.mark.parametrize("fold", [False, True])
def test_checks_of_shares_and_of_their_sums_fire(batch, heads, seq, head_dim, causal, fold):
    """With thresholds far below rounding nearly every check fires, in every share and on the sums.  Detected only, values
    stay as they are, bit for bit, and the events name rows, key tiles and columns of the whole row; corrected, an element
    moves by its rounding residual, which is far below the tolerance, where one written to another place would not be."""
    print(f"[split keys, events] {batch} x {heads} x {seq} x {head_dim} causal {causal} fold {fold}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + head_dim)
    shape = (batch, heads, seq, head_dim)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    st = torch.cuda.current_stream().cuda_stream

    def run(mode, **thresholds):
        o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
        ctx = ftattn.FtAttn(*shape, 0, causal, ft_mode=mode, rowsum_fold=fold, max_events=1 << 23, **thresholds)
        ctx.forward(q, k, v, o, None, st)
        rep = ctx.report()
        ctx.close()
        assert rep.n_events_dropped == 0
        return o, rep

    clean, rep = run(ftattn.FT_DETECT)
    assert rep.n_events == 0
    detected, rep = run(ftattn.FT_DETECT, eps1=1e-30, tau_o=1e-30)
    assert torch.equal(detected, clean)
    ev = rep.events
    assert (ev["action"] == 0).all() and ((ev["row"] >= 0) & (ev["row"] < seq)).all()
    head = ev["b"].astype(np.int64) * heads + ev["h"]
    assert ((head >= 0) & (head < batch * heads)).all()
    n_tiles, n_blocks = -(-seq // 64), -(-seq // 32)                     # a wave has 32 rows
    # scores: one event per row, key tile and class at most, some in every key tile of every wave, columns of that key tile
    s = ev["check"] == 0
    tile, row, col = ev["kv_tile"][s].astype(np.int64), ev["row"][s].astype(np.int64), ev["col"][s].astype(np.int64)
    assert ((tile >= 0) & (tile < n_tiles) & ((col == -1) | (col // 64 == tile))).all()
    key = ((head[s] * seq + row) * n_tiles + tile) * 8 + col % 8
    assert len(np.unique(key[col >= 0])) == int((col >= 0).sum())
    seen = np.zeros((batch * heads, n_blocks, n_tiles), bool)
    seen[head[s], row // 32, tile] = True
    last = np.minimum(np.arange(n_blocks) * 32 + 31, seq - 1) // 64 if causal else np.full(n_blocks, n_tiles - 1)
    assert (seen == (np.arange(n_tiles)[None, :] <= last[:, None])[None]).all()
    # outputs, and with the fold row-sums (where the location rule names them: with rounding residuals in few rows or none),
    # after the last share: no key tile, one event per row and class at most
    o = ev["check"] == 3
    assert (ev["kv_tile"][o] == -1).all() and ((ev["col"][o] >= -1) & (ev["col"][o] < head_dim)).all()
    found = o & (ev["col"] >= 0)
    key = (head[found] * seq + ev["row"][found]) * 8 + ev["col"][found] % 8
    assert len(np.unique(key)) == len(key)
    assert len(np.unique(head[o] * n_blocks + ev["row"][o] // 32)) == batch * heads * n_blocks
    l = ev["check"] == 2
    assert (ev["kv_tile"][l] == -1).all() and (ev["col"][l] == 0).all() and (fold or not l.any())
    assert len(np.unique(head[l] * seq + ev["row"][l])) == int(l.sum()) and not (ev["check"] == 1).any()

    corrected, rep = run(ftattn.FT_CORRECT, eps1=1e-30, tau_o=1e-30)
    ev = rep.events
    assert (ev["action"] == (ev["col"] >= 0)).all() and (ev["action"] == 1).any()
    num = den = 0.0
    for b, h, r0, want in reference(q, k, v, causal):
        diff = corrected[b, h, r0:r0 + want.shape[0]].double() - want
        assert bool((diff.abs() <= 2e-3).all())
        num += float((diff ** 2).sum())
        den += float((want ** 2).sum())
    assert (num / den) ** 0.5 <= 1e-3
    print(f"  events {rep.n_events}, corrected against clean {float((corrected - clean).abs().max()):.1e}", flush=True)


# whole shares at -inf: the longest row tiles have four or more
MASKED = {"end": (0.5, 1.0), "middle": (0.25, 0.75), "first": (0.0, 0.5)}
MASKED_PLANS = {(1, 1, 8192, 128, False): (0, 8), (1, 1, 8200, 128, True): (0, 10), (1, 2, 6000, 64, True): (0, 4), (1, 1, 6001, 64, False): (0, 5)}


@pytest.mark.parametrize("batch,heads,seq,head_dim,causal", MASKED_PLANS)
@pytest.mark.parametrize("mode", [ftattn.FT_OFF, ftattn.FT_DETECT])
@pytest.mark.parametrize("masked", MASKED)
def test_shares_without_a_finite_score(batch, heads, seq, head_dim, causal, mode, masked):
    """Keys masked by an infinite component (query 1 there): their scores are -inf and weigh nothing, also where a whole share
    of the keys has no other score.  Rows that have none at all are not looked at."""
    print(f"[split keys, -inf] {batch} x {heads} x {seq} x {head_dim} causal {causal} mode {mode} masked {masked}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + head_dim)
    shape = (batch, heads, seq, head_dim)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    q[..., 0] = 1.0
    lo, hi = (int(seq * x) for x in MASKED[masked])
    k[:, :, lo:hi, 0] = float("-inf")
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, 0, causal, ft_mode=mode)
    ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    ctx.close()
    num = den = 0.0
    for b, h, r0, want in reference(q, k, v, causal):
        keep = torch.isfinite(want).all(-1)
        assert int((~keep).sum()) == (min(max(hi - r0, 0), want.shape[0]) if causal and masked == "first" else 0)
        diff = (o[b, h, r0:r0 + want.shape[0]].double() - want)[keep]
        assert bool((diff.abs() <= 2e-3).all())
        num += float((diff ** 2).sum())
        den += float((want[keep] ** 2).sum())
    assert (num / den) ** 0.5 <= 1e-3


def test_a_share_of_nan_scores_is_not_lost():
    shape = (1, 1, 8192, 128)
    q, k, v = (torch.randn(shape, device="cuda").half() for _ in range(3))
    k[:, :, 4096:] = float("nan")
    o = torch.zeros(shape, dtype=torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, 0, False, ft_mode=ftattn.FT_OFF)
    ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    assert bool(torch.isnan(o).all())
    ctx.close()
