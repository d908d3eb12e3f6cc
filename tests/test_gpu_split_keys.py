"""Calls with few or unevenly many row tiles, whose keys are split over several workgroups: every row of every head,
against attention in fp64 on the device from the inputs as the kernel takes them.  Tolerance as in
test_gpu_parity.py (fp16 weights): 2e-3 absolute, 1e-3 relative Frobenius; a 16-bit result adds half a unit of its last
place (2^-11 / 2^-8 relative)."""
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


def test_faults_in_a_call_that_would_be_split():
    """A call with a fault list runs unsplit on the same context: the fault is found and repaired, and the result is that of
    the split call to within the two tolerances."""
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
    ctx.forward(q, k, v, b, None, st)
    assert ctx.report().n_events == 0 and torch.equal(a, b)
    ctx.close()


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
