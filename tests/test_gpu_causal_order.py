"""Every (head, row tile) of a causal call is computed once, for head counts with and without a remainder
by the 8 XCDs and groups of heads that are full, partial or larger than the heads there are.  Reference:
attention in fp64 on the device, from the inputs as the kernel takes them.  Tolerance as in test_gpu_parity.py
(fp16 weights): 2e-3 absolute, 1e-3 relative Frobenius."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 64), (1, 7, 600), (1, 8, 129), (3, 3, 513), (1, 16, 300), (2, 12, 1030), (5, 5, 260), (1, 67, 777), (8, 17, 100)]


@pytest.mark.parametrize("batch,heads,seq", SHAPES)
@pytest.mark.parametrize("head_dim,mode", [(64, ftattn.FT_CORRECT), (128, ftattn.FT_CORRECT), (64, ftattn.FT_OFF), (128, ftattn.FT_OFF)])
def test_every_row_tile_once(batch, heads, seq, head_dim, mode):
    print(f"[causal order] {batch} x {heads} x {seq} x {head_dim} mode {mode}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + 31 * heads + head_dim)
    shape = (batch, heads, seq, head_dim)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, 0, True, ft_mode=mode)
    for _ in range(2):
        ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
        rep = ctx.report()
        assert rep.n_events == 0 and rep.n_events_dropped == 0
        if mode != ftattn.FT_OFF:
            # the statistics of every row tile: its output residual is positive and below the threshold
            assert (rep.residual_max[..., 1] > 0).all() and (rep.residual_max[..., 1] <= ctx.config.tau_o).all()
    ctx.close()
    mask = torch.ones((seq, seq), dtype=torch.bool, device="cuda").tril()
    for b in range(batch):
        for h in range(heads):
            s = (q[b, h].double() @ k[b, h].double().t()) * head_dim ** -0.5
            want = torch.softmax(s.masked_fill(~mask, float("-inf")), -1) @ v[b, h].double()
            diff = o[b, h].double() - want
            assert float(diff.abs().max()) <= 2e-3
            assert float(diff.norm() / want.norm()) <= 1e-3


def test_clean_masked_tiles_report_nothing():
    """A clean pass reports nothing, also where a key is so large that the scores beyond the mask are far above
    the valid ones."""
    shape = (1, 2, 200, 64)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    k[:, :, 150:] *= 16.0
    o = torch.empty(shape, dtype=torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, 0, True)
    ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    rep = ctx.report()
    ctx.close()
    assert rep.n_events == 0
    mask = torch.ones((200, 200), dtype=torch.bool, device="cuda").tril()
    s = (q.double() @ k.double().transpose(-1, -2).contiguous()) * 64 ** -0.5
    want = torch.softmax(s.masked_fill(~mask, float("-inf")), -1) @ v.double()
    assert float((o.double() - want).abs().max()) <= 2e-3


@pytest.mark.parametrize("head_dim,seq,causal,margin", [(64, 333, True, 0.0), (128, 333, True, 0.0), (64, 500, True, 0.0), (128, 641, True, 0.0),
                                                        (128, 333, False, 0.0), (64, 333, False, 0.0), (64, 200, True, 3.0), (128, 333, True, 3.0)])
@pytest.mark.parametrize("dtype", [ftattn.F16, ftattn.BF16])
def test_masked_tiles_find_what_the_exact_evaluation_finds(head_dim, seq, causal, margin, dtype):
    """The kernels without the injection code look at a masked key tile through a filter before the exact
    evaluation, the injecting ones evaluate every masked tile exactly.  With a threshold far below the rounding of the
    scores every checksum class whose residual is not exactly zero is an event: a call without a fault list and one whose
    only fault is in another head report the same ones.  That there are such events in the masked tiles (the last keys,
    and the diagonal when causal) is asked for with a margin: about half of the classes of random scores have a
    residual, fewer in a last tile of a few keys, whose classes are sums of one or two."""
    print(f"[masked filter] seq {seq} head_dim {head_dim} causal {causal} margin {margin} dtype {dtype}", flush=True)
    shape = (1, 3, seq, head_dim)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + head_dim)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").to(torch.float16 if dtype == ftattn.F16 else torch.bfloat16) for _ in range(3))
    o = torch.empty(shape, dtype=torch.float32, device="cuda")
    ctx = ftattn.FtAttn(*shape, dtype, causal, ft_mode=ftattn.FT_DETECT, eps1=1e-9, max_events=1 << 20, rescale_margin=margin)
    sets = []
    for faults in (None, np.array([(0, 2, ftattn.ST_OACC, 0, 0, 0, 30)], np.int32)):
        ctx.forward(q, k, v, o, faults, torch.cuda.current_stream().cuda_stream)
        rep = ctx.report()
        assert rep.n_events_dropped == 0
        sets.append({e for e in rep.event_set() if e[1] < 2})
    ctx.close()
    assert sets[0] == sets[1]
    first = np.arange(seq) // 32 * 32                           # first row of a row's wave
    limit = np.arange(seq) if causal else np.full(seq, seq - 1)     # last key of a row
    for h in (0, 1):
        classes, found = 0, sum(1 for e in sets[0] if e[1] == h and e[2] == 0 and _masked(first[e[4]], e[3], seq, causal))
        for j in range((seq + 63) // 64):
            rows = [r for r in range(seq) if _masked(first[r], j, seq, causal) and limit[r] >= 64 * j]
            classes += sum(min(8, limit[r] - 64 * j + 1) for r in rows)
        print(f"[masked filter] head {h}: {found} events, {classes} classes", flush=True)
        assert classes // 8 < found <= classes


def _masked(row0, tile, seq, causal):
    return (causal and 64 * tile + 63 > row0) or 64 * tile + 64 > seq
