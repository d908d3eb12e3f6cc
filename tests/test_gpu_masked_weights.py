"""The weight of a masked key is an exponential like any other, of -inf: one that is not 0 enters the row-sum and the output alike, so that
no later check sees it.  A flipped bit in one, of every checksum class, above the diagonal and behind the end of the
sequence, is found in every verification scheme, and taken back where the context corrects."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn, synth

pytestmark = pytest.mark.gpu


def _run(shape, causal, faults, **options):
    g = torch.Generator(device="cuda")
    g.manual_seed(shape[2])
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    ctx = ftattn.FtAttn(*shape, synth.F16, causal, **options)
    ctx.lib.ftattn_accept_masked_faults(ctx.handle)
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    ctx.forward(q, k, v, o, faults, torch.cuda.current_stream().cuda_stream)
    rep = ctx.report()
    ctx.close()
    return o, rep


@pytest.mark.parametrize("shape,causal", [((1, 2, 300, 64), True), ((1, 2, 333, 64), False), ((1, 2, 300, 128), True), ((1, 2, 333, 128), False)])
@pytest.mark.parametrize("options", [{}, dict(ft_mode=ftattn.FT_DETECT), dict(rowsum_fold=True), dict(per_step=1), dict(per_step=2), dict(stride=1),
                                     dict(rescale_margin=4.0)], ids=str)
def test_a_masked_weight_that_is_not_zero(shape, causal, options):
    print(f"[masked weights] {shape} causal {causal} {options}", flush=True)
    n, last = shape[2], (shape[2] - 1) // 64
    faults = []
    for c in range(8):                    # bit 30 of 0 is 2; every class, both halves of a key tile
        head, row = c % 2, 64 * (c % 4) + 11 + c if causal else 37 * c + 5
        col = 64 * (row // 64) + 32 * (c // 4) + 24 + c if causal else 64 * last + 24 + 32 * (c // 4) + c
        assert (row < col < 64 * (row // 64 + 1)) if causal else n <= col < 64 * (last + 1)
        faults.append((0, head, synth.ST_EXP, col // 64, row, col, 30))
    o, rep = _run(shape, causal, np.array(faults, np.int32), **options)
    assert rep.event_set() == {(b, h, ftattn.CHECK_EXP, tile, row, col) for b, h, _, tile, row, col, _ in faults}
    assert rep.n_events == len(faults) and set(rep.events["action"].tolist()) == {0 if "ft_mode" in options else 1}
    want, clean = _run(shape, causal, None, **options)
    assert clean.n_events == 0
    rows = torch.tensor([[f[1], f[4]] for f in faults], device="cuda").t()
    if "ft_mode" in options:              # only found: the rows hold the value row of a key that they do not attend to
        changed = (o != want).any(-1)[0]
        assert bool(changed[rows[0], rows[1]].all()) and int(changed.sum()) == len(faults)
    else:
        assert torch.allclose(o, want, rtol=1e-5, atol=1e-6)
