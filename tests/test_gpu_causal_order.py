"""Every (head, row tile) of a causal call is computed once, for head counts with and without a remainder
by the 8 XCDs and groups of heads that are full, partial or larger than the heads there are.  Reference:
attention in fp64 on the device, from the inputs as the kernel takes them.  Tolerance as in test_gpu_parity.py
(fp16 weights): 2e-3 absolute, 1e-3 relative Frobenius."""
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


def test_masked_tiles_detect_a_changed_key():
    """A masked tile goes to the exact evaluation when, and only when, something in it is wrong: the encoded
    checksums are those of the keys, so a clean pass reports nothing, also where a key is so large that the
    scores beyond the mask are far above the valid ones."""
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
