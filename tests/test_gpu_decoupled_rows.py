"""The row softmax of the decoupled scheme at the edges of its register chunks (256 scores) and of the row
lengths at which it changes shape (512, 1024, 2048, 4096 scores), odd lengths among them: output against
attention in fp64 on the device, and one fault per stage of the softmax in the first and last chunk of a
row, found in that row and repaired.  Tolerance as in test_gpu_decoupled.py: 2e-3 absolute, 1e-3 relative."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftdecoupled

pytestmark = pytest.mark.gpu

ST_EXP, ST_PNORM = 1, 2


@pytest.mark.parametrize("seq", [1, 3, 64, 255, 256, 257, 512, 513, 1023, 1025, 2047, 2048, 2050, 4095, 4096, 4097])
@pytest.mark.parametrize("causal", [False, True])
def test_rows(seq, causal):
    print(f"[decoupled rows] seq {seq} causal {causal}", flush=True)
    shape = (1, 2, seq, 64)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) * 64 ** -0.5
    if causal:
        s.masked_fill_(~torch.ones((seq, seq), dtype=torch.bool, device="cuda").tril(), float("-inf"))
    want = torch.matmul(torch.softmax(s, -1), v.double())
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream

    def check():
        diff = o.double() - want
        assert float(diff.abs().max()) <= 2e-3 and float(diff.norm() / want.norm()) <= 1e-3

    for mode in (ftdecoupled.FT_CORRECT, ftdecoupled.FT_OFF):
        ctx = ftdecoupled.FtDecoupled(*shape, 0, causal, ft_mode=mode)
        o.fill_(float("nan"))
        ctx.forward(q, k, v, o, None, stream)
        rep = ctx.report()
        assert rep.n_events == 0 and rep.retried_rows == 0
        check()
        if mode == ftdecoupled.FT_CORRECT:
            # sign bit of the row's first and last exponential (2 e > eps for e > 1/8192: the scores are of order
            # one) and the top exponent bit of its last weight (p < 1 becomes p * 2^128)
            r = seq - 1
            faults = [(0, 0, ST_EXP, r, 0, 31), (0, 1, ST_PNORM, r, seq - 1, 30)]
            if seq > 1:
                faults.append((0, 0, ST_EXP, r, seq - 1, 31))
            o.fill_(float("nan"))
            ctx.forward(q, k, v, o, np.array(faults, np.int32), stream)
            rep = ctx.report()
            assert rep.event_set() == {(0, 0, ST_EXP, r, f[4]) for f in faults if f[2] == ST_EXP} | {(0, 1, ST_PNORM, r, -1)}
            assert rep.retried_rows == 2
            check()
        ctx.close()


@pytest.mark.parametrize("batch,heads,seq,head_dim,causal", [
    (1, 2, 1, 8, False), (2, 1, 63, 40, True), (1, 3, 65, 72, False), (2, 2, 70, 200, True), (1, 1, 129, 256, False),   # V^T remainders
    (3, 3, 1024, 128, True), (1, 5, 2048, 64, True), (2, 2, 512, 256, True)])                                          # XCD ranges moved per head
@pytest.mark.parametrize("bf16", [False, True])
def test_heads_and_features(batch, heads, seq, head_dim, causal, bf16):
    """V^T in blocks of 64 keys and 64 features, with remainders in both, and every tile of every head computed
    once where the XCD ranges move on per head.  Same tolerance (V and O as above, P in fp16)."""
    print(f"[decoupled heads] {batch} x {heads} x {seq} x {head_dim} causal {causal} bf16 {bf16}", flush=True)
    shape = (batch, heads, seq, head_dim)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + head_dim)
    tt = torch.bfloat16 if bf16 else torch.float16
    q, k, v = (torch.randn(shape, generator=g, device="cuda").to(tt) for _ in range(3))
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftdecoupled.FtDecoupled(*shape, 1 if bf16 else 0, causal)
    ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
    rep = ctx.report()
    ctx.close()
    assert rep.n_events == 0 and rep.retried_rows == 0
    mask = torch.ones((seq, seq), dtype=torch.bool, device="cuda").tril()
    for b in range(batch):
        for h in range(heads):
            s = (q[b, h].double() @ k[b, h].double().t().contiguous()) * head_dim ** -0.5
            if causal:
                s.masked_fill_(~mask, float("-inf"))
            want = torch.softmax(s, -1) @ v[b, h].double()
            diff = o[b, h].double() - want
            assert float(diff.abs().max()) <= 2e-3 and float(diff.norm() / want.norm()) <= 1e-3


@pytest.mark.parametrize("seq", [40, 700, 1500, 3000, 4097])
def test_weights_do_not_depend_on_the_fault_list(seq):
    """The kernel that calls without a fault list run stores the weight that it sums for eq. (12), as the
    injecting one does, whose faults show that the sum covers it: faults that are found and evaluated again
    leave the output of the fault-free call, bit for bit.  (A product contracted into the conversion to fp16
    rounds once instead of twice, which changes the last digit of about one weight in 2^13.)"""
    print(f"[decoupled weights] seq {seq}", flush=True)
    shape = (1, 4, seq, 64)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq + 1)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    outs = []
    stream = torch.cuda.current_stream().cuda_stream
    for faults in (None, np.array([(0, 1, ST_EXP, seq // 2, 3, 31), (0, 2, ST_PNORM, seq - 1, 5, 30)], np.int32)):
        ctx = ftdecoupled.FtDecoupled(*shape, 0, False)
        o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
        ctx.forward(q, k, v, o, faults, stream)
        rep = ctx.report()
        assert rep.retried_rows == (0 if faults is None else 2)
        ctx.close()
        outs.append(o)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("batch,heads,seq,head_dim", [(1, 11, 257, 64), (1, 3, 1025, 128), (2, 8, 512, 64), (1, 9, 300, 136), (3, 17, 130, 128), (1, 1, 2049, 64)])
def test_causal_tiles_of_all_heads(batch, heads, seq, head_dim):
    """Causal products launch the tiles on and below the diagonal only, and the longest tiles of all heads first: numbers of
    heads that 8 does not divide, last rows of tiles one token long, one and several tiles to a row of 256 tokens."""
    print(f"[decoupled tiles] {batch} x {heads} x {seq} x {head_dim}", flush=True)
    shape = (batch, heads, seq, head_dim)
    g = torch.Generator(device="cuda")
    g.manual_seed(seq)
    q, k, v = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) * head_dim ** -0.5
    s.masked_fill_(~torch.ones((seq, seq), dtype=torch.bool, device="cuda").tril(), float("-inf"))
    want = torch.matmul(torch.softmax(s, -1), v.double())
    o = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftdecoupled.FtDecoupled(*shape, 0, True)
    for _ in range(2):
        o.fill_(float("nan"))
        ctx.forward(q, k, v, o, None, torch.cuda.current_stream().cuda_stream)
        rep = ctx.report()
        assert rep.n_events == 0 and rep.n_events_dropped == 0 and rep.retried_rows == 0
        diff = o.double() - want
        assert float(diff.abs().max()) <= 2e-3 and float(diff.norm() / want.norm()) <= 1e-3
    ctx.close()
