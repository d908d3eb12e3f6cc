"""Linear layers whose K is at most two steps of 64 and whose result is many tiles: the tile shape that keeps one LDS stage and runs two
workgroups to a CU.  Remainders in tokens, features and K, the fewest tiles that take it, both steps whole; checked as the
other tile shapes are (test_gpu_gemm_tiles.py), and its plan on the CPU."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn, ftgemm
import test_gpu_gemm_tiles as tiles

LOW = 8
# (m, n, k): whether the one-stage tile takes it; 300 tiles of 128 x 256 and one tile row fewer
SHAPES = {(4481, 2049, 72): True, (2433, 3841, 128): True, (19200, 300, 8): True, (12900, 513, 64): True,
          (19072, 300, 64): False, (4481, 2049, 136): False}


def test_plan():
    out = (C.c_int32 * 2)()
    lib = ftattn.load_library()
    for (m, n, k), low in SHAPES.items():
        lib.ftgemm_plan_of(C.c_int64(m), C.c_int64(n), C.c_int64(k), C.c_int32(1), out)
        assert (out[0] == LOW) == low and out[1] == 1, (m, n, k)
    lib.ftgemm_plan_of(C.c_int64(700), C.c_int64(700), C.c_int64(64), C.c_int32(16), out)
    assert out[0] == LOW


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [s for s, low in SHAPES.items() if low])
@pytest.mark.parametrize("dtype,fold", [(ftgemm.F16, False), (ftgemm.BF16, True), (ftgemm.F16, True)])
def test_products(m, n, k, dtype, fold):
    tiles.test_tile_shapes(*((n, m) if fold else (m, n)), k, dtype, fold)


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(4481, 2049, 72), (2433, 3841, 128)])
@pytest.mark.parametrize("dtype,correct", [(ftgemm.F16, True), (ftgemm.BF16, False)])
def test_location_and_repair(m, n, k, dtype, correct):
    tiles.test_location_and_repair_in_every_tile_shape(m, n, k, dtype, correct)


@pytest.mark.gpu
def test_checks_off():
    m, n, k = 4481, 2049, 72
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x, w = torch.randn((m, k), generator=g, device="cuda").half(), (torch.randn((n, k), generator=g, device="cuda") * k ** -0.5).half()
    y = torch.full((m, n), float("nan"), dtype=torch.float32, device="cuda")
    ctx = ftgemm.FtGemm(m, n, k, in_dtype=ftgemm.F16, ft_mode=ftgemm.FT_OFF)
    ctx.forward(x, w, y)
    assert ctx.report().n_events == 0
    ctx.close()
    want = x.double() @ w.double().t()
    assert float((y.double() - want).abs().max()) <= 1e-4
