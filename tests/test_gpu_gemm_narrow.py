"""Matrices of at most 128 features: the high and the low tiles of that width and the 32-token tiles with K split, each
with a remainder of tokens, features and K.  Same checks and tolerances as test_gpu_gemm_tiles.py."""
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftgemm
import test_gpu_gemm_tiles as tiles

pytestmark = pytest.mark.gpu

SHAPES = [(16500, 100, 2056), (60001, 40, 1032),      # 128 and 64 features, high tiles
          (1001, 100, 1000), (20003, 50, 1032),       # low tiles
          (37, 100, 4088), (2001, 128, 4040)]         # 32-token tiles of 256 features, K split


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype,fold", [(ftgemm.F16, False), (ftgemm.BF16, False), (ftgemm.BF16, True)])
def test_products(m, n, k, dtype, fold):
    tiles.test_tile_shapes(m, n, k, dtype, fold)


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_location_and_repair(m, n, k):
    tiles.test_location_and_repair_in_every_tile_shape(m, n, k, ftgemm.F16, True)
