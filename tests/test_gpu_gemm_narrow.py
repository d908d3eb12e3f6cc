"""Matrices of at most 128 features, or tokens where the checksums fold tokens: the high and the low tiles of that width and
the 32-token tiles with K split, each with a remainder of tokens, features and K.  Same checks and tolerances as
test_gpu_gemm_tiles.py."""
import pytest

torch = pytest.importorskip("torch")

from paper_2504_02211_amd import ftgemm
import test_gpu_gemm_tiles as tiles

pytestmark = pytest.mark.gpu

# (m, n, k): tile shape and shares of K; with the checksums over the tokens the same kernels run for (n, m, k)
PLANS = {(16500, 100, 2056): ("narrow", 1), (60001, 40, 1032): ("slim", 1),
         (1001, 100, 1000): ("narrow2", 1), (20003, 50, 1032): ("slim2", 1),
         (37, 100, 4088): ("strip", 16), (2001, 128, 4040): ("strip", 4), (3001, 33, 4040): ("strip", 2)}
SHAPES = list(PLANS)


def seen_by_the_kernel(m, n, k, fold):
    return (n, m, k) if fold else (m, n, k)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype,fold", [(ftgemm.F16, False), (ftgemm.BF16, False), (ftgemm.BF16, True)])
def test_products(m, n, k, dtype, fold):
    tiles.test_tile_shapes(*seen_by_the_kernel(m, n, k, fold), dtype, fold)


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_location_and_repair(m, n, k):
    tiles.test_location_and_repair_in_every_tile_shape(m, n, k, ftgemm.F16, True)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("dtype", [ftgemm.F16, ftgemm.BF16])
def test_restore_of_16_bit_results_and_of_infinities(m, n, k, dtype):
    tiles.test_restore_of_16_bit_results_and_of_infinities(m, n, k, dtype)


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("out", [ftgemm.F32, ftgemm.F16])
def test_every_class_flagged_is_restored_in_place(m, n, k, fold, out):
    tiles.test_every_class_flagged_is_restored_in_place(*seen_by_the_kernel(m, n, k, fold), fold, out)
