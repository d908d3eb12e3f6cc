"""The kernels that the shapes of the GPU tests reach: the plans are made on the host, so that a change of their costs cannot
leave a kernel without the test that names it."""
import ctypes as C

import pytest

pytest.importorskip("torch")

from paper_2504_02211_amd import ftattn
import test_gpu_gemm_narrow as narrow
import test_gpu_gemm_tiles as tiles
import test_gpu_one_launch as one_launch
import test_gpu_report_after_replay as replay
import test_gpu_split_keys as split_keys
import test_short_contractions as short

TILES = ["wide", "half", "quarter", "strip", "narrow", "slim", "narrow2", "slim2", "low"]


def config(batch, heads, seq, head_dim, causal, **options):
    return ftattn.Config(struct_size=C.sizeof(ftattn.Config), batch=batch, heads=heads, seq=seq, head_dim=head_dim, in_dtype=0, out_dtype=2,
                         causal=int(causal), **{"ft_mode": ftattn.FT_CORRECT, **options})


def split_of(*shape, **options):
    """(row tiles that are not split, shares of the longest row tile that is, or 1, key tiles of a share at most, bytes of state)"""
    lib = ftattn.load_library()
    cfg, seq = config(*shape, **options), shape[2]
    out = (C.c_int64 * 4)()
    assert lib.ftattn_split_of(C.byref(cfg), out) == 0
    first, piece, shares, state = out
    return first, (-(-(-(-seq // 64)) // piece) if shares else 1), piece, state


def gemm_plan_of(m, n, k, batch=1):
    out = (C.c_int32 * 2)()
    ftattn.load_library().ftgemm_plan_of(C.c_int64(m), C.c_int64(n), C.c_int64(k), C.c_int32(batch), out)
    return TILES[out[0]], out[1]


def test_keys_are_divided_as_the_tests_of_it_say():
    plans = {**split_keys.PLANS, **split_keys.MASKED_PLANS}
    assert {shape: split_of(*shape)[:2] for shape in plans} == plans
    assert max(parts for _, parts in plans.values()) == 16            # all that ftattn_finish takes
    for lo, hi in split_keys.MASKED.values():                         # ... and half of the keys hold a whole share of the longest row tiles
        for shape, (_, parts) in split_keys.MASKED_PLANS.items():
            n, piece = -(-shape[2] // 64), split_of(*shape)[2]
            firsts = [n * p // parts for p in range(parts + 1)]
            assert any(lo * n <= a and b <= hi * n for a, b in zip(firsts, firsts[1:])) and max(b - a for a, b in zip(firsts, firsts[1:])) <= piece


def test_static_call_whose_state_does_not_fit():
    batch, heads, seq, head_dim, causal = shape = split_keys.TOO_LARGE_FOR_STATIC_STATE
    *_, parts, _, state = split_of(*shape)
    tiles_bytes = batch * heads * (seq // 64) * ((64 + 32) * head_dim + (head_dim + 32) * 64) * 2
    assert parts > 1 and tiles_bytes < 60 << 20 and state > 64 << 20


@pytest.mark.parametrize("options", [dict(per_step=1), dict(stride=1), dict(rescale_margin=4.0)])
def test_ablation_modes_are_not_divided(options):
    assert split_of(1, 1, 1024, 128, False, **options)[1] == 1


def test_the_calls_that_are_one_launch():
    lib = ftattn.load_library()
    for shape in one_launch.SHAPES:
        for causal in (False, True):
            for options in ({}, dict(ft_mode=ftattn.FT_OFF), dict(ft_mode=ftattn.FT_DETECT), dict(rowsum_fold=1)):
                one = lib.ftattn_in_one_launch(C.byref(config(*shape, causal, **options)))
                assert one == (shape[2] <= {64: 128, 128: 192}[shape[3]]), (shape, causal, options)
            for options in (dict(per_step=1), dict(per_step=2), dict(stride=1), dict(rescale_margin=4.0)):
                assert lib.ftattn_in_one_launch(C.byref(config(*shape, causal, **options))) == 0
    assert {lib.ftattn_in_one_launch(C.byref(config(*shape, True))) for shape in one_launch.SHAPES} == {0, 1}


def test_tile_shapes_of_the_linear_layer_are_what_the_tests_of_them_say():
    assert {s: (gemm_plan_of(*s), gemm_plan_of(s[1], s[0], s[2])) for s in tiles.PLANS} == tiles.PLANS
    assert {s: gemm_plan_of(*s) for s in narrow.PLANS} == narrow.PLANS
    seen = [plan for pair in tiles.PLANS.values() for plan in pair] + list(narrow.PLANS.values()) + [gemm_plan_of(*s) for s, low in short.SHAPES.items() if low]
    assert TILES[short.LOW] == "low"
    assert {tile for tile, _ in seen} == set(TILES) and {parts for _, parts in seen} == {1, 2, 4, 8, 16}


def test_calls_before_a_replay_have_another_number_of_slots():
    rows = {"wide": 256, "half": 128, "quarter": 64, "strip": 32}
    for (m, n, k), (tile, parts, slots, slots_with_faults) in replay.PLANS.items():
        assert gemm_plan_of(m, n, k) == (tile, parts)
        features = -(-n // 256)
        assert slots == -(-m // (16 if parts > 1 else rows[tile])) * features != slots_with_faults == -(-m // rows["quarter"]) * features
