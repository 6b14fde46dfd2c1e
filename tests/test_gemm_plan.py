"""CPU checks of the tile and split choice, and that the sizes of the GPU tests
reach every tile, split and epilogue: a change of the estimate that takes a
kernel out of their reach fails here."""
import random

import pytest

import test_gpu_gemm as g
from paper_2609_13645_amd import _lib

LAYOUTS = [(0, 0), (0, 1), (1, 1)]
TILES = {(256, 256), (128, 256), (128, 128), (64, 64)}
PLENTY = 1 << 40


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_gpu_sizes_reach_every_tile(la, lb):
    assert {_lib.forge_gemm_plan(la, lb, *s)[:2] for s in g.TILE_SIZES} == TILES


@pytest.mark.parametrize("la,lb", LAYOUTS)
def test_padding_counts_against_large_tiles(la, lb):
    """A chip of 256 x 256 tiles that are mostly padding is no reason to take
    them: no jump where their number reaches the CUs'."""
    for M, N in ((64, 65280), (64, 65536), (65536, 64), (8, 100000), (128, 131072)):
        assert _lib.forge_gemm_plan(la, lb, M, N, 2048)[:2] != (256, 256), (M, N)
    for M, N in ((4096, 4096), (4000, 4008), (192, 131072), (16384, 1024)):
        assert _lib.forge_gemm_plan(la, lb, M, N, 2048)[:2] == (256, 256), (M, N)


def test_short_reductions_on_many_small_tiles():
    # data gradients of 40 to 200: more than a round of 64 x 64 tiles
    for M, N, K in ((1792, 1800, 40), (2016, 1480, 72), (3056, 1120, 72), (328, 7520, 184)):
        assert _lib.forge_gemm_plan(0, 1, M, N, K)[:2] == (128, 128), (M, N, K)


@pytest.mark.parametrize("la,lb,M,N,K,tile,splits", g.SPLITS)
def test_gpu_split_sizes_split_as_they_say(la, lb, M, N, K, tile, splits):
    tm, tn, s, n = _lib.forge_gemm_plan(la, lb, M, N, K, PLENTY)
    assert ((tm, tn), s) == (tile, splits)
    assert n == 4 * s * M * ((N + 7) // 8 * 8)
    assert _lib.forge_gemm_plan(la, lb, M, N, K)[2:] == (1, 0)
    # scratch for fewer: fewer splits that fit it
    t = _lib.forge_gemm_plan(la, lb, M, N, K, n - 1)
    assert t[2] < s and t[3] < n


def test_gpu_split_sizes_reach_every_split_tile():
    assert {(la, lb, tile) for la, lb, _, _, _, tile, _ in g.SPLITS} == {
        (la, lb, t) for la, lb in LAYOUTS for t in TILES}


@pytest.mark.parametrize("sizes,N,K,tile", g.GROUPED)
def test_gpu_grouped_sizes_take_the_tile_they_say(sizes, N, K, tile):
    for lb in (0, 1):
        assert _lib.forge_gemm_grouped_rows_tile(lb, len(sizes), sum(sizes) + 40, N, K) == tile


def test_plan_of_any_size():
    """Splits cover the reduction with none empty, stay within a round of
    workgroups and within 64 MB, and never need more than the scratch."""
    rng = random.Random(5)
    for la, lb in LAYOUTS:
        for _ in range(3000):
            M, N, K = (8 * int(2 ** rng.uniform(0, 11)) for _ in range(3))
            scratch = rng.choice([0, 1 << 16, 1 << 22, PLENTY])
            tm, tn, s, n = _lib.forge_gemm_plan(la, lb, M, N, K, scratch)
            assert (tm, tn) in TILES and 1 <= s <= 16 and n <= scratch and n <= 64 << 20
            if s > 1:
                ks = ((K + s - 1) // s + 63) // 64 * 64
                assert (s - 1) * ks < K <= s * ks
                assert s * -(-M // tm) * -(-N // tn) <= 256


def test_plan_argument_rules():
    for args, status in [((1, 0, 64, 64, 64), _lib.FORGE_ERR_UNSUPPORTED),
                         ((0, 0, 64, 64, 12), _lib.FORGE_ERR_INVALID_ARG),
                         ((0, 1, 64, 12, 64), _lib.FORGE_ERR_INVALID_ARG),
                         ((1, 1, 12, 64, 64), _lib.FORGE_ERR_INVALID_ARG),
                         ((0, 0, 0, 64, 64), _lib.FORGE_ERR_INVALID_ARG)]:
        with pytest.raises(_lib.ForgeError) as e:
            _lib.forge_gemm_plan(*args)
        assert e.value.status == status
    P = (0x1000, 0x2000, 0x3000, None, 64, 64, 64, 64, 64, 64, 0)
    for tail, status in [((1.0, None, 16, 0), _lib.FORGE_ERR_INVALID_ARG),
                         ((1.0, 0x1008, 1 << 20, 0), _lib.FORGE_ERR_ALIGNMENT),
                         ((float("inf"), 0x1000, 1 << 20, 0), _lib.FORGE_ERR_INVALID_ARG)]:
        with pytest.raises(_lib.ForgeError) as e:
            _lib.forge_gemm_scratch(0, 0, 0, *P, *tail)
        assert e.value.status == status
    with pytest.raises(_lib.ForgeError):
        _lib.forge_gemm_grouped_rows_tile(0, 0, 64, 64, 64)
