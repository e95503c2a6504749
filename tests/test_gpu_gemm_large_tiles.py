"""The tiles that only large GEMMs take (96 x 64, 192 x 128, 192 x 256): which calls take them, and those against the fp64
oracle one row and one column chunk past a tile, one short of it, with rows of A on lines and off them.  Tolerance as in
test_gpu_gemm.py."""
import numpy as np
import pytest

from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check, run_gpu
from test_gpu_gemm_block import block_of

SHAPES = {
    (96, 64): [(961, 1096, 2056), (1055, 1024, 1984), (247, 4160, 1704)],
    (192, 128): [(3455, 1544, 1024), (3455, 1528, 1016), (3430, 1536, 1856)],
    (192, 256): [(2113, 3848, 960), (3071, 3576, 968), (5963, 1528, 1272)],
}


@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_shapes_take_the_tile_they_are_meant_for(tile):
    for M, N, K in SHAPES[tile]:
        assert block_of(M, N, K) == tile, (M, N, K)


def test_calls_that_are_not_large_keep_to_the_other_tiles():
    new = set(SHAPES)
    for M, N, K in ((32, 8192, 8192), (1, 4096, 4096), (512, 512, 1136), (8192, 8192, 248), (4096, 4096, 4096), (512, 512, 2048)):
        assert block_of(M, N, K) not in new, (M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_tile_against_the_oracle(tile):
    for n, (M, N, K) in enumerate(SHAPES[tile]):
        for dtype in (I.F16, I.BF16):
            print(f"M{M} N{N} K{K} tile {tile} dtype {dtype}", flush=True)
            ab, bb = I.make_gemm(M, N, K, dtype, seed=900 + n)
            check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"M{M} N{N} K{K} tile {tile}")


@pytest.mark.gpu
@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_zero_fill_past_k_never_meets_an_infinity(tile):
    M, N, K = SHAPES[tile][0]
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=4)
    ab, bb = ab.copy(), np.where(bb == 0, np.uint16(0x3F80), bb).astype(np.uint16)
    ab[M // 2, K - 1] = 0x7F80
    c = run_gpu(ab, bb, 0.1, I.BF16)
    assert not np.isfinite(c[M // 2]).any() and np.isfinite(np.delete(c, M // 2, axis=0)).all()
