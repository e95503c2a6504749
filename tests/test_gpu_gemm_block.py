"""GPU parity of every tile shape gemm_lrelu chooses from with the fp64 oracle, at sizes where a tile
can go wrong: one row or column chunk past a tile edge, one chunk short of it, k inside, at and past a
stage.  Tolerance as in test_gpu_gemm.py (derived from the fp32 sums and one rounding)."""
import ctypes

import numpy as np
import pytest

from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check, run_gpu


def block_of(M, N, K):
    from paper_2403_16863_amd import gemm
    bm, bn = ctypes.c_int(0), ctypes.c_int(0)
    assert gemm.lib().gemm_lrelu_block_of(M, N, K, ctypes.byref(bm), ctypes.byref(bn)) == 0
    return bm.value, bn.value


def launch_of(M, N, K, base=0, scratch=True):
    """(bm, bn, threads, workgroups per unit, 1 for A by whole lines, ranges of K, kc) for A at `base` bytes behind a line."""
    from paper_2403_16863_amd import gemm
    out = (ctypes.c_int * 7)()
    assert gemm.lib().gemm_lrelu_launch_of(M, N, K, base, int(scratch), out) == 0
    return tuple(out)


SHAPES = {
    (32, 32): [(1, 8, 240), (31, 264, 520), (65, 40, 1000), (33, 608, 2384)],
    (32, 64): [(97, 2088, 328), (511, 720, 392), (2047, 256, 1000)],
    (64, 64): [(1, 8, 24), (33, 24, 128), (193, 2824, 384), (5055, 96, 72), (4033, 136, 1000)],
    (64, 128): [(5185, 360, 456), (1000, 1032, 776), (1025, 1000, 792)],
    (128, 128): [(1281, 1544, 520), (4095, 568, 248), (3841, 776, 8)],
    (128, 256): [(3090, 2008, 8), (4095, 1520, 160), (1889, 2224, 952)],
    (256, 256): [(3841, 2128, 136), (4095, 2136, 456)],
}


@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_shapes_take_the_tile_they_are_meant_for(tile):
    for M, N, K in SHAPES[tile]:
        assert block_of(M, N, K) == tile, (M, N, K)


def test_huge_k_falls_back_to_tiles_whose_offsets_fit():
    """(bm - 1) * K * 2 has to stay below 2^31."""
    for K in ((1 << 22) - 8, 1 << 22, (1 << 24) - 8):
        bm, _ = block_of(1 << 16, 1 << 16, K)
        assert (bm - 1) * K * 2 + 128 < 1 << 31


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_tile_against_the_oracle(tile, dtype):
    for n, (M, N, K) in enumerate(SHAPES[tile]):
        print(f"M{M} N{N} K{K} tile {tile} dtype {dtype}", flush=True)
        ab, bb = I.make_gemm(M, N, K, dtype, seed=300 + n)
        check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"M{M} N{N} K{K} tile {tile}")


@pytest.mark.gpu
@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}")
def test_zero_fill_past_k_never_meets_an_infinity(tile):
    """An infinity in the last column of A stays in its row of C: the chunks past K are exact zeros on both sides."""
    M, N, K = next(s for s in SHAPES[tile] if s[2] % 64)
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=4)
    ab, bb = ab.copy(), np.where(bb == 0, np.uint16(0x3F80), bb).astype(np.uint16)
    ab[M // 2, K - 1] = 0x7F80
    c = run_gpu(ab, bb, 0.1, I.BF16)
    assert not np.isfinite(c[M // 2]).any() and np.isfinite(np.delete(c, M // 2, axis=0)).all()
