"""GEMM + LeakyReLU where rows of A do not start on 128-byte lines: every phase of a row against the lines (K / 8 modulo
8, and the base of A in 16-byte steps), on every tile that takes A by whole lines, and both that do so with K split.  Tolerance as in test_gpu_gemm.py."""
import numpy as np
import pytest

from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check
from test_gpu_gemm_block import launch_of

# (tile, ranges of K): (M, N, K of the eight phases): a row and a column chunk past a tile, or one short of it
SHAPES = {
    (64, 64, 0): (833, 840, 2112),
    (64, 128, 0): (2049, 776, 1344),
    (96, 64, 0): (961, 1096, 2048),
    (128, 128, 0): (1281, 1544, 768),
    (128, 256, 0): (2113, 2824, 960),
    (192, 128, 0): (3455, 1544, 1024),
    (192, 256, 0): (3071, 3576, 960),
    (256, 256, 0): (3841, 2128, 768),
    (128, 128, 6): (577, 616, 4544),
    (192, 128, 8): (180, 2888, 8128),
}


def run_tensor(ab, bb, dtype, offset):
    """C (a tensor) with A at `offset` 16-byte chunks behind a line, and NaN in front of and behind it."""
    import torch
    from paper_2403_16863_amd import gemm
    M, K = ab.shape
    room = torch.full((M * K + 128,), 0x7FFF, dtype=torch.int16, device="cuda:0")
    a = room[64 + 8 * offset:][:M * K].view(M, K)
    a.copy_(torch.from_numpy(ab.view(np.int16)))
    tdt = torch.bfloat16 if dtype == I.BF16 else torch.float16
    b = torch.from_numpy(bb.view(np.int16)).to("cuda:0").view(tdt)
    assert (a.data_ptr() & 127) == 16 * offset
    c = torch.full((M, bb.shape[1]), float("nan"), dtype=tdt, device="cuda:0")
    gemm.gemm_lrelu(a.view(tdt), b, c, 0.1)
    torch.cuda.synchronize()
    return c


def run(ab, bb, dtype, offset):
    return run_tensor(ab, bb, dtype, offset).double().cpu().numpy()


@pytest.mark.parametrize("M,N,K,base,tile,lines", [
    (1025, 1000, 776, 0, (64, 128), 0), (2049, 776, 1272, 0, (64, 128), 0), (2049, 776, 1280, 0, (64, 128), 0),
    (2049, 776, 1280, 16, (64, 128), 1), (2049, 776, 1288, 0, (64, 128), 1), (1281, 1544, 760, 0, (128, 128), 0),
    (1281, 1544, 768, 0, (128, 128), 0), (1281, 1544, 768, 112, (128, 128), 1), (1281, 1544, 776, 0, (128, 128), 1),
    (833, 840, 2112, 16, (64, 64), 0), (833, 840, 2120, 0, (64, 64), 1), (961, 1032, 1664, 16, (96, 64), 0), (961, 1032, 1672, 16, (96, 64), 1)])
def test_which_calls_take_a_by_whole_lines(M, N, K, base, tile, lines):
    """From a K on that is measured for each tile; a base off the line alone only where the order of the sums stays the same."""
    got = launch_of(M, N, K, base)
    assert (got[:2], got[4], got[5]) == (tile, lines, 0)


def offset_of(n):
    return (0, 1, 0, 7, 4, 0, 2, 5)[n]


@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}" + f" {t[2]} ranges" * (t[2] > 0))
def test_shapes_take_the_kernel_they_are_meant_for(tile):
    M, N, K0 = SHAPES[tile]
    groups = tile in ((64, 64, 0), (96, 64, 0))     # two groups of waves: off the lines by K alone
    for n in range(9):
        K, offset = (K0 + 8 * n, offset_of(n)) if n < 8 else (K0, 3)
        bm, bn, threads, _, lines, ranges, _ = launch_of(M, N, K, 16 * offset)
        assert (bm, bn, ranges) == tile and lines == (K % 64 != 0 or (offset > 0 and not groups)), (K, offset)
        assert tile != (64, 64, 0) or threads == 512


@pytest.mark.gpu
@pytest.mark.parametrize("tile", sorted(SHAPES), ids=lambda t: f"{t[0]}x{t[1]}" + f" {t[2]} ranges" * (t[2] > 0))
def test_every_phase_of_the_rows(tile):
    M, N, K0 = SHAPES[tile]
    for n in range(8):
        K, offset, dtype = K0 + 8 * n, offset_of(n), (I.F16, I.BF16)[n & 1]
        print(f"M{M} N{N} K{K} base {offset} dtype {dtype}", flush=True)
        ab, bb = I.make_gemm(M, N, K, dtype, seed=700 + n)
        check(run(ab, bb, dtype, offset), ab, bb, 0.1, dtype, f"M{M} N{N} K{K} base {offset}")
    K, dtype = K0, I.BF16               # rows that are whole lines, off the lines by the base alone
    ab, bb = I.make_gemm(M, N, K, dtype, seed=710)
    check(run(ab, bb, dtype, 3), ab, bb, 0.1, dtype, f"M{M} N{N} K{K} base 3")


# both forms of every tile that has two, and K no multiple of 64; the last two split K (128 x 128 and 192 x 128 tiles)
PLACES = [(833, 840, 2112), (833, 840, 2120), (1055, 1024, 1984), (1055, 1024, 1992), (2049, 776, 1280), (1281, 1544, 1024), (3455, 1544, 1024),
          (2113, 2824, 1024), (3071, 3576, 1024), (3841, 2128, 1024), (969, 640, 7232), (180, 2880, 8192)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", PLACES)
def test_the_place_of_a_does_not_change_a_bit(M, N, K):
    import torch
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=720)
    want = run_tensor(ab, bb, I.BF16, 0).view(torch.int16)
    for offset in (1, 4):
        assert torch.equal(run_tensor(ab, bb, I.BF16, offset).view(torch.int16), want), offset
