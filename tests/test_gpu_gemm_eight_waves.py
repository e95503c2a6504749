"""The 64 x 64 tile on eight waves (two groups of four that split K): which calls take it, and those against the fp64
oracle at the edges of tiles and of the groups' stages.  Tolerance as in test_gpu_gemm.py."""
import numpy as np
import pytest

from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check, run_gpu
from test_gpu_gemm_block import block_of

SHAPES = [(833, 840, 2120), (833, 840, 1280), (449, 1096, 2440), (1023, 968, 2184), (769, 776, 3000), (833, 832, 2048)]


def test_which_calls_take_it():
    from paper_2403_16863_amd import gemm
    L = gemm.lib()
    for M, N, K in SHAPES:
        assert block_of(M, N, K) == (64, 64) and L.gemm_lrelu_block_threads_of(M, N, K) == 512
    # a short K
    for M, N, K in ((705, 712, 1000), (193, 2824, 384), (705, 712, 960)):
        assert block_of(M, N, K) == (64, 64) and L.gemm_lrelu_block_threads_of(M, N, K) == 256
    # K a multiple of 64 (whole lines of A) or not, on both sides of the line for the latter
    for K, threads in ((1152, 512), (1144, 256), (1160, 256), (1920, 512), (1928, 256), (2104, 256), (2112, 512), (2120, 512)):
        assert block_of(833, 840, K) == (64, 64) and L.gemm_lrelu_block_threads_of(833, 840, K) == threads


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
def test_eight_waves_against_the_oracle(dtype):
    for n, (M, N, K) in enumerate(SHAPES):
        print(f"M{M} N{N} K{K} dtype {dtype}", flush=True)
        ab, bb = I.make_gemm(M, N, K, dtype, seed=500 + n)
        check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"M{M} N{N} K{K}")


@pytest.mark.gpu
def test_zero_fill_past_k_never_meets_an_infinity():
    M, N, K = SHAPES[0]
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=4)
    ab, bb = ab.copy(), np.where(bb == 0, np.uint16(0x3F80), bb).astype(np.uint16)
    ab[M // 2, K - 1] = 0x7F80
    c = run_gpu(ab, bb, 0.1, I.BF16)
    assert not np.isfinite(c[M // 2]).any() and np.isfinite(np.delete(c, M // 2, axis=0)).all()
