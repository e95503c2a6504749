"""GEMMs of a short K on 128 x 128 tiles in more than one round, which run two workgroups on a unit: the edges of tiles, and K
of one chunk, one stage, one chunk past it and several, against the fp64 oracle.  Tolerance as in test_gpu_gemm.py."""
import numpy as np
import pytest

from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check, run_gpu
from test_gpu_gemm_block import launch_of

SHAPES = [(6529, 1032, 8), (6655, 1032, 64), (5377, 1288, 72), (6529, 1032, 136), (6655, 1032, 504), (6529, 1032, 632)]


def test_shapes_are_what_they_stand_for():
    """Two workgroups on a unit for these; one from K = 640 on and for 256 tiles."""
    for M, N, K in SHAPES:
        assert launch_of(M, N, K)[:4] == (128, 128, 512, 2) and -(-M // 128) * -(-N // 128) > 256, (M, N, K)
    for M, N, K in ((6529, 1032, 640), (2048, 2048, 504), (2048, 2048, 632)):
        assert launch_of(M, N, K)[:4] == (128, 128, 512, 1), (M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_against_the_oracle(M, N, K, dtype):
    ab, bb = I.make_gemm(M, N, K, dtype, seed=K)
    check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"M{M} N{N} K{K}")


@pytest.mark.gpu
def test_zero_fill_past_k_never_meets_an_infinity():
    M, N, K = SHAPES[3]
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=4)
    ab, bb = ab.copy(), np.where(bb == 0, np.uint16(0x3F80), bb).astype(np.uint16)
    ab[M // 2, K - 1] = 0x7F80
    c = run_gpu(ab, bb, 0.1, I.BF16)
    assert not np.isfinite(c[M // 2]).any() and np.isfinite(np.delete(c, M // 2, axis=0)).all()
