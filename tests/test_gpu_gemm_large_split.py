"""Large GEMMs with K split between workgroups on 128 x 128, 192 x 128 and 64 x 64 tiles: which calls take it and how much scratch
memory, those against the fp64 oracle at the edges of tiles and ranges, with rows of A on lines and off them, and the call that
gets none.  Tolerance as in test_gpu_gemm.py."""
import numpy as np
import pytest

from paper_2403_16863_amd import gemm
from paper_2403_16863_amd import inputs as I

from test_gpu_gemm import check, run_gpu
from test_gpu_gemm_block import launch_of

# (M, N, K, ranges, tile, 1 for A by whole lines)
SPLIT = [(969, 664, 7256, 5, (128, 128), 1), (2097, 464, 5744, 5, (192, 128), 1), (1153, 648, 7240, 6, (192, 128), 1), (180, 2880, 8192, 8, (192, 128), 0),
         (4385, 192, 6976, 5, (192, 128), 0), (577, 616, 4552, 6, (128, 128), 1), (162, 800, 4512, 6, (64, 64), 0), (127, 1272, 3560, 6, (64, 64), 0),
         (969, 640, 7232, 6, (128, 128), 0), (577, 616, 4544, 6, (128, 128), 0)]


def ranges_of(M, N, K):
    need = gemm.lib().gemm_lrelu_workspace(M, N, K)
    assert need % (M * N * 4) == 0 and need <= 24 << 20
    return need // (M * N * 4)


def test_which_calls_are_split():
    for M, N, K, ranges, tile, lines in SPLIT:
        got = launch_of(M, N, K)
        assert ranges_of(M, N, K) == ranges and (got[:2], got[4], got[5]) == (tile, lines, ranges), (M, N, K)
        assert launch_of(M, N, K, scratch=False)[5] == 0
    for M, N, K in ((4096, 4096, 4096), (2048, 8192, 2048), (1000, 1032, 2056), (969, 664, 1016), (8192, 8192, 8192), (300, 8192, 1 << 17),
                    (451, 1184, 3648), (410, 200, 3800), (65, 2016, 3536)):
        assert ranges_of(M, N, K) == 0, (M, N, K)


def test_parts_stay_below_the_limit():
    """One tile of 192 x 128 floats for each of 256 units at most, as the header says."""
    assert ranges_of(384, 4096, 7936) * 384 * 4096 * 4 == 24 << 20
    for M in range(33, 8192, 411):
        for N in range(64, 8192, 808):
            for K in (1024, 2056, 4104, 8192, 65536):
                assert ranges_of(M, N, K) <= 16


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
def test_split_against_the_oracle(dtype):
    for n, (M, N, K, *_) in enumerate(SPLIT):
        print(f"M{M} N{N} K{K} dtype {dtype}", flush=True)
        ab, bb = I.make_gemm(M, N, K, dtype, seed=950 + n)
        check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"split M{M} N{N} K{K}")


@pytest.mark.gpu
def test_zero_fill_past_a_range_never_meets_an_infinity():
    """An infinity in the last column of A, and one in the first column of a range, stay in their rows of C."""
    M, N, K, ranges = SPLIT[2][:4]
    ab, bb = I.make_gemm(M, N, K, I.BF16, seed=4)
    ab, bb = ab.copy(), np.where(bb == 0, np.uint16(0x3F80), bb).astype(np.uint16)
    kc = (-(-K // ranges) + 63) // 64 * 64
    ab[M // 2, K - 1] = ab[M // 3, kc] = 0x7F80
    c = run_gpu(ab, bb, 0.1, I.BF16)
    rows = [M // 2, M // 3]
    assert not np.isfinite(c[rows]).any() and np.isfinite(np.delete(c, rows, axis=0)).all()


@pytest.mark.gpu
def test_without_scratch_memory_the_whole_call_runs():
    import torch
    L = gemm.lib()
    M, N, K = SPLIT[0][:3]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    a, b = (torch.randn(s, device="cuda", generator=g).half() for s in ((M, K), (K, N)))
    plain, out, split = (torch.empty(M, N, device="cuda", dtype=torch.float16) for _ in range(3))
    args = (M, N, K, 0.1, 0, torch.cuda.current_stream().cuda_stream)
    assert L.gemm_lrelu(a.data_ptr(), b.data_ptr(), plain.data_ptr(), *args) == 0
    need = L.gemm_lrelu_workspace(M, N, K)
    ws = torch.full((need // 4,), float("nan"), device="cuda")
    assert L.gemm_lrelu_in(a.data_ptr(), b.data_ptr(), out.data_ptr(), *args, ws.data_ptr(), need - 1) == 0
    assert L.gemm_lrelu_in(a.data_ptr(), b.data_ptr(), split.data_ptr(), *args, ws.data_ptr(), need) == 0
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), plain.view(torch.int16))
    assert not torch.equal(split.view(torch.int16), plain.view(torch.int16))
    gemm.gemm_lrelu(a, b, out, 0.1)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), split.view(torch.int16))
    # two fp32 sums of 7256 products each, rounded once: half an ulp of binary16 apart and a little
    assert (split.float() - plain.float()).abs().max() <= 2.0 ** -10 * plain.float().abs().max()
