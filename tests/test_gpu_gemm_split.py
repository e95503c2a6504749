"""GEMM + LeakyReLU with K split between workgroups (few tiles of C, a long K): the shapes that take it, against
the fp64 oracle at ragged edges of every tile, and the calls that must do without scratch memory."""
import numpy as np
import pytest

from paper_2403_16863_amd import gemm
from paper_2403_16863_amd import inputs as I

# (M, N, K): one past and one short of a tile, last k range short, one key of K past a stage
SPLIT = [(1, 64, 4864), (4, 72, 8136), (33, 40, 5000), (31, 2056, 4872), (3, 3000, 4104), (24, 4096, 4096),
         (65, 1096, 4616), (63, 3592, 4104), (129, 328, 8192), (500, 200, 6008)]
WHOLE = [(1, 64, 4856), (24, 8192, 1024), (512, 512, 2048), (10, 7472, 7680), (4096, 4096, 4096), (24, 4096, 1 << 17)]


def test_few_tiles_and_a_long_k_ask_for_scratch_memory():
    L = gemm.lib()
    for M, N, K in SPLIT:
        need = L.gemm_lrelu_workspace(M, N, K)
        assert need % (M * N * 4) == 0 and 2 <= need // (M * N * 4) <= 16 and need <= 4 << 20, (M, N, K)
    for M, N, K in WHOLE + [(0, 8, 8), (8, 0, 8), (-1, 64, 8192)]:
        assert L.gemm_lrelu_workspace(M, N, K) == 0, (M, N, K)


def test_sizes_near_the_largest_int_ask_for_none():
    """The number of tiles must not overflow (a negative one ended the process with a division by zero)."""
    L = gemm.lib()
    for M, N, K in ((2 ** 31 - 1, 8, 8192), (2 ** 31 - 20, 4096, 8192), (64, 2 ** 31 - 1, 8192), (2 ** 31 - 1,) * 3):
        assert L.gemm_lrelu_workspace(M, N, K) == 0, (M, N, K)


def test_bad_scratch_memory_is_refused_before_any_launch():
    """(fake pointers: nothing is dereferenced)"""
    L = gemm.lib()
    M, N, K = 24, 4096, 4096
    a, b, c, need = 1 << 40, 1 << 41, 1 << 42, L.gemm_lrelu_workspace(M, N, K)
    for ws in ((1 << 43) + 8, a, a - 16, b + 2 * K * N - 16, c, c - need + 16):
        assert L.gemm_lrelu_in(a, b, c, M, N, K, 0.1, 0, None, ws, need) == gemm.GEMM_EINVAL
    assert L.gemm_lrelu_in(a, b, a, M, N, K, 0.1, 0, None, 1 << 43, need) == gemm.GEMM_EINVAL
    assert L.gemm_lrelu_in(a, b, c, M, N, K + 4, 0.1, 0, None, 1 << 43, need) == gemm.GEMM_EINVAL


def test_scratch_memory_is_asked_for_once_in_the_call():
    """After the checks, for the bytes that the shape asks for; what comes back is checked before any launch (fake pointers).
    The native path of a call goes this way, so that a shape is looked at once."""
    L = gemm.lib()
    a, b, c, asked = 1 << 40, 1 << 41, 1 << 42, []

    @gemm.SCRATCH_FN
    def give(owner, nbytes):
        asked.append((owner, nbytes))
        return (1 << 43) + 8
    for M, N, K in ((24, 4096, 4096), (969, 664, 7256)):
        del asked[:]
        assert L.gemm_lrelu_with(a, b, c, M, N, K, 0.1, 0, None, give, 77) == gemm.GEMM_EINVAL
        assert asked == [(77, L.gemm_lrelu_workspace(M, N, K))]
        assert L.gemm_lrelu_with(a, b, a, M, N, K, 0.1, 0, None, give, 77) == gemm.GEMM_EINVAL
        assert L.gemm_lrelu_with(a, b, c, M, N, K + 4, 0.1, 0, None, give, 77) == gemm.GEMM_EINVAL
        assert len(asked) == 1


@pytest.mark.gpu
def test_scratch_memory_that_is_given_given_not_or_not_asked_for():
    import torch
    L = gemm.lib()
    for (M, N, K), split in (((33, 40, 5000), True), ((577, 616, 4552), True), ((100, 72, 328), False)):
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        a, b = (torch.randn(s, device="cuda", generator=g).half() for s in ((M, K), (K, N)))
        plain, want, out = (torch.empty(M, N, device="cuda", dtype=torch.float16) for _ in range(3))
        args = (M, N, K, 0.1, 0, torch.cuda.current_stream().cuda_stream)
        ws, asked = torch.empty(1 << 22, device="cuda"), []
        assert L.gemm_lrelu(a.data_ptr(), b.data_ptr(), plain.data_ptr(), *args) == 0
        assert L.gemm_lrelu_in(a.data_ptr(), b.data_ptr(), want.data_ptr(), *args, ws.data_ptr(), 16 << 20) == 0
        give = gemm.SCRATCH_FN(lambda owner, nbytes: asked.append(nbytes) or owner)
        for fn, owner, expect in ((give, ws.data_ptr(), want), (give, None, plain), (gemm.SCRATCH_FN(0), ws.data_ptr(), plain)):
            out.fill_(float("nan"))
            assert L.gemm_lrelu_with(a.data_ptr(), b.data_ptr(), out.data_ptr(), *args, fn, owner) == 0
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), expect.view(torch.int16))
        assert len(asked) == (2 if split else 0) and all(n <= 16 << 20 for n in asked)
        assert torch.equal(want.view(torch.int16), plain.view(torch.int16)) != split


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
def test_split_against_the_oracle(dtype):
    from test_gpu_gemm import check, run_gpu
    for n, (M, N, K) in enumerate(SPLIT):
        print(f"M{M} N{N} K{K} dtype {dtype}", flush=True)
        ab, bb = I.make_gemm(M, N, K, dtype, seed=500 + n)
        check(run_gpu(ab, bb, 0.1, dtype), ab, bb, 0.1, dtype, f"split M{M} N{N} K{K}")


@pytest.mark.gpu
def test_without_scratch_memory_the_plain_kernel_runs():
    import torch
    L = gemm.lib()
    M, N, K = 33, 40, 5000
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    a, b = (torch.randn(s, device="cuda", generator=g).half() for s in ((M, K), (K, N)))
    plain, out, split = (torch.empty(M, N, device="cuda", dtype=torch.float16) for _ in range(3))
    args = (M, N, K, 0.1, 0, torch.cuda.current_stream().cuda_stream)
    assert L.gemm_lrelu(a.data_ptr(), b.data_ptr(), plain.data_ptr(), *args) == 0
    need = L.gemm_lrelu_workspace(M, N, K)
    ws = torch.full((need // 4,), float("nan"), device="cuda")
    for p, bytes_ in ((None, 0), (None, need), (ws.data_ptr(), need - 1)):
        out.fill_(float("nan"))
        assert L.gemm_lrelu_in(a.data_ptr(), b.data_ptr(), out.data_ptr(), *args, p, bytes_) == 0
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), plain.view(torch.int16))
    assert L.gemm_lrelu_in(a.data_ptr(), b.data_ptr(), split.data_ptr(), *args, ws.data_ptr(), need) == 0
    gemm.gemm_lrelu(a, b, out, 0.1)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), split.view(torch.int16))       # what gemm_lrelu does by itself
    # two fp32 sums of 5000 products each, rounded once: half an ulp of binary16 apart and a little
    assert (split.float() - plain.float()).abs().max() <= 2.0 ** -10 * plain.float().abs().max()
    # a recorded call keeps to the plain kernel, and replays right
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        gemm.gemm_lrelu(a, b, out, 0.1)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        gemm.gemm_lrelu(a, b, split, 0.1)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), plain.view(torch.int16))


@pytest.mark.gpu
def test_calls_on_several_streams_keep_their_parts_apart():
    import torch
    shapes = [(24, 4096, 4096), (16, 512, 8192), (65, 1096, 4616)]
    work = []
    for n, (M, N, K) in enumerate(shapes * 2):
        g = torch.Generator(device="cuda")
        g.manual_seed(n)
        a, b = (torch.randn(s, device="cuda", generator=g).bfloat16() for s in ((M, K), (K, N)))
        want, got = (torch.empty(M, N, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        gemm.gemm_lrelu(a, b, want, 0.01)
        work.append((a, b, want, got, torch.cuda.Stream()))
    torch.cuda.synchronize()
    for rep in range(10):
        for a, b, _, got, st in work:
            with torch.cuda.stream(st):
                gemm.gemm_lrelu(a, b, got, 0.01)
    torch.cuda.synchronize()
    for a, b, want, got, _ in work:
        assert torch.equal(want.view(torch.int16), got.view(torch.int16))


def _case():
    import torch
    M, N, K = 33, 40, 5000
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    a, b = (torch.randn(s, device="cuda", generator=g).half() for s in ((M, K), (K, N)))
    plain, split, out = (torch.empty(M, N, device="cuda", dtype=torch.float16) for _ in range(3))
    L = gemm.lib()
    assert L.gemm_lrelu(a.data_ptr(), b.data_ptr(), plain.data_ptr(), M, N, K, 0.1, 0, torch.cuda.current_stream().cuda_stream) == 0
    gemm.gemm_lrelu(a, b, split, 0.1)
    torch.cuda.synchronize()
    assert not torch.equal(plain, split)               # (other sums: the two can be told apart)
    return a, b, out, plain, split


@pytest.mark.gpu
def test_scratch_memory_only_on_torchs_current_stream():
    """A handle of the caller's own may name another queue than the allocator thinks (2, the per-thread stream, a
    different one in every thread) or be destroyed while its work runs: such calls do without."""
    import torch
    a, b, out, plain, split = _case()
    pool, ext = torch.cuda.Stream(), torch.cuda.ExternalStream(2)
    for stream, current, want in ((None, None, split), (torch.cuda.current_stream().cuda_stream, None, split), (pool.cuda_stream, pool, split),
                                  (None, pool, split), (pool.cuda_stream, None, plain), (2, None, plain), (1, None, plain), (None, ext, plain),
                                  (2, ext, plain)):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(current):
            gemm.gemm_lrelu(a, b, out, 0.1, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), (stream, current)


@pytest.mark.gpu
def test_a_call_beside_a_recording_in_another_thread():
    """A recording in torch's default mode refuses allocations of every thread; the call's scratch memory must not
    end it, nor come from the recording's pool."""
    import threading
    import torch
    a, b, out, plain, split = _case()
    own, side = torch.cuda.Stream(), torch.cuda.Stream()
    x, y = torch.arange(8.0, device="cuda"), torch.zeros(8, device="cuda")
    errors = []

    def call():
        try:
            with torch.cuda.stream(own):
                gemm.gemm_lrelu(a, b, out, 0.1)
        except Exception as e:
            errors.append(e)

    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    with torch.cuda.graph(graph, stream=side):
        torch.add(x, 1, out=y)
        t = threading.Thread(target=call)
        t.start()
        t.join()
        y.mul_(2)
    assert not errors
    torch.cuda.synchronize()
    assert torch.equal(out, split) or torch.equal(out, plain)
    for _ in range(3):
        y.zero_()
        graph.replay()
        gemm.gemm_lrelu(a, b, out, 0.1)
        torch.cuda.synchronize()
        assert torch.equal(y, 2 * (x + 1)) and torch.equal(out, split)
