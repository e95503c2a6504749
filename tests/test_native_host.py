"""The native call path refuses whatever is not a plain call, and the Python path then names what is wrong."""
import numpy as np
import pytest
import torch

import paper_2403_16863_amd as A
from paper_2403_16863_amd import binding, gemm


def test_calls_that_are_not_plain_are_left_to_python():
    n = binding.native()
    t = torch.zeros(1, 1, 8, 64, dtype=torch.float16)
    for args in ((), (t,) * 8, (1, 2, 3, 4, 5, 6, 7, 8), (t, t, t, t, t[..., 0].float(), False, 1.0, None),
                 (t, t, t, t, t[..., 0].float(), False, "x", None), (np.zeros(3),) * 8):
        assert n.attn_fwd(*args) == n.NOT_PLAIN
    for args in ((), (t[0, 0],) * 5, (t[0, 0], t[0, 0].t(), t[0, 0], 0.1, None), (1, 2, 3, 4, 5)):
        assert n.gemm_lrelu(*args) == n.NOT_PLAIN


def test_errors_are_those_of_the_python_path():
    t = torch.zeros(1, 1, 8, 64, dtype=torch.float16)
    with pytest.raises(ValueError, match="device memory"):
        A.attn_fwd(t, t, t, t, t[..., 0].float(), False, 1.0)
    with pytest.raises(ValueError, match="device memory"):
        gemm.gemm_lrelu(t[0, 0], t[0, 0], t[0, 0], 0.1)


def test_tensors_without_storage_raise_in_python():
    """Inside vmap a tensor has no data pointer: torch's exception must not end the process."""
    from torch._subclasses.fake_tensor import FakeTensorMode
    n = binding.native()
    with FakeTensorMode():
        x, y = torch.empty(2, 1, 1, 8, 64, dtype=torch.float16, device="cuda"), torch.empty(2, 1, 1, 8, device="cuda")

        def native_calls(t, l):
            s = torch.empty_like(t[0, 0, :, :8].contiguous())
            assert n.attn_fwd(t, t, t, t, l, False, 1.0, 0) == n.NOT_PLAIN
            assert n.gemm_lrelu(s, s, s, 1.0, 0) == n.NOT_PLAIN
            with pytest.raises(RuntimeError):
                A.attn_fwd(t, t, t, t, l, False, 1.0, stream=0)
            return l
        torch.func.vmap(native_calls)(x, y)


@pytest.mark.gpu
def test_native_and_python_paths_agree_on_results_errors_and_streams():
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q, k, v = (torch.randn(1, 3, 200, 64, device="cuda", generator=g).half() for _ in range(3))
    want, lse_w = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
    A.attn_fwd_variant(q, k, v, want, lse_w, True, 0.125, A.attn_deployed(200, 64, 0, True)[1])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    for how in ("current", "with", "argument"):
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
        torch.cuda.synchronize()
        if how == "with":
            with torch.cuda.stream(side):
                A.attn_fwd(q, k, v, out, lse, 1, np.float32(0.125))
        else:
            A.attn_fwd(q, k, v, out, lse, True, 0.125, stream=side.cuda_stream if how == "argument" else None)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)) and torch.equal(lse, lse_w), how
    with pytest.raises(A.AttnError):
        A.attn_fwd(q, k, v, q, lse, True, 0.125)                       # out aliases q: the library's own code
    with pytest.raises(A.AttnError):
        A.attn_fwd(q, k, v, out, lse, True, float("inf"))
    with pytest.raises(ValueError):
        A.attn_fwd(q, k, v.transpose(1, 2), out, lse, True, 0.125)
    with pytest.raises(ValueError):
        A.attn_fwd(q, k, v, out, lse.half(), True, 0.125)
    with pytest.raises(TypeError):
        A.attn_fwd(*(t.float() for t in (q, k, v, out)), lse, True, 0.125)
