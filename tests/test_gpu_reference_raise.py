"""Scores that step up between one key tile and the next, by a little less and a little more than the
room the kernels leave above the reference maximum (14 binades in binary16, 16 in bfloat16, per lane's
partial row sum), and by far more: every variant against the fp64 oracle."""
import numpy as np
import pytest

from oracle import ref
from paper_2403_16863_amd import inputs as I

from gpu_util import check, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("binades", [7, 9, 13, 15, 17, 60])
def test_step_between_tiles(binades, d, dtype):
    import paper_2403_16863_amd as A
    N, causal = 200, False
    w = I.Workload("step", 1, 2, N, d, causal, dtype)
    g = np.random.default_rng(binades)
    q = np.zeros((1, 2, N, d), np.float32)
    k = g.standard_normal((1, 2, N, d)).astype(np.float32)
    q[..., 0] = 8.0
    k[..., 0] = 0.0
    # one key of every 64-key tile after the first (its score alone decides the lane's sum)
    k[..., 70, 0] = binades * np.log(2.0) / (8.0 * w.scale)
    k[..., 140, 0] = 2 * binades * np.log(2.0) / (8.0 * w.scale)
    v = g.standard_normal((1, 2, N, d)).astype(np.float32)
    qb, kb, vb = (I.f32_to_bits(x, dtype) for x in (q, k, v))
    O_ref, l_ref, _ = ref.attn_ref(qb, kb, vb, causal, w.scale, dtype)
    for var in [None] + [x for x in range(A.attn_num_variants()) if A.attn_variant_supported(x, d, dtype, causal)]:
        O, l = run_gpu(qb, kb, vb, causal, w.scale, dtype, variant=var)
        check(O, l, O_ref, l_ref, dtype, what=f"step of {binades} binades d={d} dt={dtype} var={var}")
