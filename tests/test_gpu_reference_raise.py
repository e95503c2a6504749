"""Scores that step up between one key tile and the next, by a little less and a little more than the
room the kernels leave above the reference maximum (8 binades, per lane's partial row sum), and by far more:
every variant against the fp64 oracle."""
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


@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_a_dominating_key_is_not_rounded(d, dtype):
    """A key 9.3 to 13.7 binades above all others raises the reference, and its probability is then exactly 1: what
    is left is the rounding of the result and of the other keys' probabilities, |dO| <= u |O| + u sum p |v| over the
    others + 2^-20 max|v| for the fp32 terms.  Rounded to 16 bits itself, it would add up to u |v|."""
    import paper_2403_16863_amd as A
    from gpu_util import U
    N = 200
    w = I.Workload("dominating", 1, 4, N, d, False, dtype)
    g = np.random.default_rng(d)
    q = np.zeros((1, 4, N, d), np.float32)
    k = np.zeros((1, 4, N, d), np.float32)
    q[..., 0] = 8.0
    for h, binades in enumerate((9.3, 10.6, 12.4, 13.7)):
        k[0, h, 150, 0] = binades * np.log(2.0) / (8.0 * w.scale)
    v = g.standard_normal((1, 4, N, d)).astype(np.float32)
    qb, kb, vb = (I.f32_to_bits(x, dtype) for x in (q, k, v))
    O_ref, l_ref, _ = ref.attn_ref(qb, kb, vb, False, w.scale, dtype)
    v64 = I.bits_to_f64(vb, dtype)
    p_other = np.exp(-l_ref[..., 0])                         # (the other scores are 0)
    others = np.abs(np.delete(v64, 150, axis=2)).sum(axis=2) * p_other[..., None]
    bound = U[dtype] * (np.abs(O_ref) + others[:, :, None]) + 2.0 ** -20 * np.abs(v64).max()
    for var in [None] + [x for x in range(A.attn_num_variants()) if A.attn_variant_supported(x, d, dtype, False)]:
        O, l = run_gpu(qb, kb, vb, False, w.scale, dtype, variant=var)
        worst = float((np.abs(O - O_ref) / bound).max())
        print(f"case d={d} dt={dtype} var={var}: {worst:.3f} of the bound", flush=True)
        assert worst <= 1.0, (var, worst)
