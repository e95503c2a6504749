"""The work that a user of this framework has it do, as measurable cases: fused attention forward
(`attn_fwd`) and fused GEMM + LeakyReLU (`gemm.gemm_lrelu`), through the package's own entry points.

Inputs are already in device memory and the outputs are caller-owned buffers, as both entry points
ask; a pass is one call.  The library has no backward pass and no separate decode path: every
attention call is self-attention over N queries and N keys.
"""
import math

import torch

import paper_2403_16863_amd as A
from paper_2403_16863_amd import gemm

_DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


def _attn(name, B, H, N, d, causal, dtype, qk_sigma=1.0):
    return {"name": name, "op": "attn", "B": B, "H": H, "N": N, "d": d, "causal": causal, "dtype": dtype, "qk_sigma": qk_sigma}


def _gemm(name, M, N, K, dtype, slope=0.01):
    return {"name": name, "op": "gemm", "M": M, "N": N, "K": K, "dtype": dtype, "slope": slope}


def listed():
    return [
        # the smallest call: one short prompt, two heads; launch and host time count
        _attn("attn_tiny_f16", 1, 2, 128, 64, False, "f16"),
        # few heads and a length that is no multiple of any tile: one request of a small model
        _attn("attn_ragged_f16", 2, 3, 1000, 128, False, "f16"),
        # short training sequences, head dimension 64
        _attn("attn_short_f16", 4, 16, 1024, 64, True, "f16"),
        # encoder-style attention with a peaked softmax, head dimension 64
        _attn("attn_encoder_f16", 8, 16, 2048, 64, False, "f16", qk_sigma=2.0),
        # the shape the paper tunes its attention kernel on: one long sequence, four heads
        _attn("attn_paper_f16", 1, 4, 16384, 64, False, "f16"),
        # pre-training layer: two sequences, 32 heads, causal
        _attn("attn_train_bf16", 2, 32, 4096, 128, True, "bf16"),
        # long-context prefill of one sequence (the benchmark's default workload)
        _attn("attn_prefill_bf16", 1, 32, 16384, 128, True, "bf16"),
        # the shape the paper tunes its GEMM + LeakyReLU kernel on
        _gemm("gemm_paper_f16", 512, 512, 2048, "f16"),
        # a batch of 24 rows through one layer: the weights are read once, memory-bound
        _gemm("gemm_rows24_bf16", 24, 4096, 4096, "bf16"),
        # sizes that are no multiples of a tile
        _gemm("gemm_ragged_f16", 1000, 1032, 2056, "f16"),
        # a widening layer of a small model
        _gemm("gemm_wide_f16", 2048, 8192, 2048, "f16"),
        # a square layer of a large batch
        _gemm("gemm_square_bf16", 4096, 4096, 4096, "bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: attention over 64 to 16384 keys and 2 to 128 heads, GEMM over
    1 to 8192 rows and multiples of 8 from 64 to 8192 in the other two sizes."""
    if rng.random() < 0.6:
        while True:
            B, H = rng.choice((1, 2, 4, 8)), rng.choice((2, 3, 4, 6, 8, 12, 16, 32))
            N = _log_uniform(rng, 64, 16384)
            d, causal, dtype = rng.choice((64, 128)), rng.random() < 0.5, rng.choice(("f16", "bf16"))
            c = _attn("", B, H, N, d, causal, dtype, qk_sigma=rng.choice((1.0, 1.0, 2.0)))
            # no dearer than the listed prefill (d = 64 runs at a lower rate: the exponentials bind there)
            if B * H <= 128 and work(c)["flops"] <= (1.6e12 if d == 128 else 1e12):
                break
    else:
        while True:
            M, N, K = _log_uniform(rng, 1, 8192), 8 * _log_uniform(rng, 8, 1024), 8 * _log_uniform(rng, 8, 1024)
            c = _gemm("", M, N, K, rng.choice(("f16", "bf16")), slope=rng.choice((0.0, 0.01, 0.2)))
            if work(c)["flops"] <= 1.4e11:
                break
    del c["name"]
    return c


def _normal(g, shape, dtype, sigma=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(sigma).to(dtype)


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = _DTYPES[case["dtype"]]
    if case["op"] == "attn":
        shape = (case["B"], case["H"], case["N"], case["d"])
        q, k = _normal(g, shape, dt, case["qk_sigma"]), _normal(g, shape, dt, case["qk_sigma"])
        v = _normal(g, shape, dt)
        return {"op": "attn", "q": q, "k": k, "v": v, "out": torch.empty_like(q),
                "lse": torch.empty(shape[:3], device="cuda", dtype=torch.float32),
                "causal": case["causal"], "scale": case["d"] ** -0.5}
    M, N, K = case["M"], case["N"], case["K"]
    return {"op": "gemm", "a": _normal(g, (M, K), dt), "b": _normal(g, (K, N), dt),
            "c": torch.empty((M, N), device="cuda", dtype=dt), "slope": case["slope"]}


def run(state):
    if state["op"] == "attn":
        A.attn_fwd(state["q"], state["k"], state["v"], state["out"], state["lse"], state["causal"], state["scale"])
        return state["out"], state["lse"]
    gemm.gemm_lrelu(state["a"], state["b"], state["c"], state["slope"])
    return state["c"]


def work(case):
    if case["op"] == "attn":
        B, H, N, d = case["B"], case["H"], case["N"], case["d"]
        pairs = N * (N + 1) // 2 if case["causal"] else N * N  # (query, visible key)
        return {"bytes": B * H * N * (4 * d * 2 + 4), "flops": 4 * B * H * pairs * d}
    M, N, K = case["M"], case["N"], case["K"]
    return {"bytes": 2 * (M * K + K * N + M * N), "flops": 2 * M * N * K}


def tolerance(case):
    # 2-norm and largest error of the path against the same products in float64 (largest over a dozen
    # shapes, times four): attention rounds the probabilities and the result to 16 bits (2.99e-4 and
    # 2.4e-3 in binary16, 2.3e-3 and 4.2e-2 in bfloat16, where the largest is a dominant probability of a
    # short causal row), the GEMM only the result (2.08e-4 and 4.9e-4; 1.67e-3 and 3.9e-3).
    if case["op"] == "attn":
        return {"rel": 1.2e-3, "max": 1e-2} if case["dtype"] == "f16" else {"rel": 9e-3, "max": 0.17}
    return {"rel": 8e-4, "max": 2e-3} if case["dtype"] == "f16" else {"rel": 6.7e-3, "max": 1.6e-2}
