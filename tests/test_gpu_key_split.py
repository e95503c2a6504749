"""The key split of the free-running order, which attn_fwd takes for launches of few query tiles: the choice,
and the two variants against the fp64 oracle where they can go wrong: fewer key tiles than waves, one key or
row past a 32-row tile, waves that see their first tile late or never, scores that climb from wave to wave."""
import numpy as np
import pytest

import paper_2403_16863_amd as A
from oracle import ref
from paper_2403_16863_amd import inputs as I

SPLIT = [v for v in range(A.attn_num_variants()) if "pipe=0" in A.attn_variant_desc(v) and "ldpos=1" in A.attn_variant_desc(v)]
DESC = {v: dict(kv.split("=") for kv in A.attn_variant_desc(v).split()) for v in SPLIT}


def test_few_query_tiles_take_the_split_and_many_do_not():
    assert len(SPLIT) == 2 and all(DESC[v]["bm"] == "32" for v in SPLIT)
    for d in (64, 128):
        for causal in (False, True):
            assert A.attn_default_variant(300, d, A.ATTN_F16, causal) in SPLIT
            for N in (1024, 4096, 1 << 20):          # named for many heads
                assert A.attn_default_variant(N, d, A.ATTN_F16, causal) not in SPLIT


def test_every_row_block_has_a_workgroup():
    for B, H, N in ((1, 3, 1000), (2, 4, 129), (1, 1, 1), (1, 16, 64)):
        for v in SPLIT:
            nqt = -(-N // 32)
            grid = A.attn_schedule_grid(v, 256, B, H, N)
            assert grid == B * H * nqt
            for d in (64, 128):
                for causal in (False, True):
                    items = [launched_item(v, d, causal, grid, g, B * H, nqt, 0) for g in range(grid)]
                    assert sorted(items) == [(b, q) for b in range(B * H) for q in range(nqt)]
                    assert all(launched_item(v, d, causal, grid, g, B * H, nqt, 1) is None for g in range(grid))


def launched_item(variant, d, causal, grid, workgroup, BH, nqt, rnd):
    import ctypes
    bh, qt = ctypes.c_int(0), ctypes.c_int(0)
    rc = A.binding.lib().attn_schedule_item_launched(variant, d, int(causal), grid, workgroup, BH, nqt, rnd, ctypes.byref(bh), ctypes.byref(qt))
    assert rc in (0, 1)
    return (bh.value, qt.value) if rc else None


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_split_against_the_oracle(d, dtype, causal):
    from gpu_util import check, run_gpu
    for N in (1, 31, 32, 33, 127, 129, 257, 289, 600):
        for kind in ("normal", "rising_scores", "peaked"):
            if kind == "normal":
                qb, kb, vb = I.make_qkv(I.Workload("split", 1, 3, N, d, causal, dtype, qk_sigma=2.0), seed=N)
            else:
                qb, kb, vb = I.make_adversarial(kind, 1, 3, N, d, dtype, seed=N)
            for scale in (float(np.float32(d ** -0.5)), -0.1, 0.0):
                O_ref, l_ref, _ = ref.attn_ref(qb, kb, vb, causal, float(np.float32(scale)), dtype)
                out_scale = max(1.0, float(np.abs(I.bits_to_f64(vb, dtype)).max()))
                for v in SPLIT:
                    print(f"case {kind} N={N} d={d} causal={causal} dtype={dtype} scale={scale} variant={v}", flush=True)
                    O, l = run_gpu(qb, kb, vb, causal, scale, dtype, variant=v)
                    check(O, l, O_ref, l_ref, dtype, out_scale=out_scale, what=f"{kind} N={N} scale={scale} variant {v}")


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("dtype", [I.F16, I.BF16], ids=["f16", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
def test_keys_masked_by_their_scores(d, dtype, causal):
    """Scores of -inf (or of the lowest finite number, with a scale that takes it past the range of fp32, or so low
    that its scaled value is rounded by more than that range) in all keys a wave meets first, or in all it ever
    meets: no weight, whatever the wave."""
    from gpu_util import check, run_gpu
    lowest = float(np.float32(-65504.0)) if dtype == I.F16 else float(np.array(0xFF7F0000, np.uint32).view(np.float32))
    for v in SPLIT:
        nw = int(DESC[v]["nw"])
        N = 32 * 2 * nw + 5
        tile = np.arange(N) // 32
        masks = [(f"wave {w} never", tile % nw == w) for w in range(nw)] + [(f"wave {w} late", tile == w) for w in range(nw)]
        masks += [("all but tile 0", tile > 0), ("all but the last wave", tile % nw != nw - 1)]
        w = I.Workload("masked", 1, 2, N, d, causal, dtype)
        qb, kb, vb = I.make_qkv(w, seed=5)
        one = I.f32_to_bits(np.ones(1, np.float32), dtype)[0]
        for value, scale in [(-np.inf, w.scale), (lowest, 0.9)] + [(-1e30, w.scale), (-1.5e30, w.scale)] * (dtype == I.BF16):
            # (the last one twice as low in every other group of four keys, which is one half of the wave)
            low = I.f32_to_bits(np.where((np.arange(N) & 4 == 0) & (value == -1.5e30), 2 * value, value).astype(np.float32), dtype)
            for name, m in masks:
                q, k = qb.copy(), kb.copy()
                q[..., 0] = one
                k[:, :, m, 0] = low[m]
                seen = np.cumsum(~m) > 0 if causal else np.ones(N, bool)      # rows that see an unmasked key
                print(f"case {name} value={value} N={N} d={d} causal={causal} dtype={dtype} variant={v}", flush=True)
                O_ref, l_ref, _ = ref.attn_ref(q, k, vb, causal, float(np.float32(scale)), dtype)
                O, l = run_gpu(q, k, vb, causal, scale, dtype, variant=v)
                check(O[:, :, seen], l[:, :, seen], O_ref[:, :, seen], l_ref[:, :, seen], dtype, what=f"{name} {value} variant {v}")
                if value == -np.inf:                              # no weight at all: 0 / 0, as every variant gives it
                    assert np.isnan(O[:, :, ~seen]).all() and not np.isfinite(l[:, :, ~seen]).any(), name


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
def test_memory_behind_the_last_row_is_never_used(d):
    """Rows past the end and tiles past the last one arrive as zeros (the range check of the buffer loads): NaN
    behind the tensors changes nothing, for the variants that load that way (the split, the interleaved order)."""
    import torch
    ids = SPLIT + [v for v in range(A.attn_num_variants()) if "pipe=3" in A.attn_variant_desc(v) and A.attn_variant_supported(v, d, A.ATTN_F16, False)]
    for N in (1, 31, 33, 65, 95, 129, 200, 257):
        g = torch.Generator(device="cuda")
        g.manual_seed(N)
        data = [torch.randn(N * d, device="cuda", generator=g).half() for _ in range(3)]
        for v in ids:
            print(f"case N={N} d={d} variant={v}", flush=True)
            got = []
            for behind in (0.0, float("nan")):
                flat = [torch.full((N * d + (1 << 19),), behind, device="cuda", dtype=torch.float16) for _ in range(3)]
                for f, x in zip(flat, data):
                    f[:N * d] = x
                q, k, v_ = (f[:N * d].view(1, 1, N, d) for f in flat)
                out, lse = torch.empty(1, 1, N, d, device="cuda", dtype=torch.float16), torch.empty(1, 1, N, device="cuda")
                A.attn_fwd_variant(q, k, v_, out, lse, False, d ** -0.5, v)
                torch.cuda.synchronize()
                got.append((out, lse))
            assert torch.isfinite(got[0][0]).all() and torch.isfinite(got[0][1]).all()
            assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16)) and torch.equal(got[0][1], got[1][1]), (N, v)


@pytest.mark.gpu
def test_non_finite_scores_stay_in_their_rows():
    """A NaN or an infinity in one query reaches that row alone, whichever wave's keys meet it (bfloat16; in
    binary16 the overflow mode leaves no rule for what a NaN or an infinity in the inputs becomes)."""
    import torch
    from gpu_util import run_gpu
    for bad in (float("nan"), float("inf")):
        qb, kb, vb = I.make_qkv(I.Workload("split", 1, 2, 200, 64, False, I.BF16), seed=3)
        q = torch.from_numpy(qb.view(np.int16)).view(torch.bfloat16)
        q[0, 1, 77, 5] = bad
        for v in SPLIT:
            O, l = run_gpu(q.view(torch.int16).numpy().view(np.uint16), kb, vb, False, 0.125, I.BF16, variant=v)
            assert np.isnan(O[0, 1, 77]).all() and np.isnan(l[0, 1, 77])
            O[0, 1, 77], l[0, 1, 77] = 0, 0
            assert np.isfinite(O).all() and np.isfinite(l).all()
