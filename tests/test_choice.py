"""What attn_fwd launches where nothing is deployed: the choice on both sides of every line (host), and, on the
GPU, that attn_fwd runs what attn_choose_variant names, against the fp64 oracle, in every regime of the key split's
grids and orders (one layer, a second one, the padded grid, by weight mirrored and not; heads that divide over the XCDs
and not), each case with the variant and the grid that it stands for."""
import numpy as np
import pytest

import paper_2403_16863_amd as A
from paper_2403_16863_amd import inputs as I

SPLIT4, SPLIT8, ROWS128, D128, D64_LONG, D64_SHORT = 37, 38, 1, 36, 18, 3


@pytest.mark.parametrize("heads,N,d,causal,want", [
    # key split: up to so many tiles of 32 rows
    (512, 32, 128, False, SPLIT4), (513, 32, 128, False, ROWS128),
    (736, 32, 128, True, SPLIT4), (737, 32, 128, True, D128), (44, 768, 128, True, SPLIT4), (45, 768, 128, True, ROWS128),
    (36, 1024, 128, True, SPLIT4), (37, 1024, 128, True, ROWS128),
    (704, 32, 64, False, SPLIT4), (705, 32, 64, False, D64_LONG), (38, 640, 64, False, SPLIT4), (39, 640, 64, False, D64_SHORT),
    (960, 32, 64, True, SPLIT4), (961, 32, 64, True, D64_LONG),
    (64, 640, 64, True, SPLIT4), (65, 640, 64, True, D64_SHORT), (60, 768, 64, True, SPLIT4), (61, 768, 64, True, D64_SHORT),
    (40, 1200, 64, True, SPLIT4), (41, 1200, 64, True, D64_SHORT),
    # eight waves while every workgroup has a unit to itself
    (16, 512, 64, False, SPLIT8), (17, 512, 64, False, SPLIT4), (16, 511, 128, True, SPLIT4), (16, 512, 128, True, SPLIT8),
    (2, 6144, 128, True, SPLIT8), (2, 6145, 128, True, SPLIT4), (2, 5999, 64, True, SPLIT4), (1, 12288, 64, False, SPLIT4),
    (1, 16384, 64, True, SPLIT8), (1, 16385, 128, True, SPLIT4), (1, 11999, 64, True, SPLIT8),
    # d = 128: 128-row tiles
    (256, 128, 128, False, ROWS128), (257, 128, 128, False, D128), (512, 128, 128, False, D128), (513, 128, 128, False, ROWS128),
    (640, 128, 128, False, ROWS128), (641, 128, 128, False, D128), (576, 128, 128, True, ROWS128), (577, 128, 128, True, D128),
    # d = 64: three workgroups per unit
    (512, 128, 64, False, D64_SHORT), (513, 128, 64, False, D64_LONG), (755, 128, 64, True, D64_SHORT), (756, 128, 64, True, D64_LONG),
    # the shapes of the benchmark and of the paper's attention kernel
    (64, 4096, 128, True, D128), (32, 16384, 128, True, D128), (128, 2048, 64, False, D64_LONG), (4, 16384, 64, False, D64_SHORT),
])
def test_both_sides_of_every_line(heads, N, d, causal, want):
    for dtype in (A.ATTN_F16, A.ATTN_BF16):
        assert A.attn_choose_variant(1, heads, N, d, dtype, causal) == want
        assert A.attn_choose_variant(heads, 1, N, d, dtype, causal) == want
        assert A.attn_variant_supported(want, d, dtype, causal)


def test_bad_problems_have_no_choice():
    for args, code in (((0, 1, 16, 64, 0, False), -1), ((1, 1, 0, 64, 0, False), -1), ((1, 1, 16, 64, 2, False), -1), ((1, 1, 16, 96, 0, False), -2)):
        with pytest.raises(A.AttnError) as e:
            A.attn_choose_variant(*args)
        assert e.value.code == code


CASES = [
    # key split, four waves: a second layer, heads that divide over the XCDs and not
    (1, 16, 640, 64, False, I.F16, 37, 320), (1, 9, 930, 64, False, I.BF16, 37, 270), (1, 20, 860, 128, True, I.F16, 37, 776),
    # the padded grid, per XCD and dealt over all
    (1, 24, 1024, 64, False, I.BF16, 37, 776), (1, 32, 680, 64, False, I.F16, 37, 776), (1, 5, 3290, 64, True, I.F16, 37, 776),
    # by weight in mirrored layers, over groups of XCDs, over all and per XCD; more than four layers
    (1, 10, 2600, 64, True, I.BF16, 37, 820), (1, 7, 3700, 64, True, I.F16, 37, 812), (1, 64, 512, 64, True, I.BF16, 37, 1024), (1, 32, 1150, 128, True, I.F16, 37, 1152),
    # eight waves: one to a unit, a second one, by weight where there is only one
    (1, 7, 1100, 128, True, I.F16, 38, 245), (1, 3, 3663, 64, True, I.BF16, 38, 345), (1, 5, 2002, 128, True, I.BF16, 38, 315),
    # wave groups
    (1, 8, 1200, 64, False, I.F16, 40, 152), (1, 3, 5000, 128, False, I.BF16, 40, 237), (1, 5, 5000, 128, True, I.F16, 40, 395),
    (2, 8, 2000, 128, True, I.BF16, 40, 512),
    # 256-row tiles, 128-row tiles; a partial second layer of short heads, whole ones, three workgroups per unit
    (1, 33, 1000, 128, False, I.F16, 36, 132), (1, 96, 250, 128, False, I.F16, 1, 192), (1, 100, 384, 64, True, I.BF16, 3, 300),
    (4, 16, 1024, 64, True, I.F16, 18, 512), (8, 12, 700, 64, False, I.BF16, 18, 576),
]


def test_the_cases_are_what_they_stand_for():
    for B, H, N, d, causal, dtype, want, grid in CASES:
        assert A.attn_choose_variant(B, H, N, d, dtype, causal) == want, (B, H, N, d, causal)
        assert A.attn_schedule_grid(want, 256, B, H, N) == grid, (B, H, N, d, causal)


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,N,d,causal,dtype,want,grid", CASES)
def test_attn_fwd_runs_the_choice(B, H, N, d, causal, dtype, want, grid):
    from gpu_util import check, run_gpu
    from oracle import ref
    w = I.Workload("choice", B, H, N, d, causal, dtype)
    qb, kb, vb = I.make_qkv(w, seed=N)
    var = A.attn_choose_variant(B, H, N, d, dtype, causal)
    assert (var, A.attn_schedule_grid(var, 256, B, H, N)) == (want, grid)
    print(f"case {w.label} variant {var}", flush=True)
    O, l = run_gpu(qb, kb, vb, causal, w.scale, dtype)
    O2, l2 = run_gpu(qb, kb, vb, causal, w.scale, dtype, variant=var)
    assert np.array_equal(O, O2) and np.array_equal(l, l2) and np.isfinite(O).all() and np.isfinite(l).all()
    # a row of every 32-row tile of every head (tiles are what the schedule deals out), both ends of a few
    tiles = -(-N // 32)
    rows = {bh * N + min(N - 1, 32 * t + (7 * t + 3 * bh) % 32) for bh in range(B * H) for t in range(tiles)}
    rows |= {bh * N + i for bh in (0, B * H - 1) for i in (0, 31, 32, N - 1)}
    rows = np.array(sorted(rows), dtype=np.int64)
    O_ref, l_ref, _ = ref.attn_ref(qb, kb, vb, causal, w.scale, dtype, rows=rows)
    check(O.reshape(-1, d)[rows], l.reshape(-1)[rows], O_ref, l_ref, dtype, what=w.label)
