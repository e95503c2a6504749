"""d = 128, many query tiles in few rounds: which launches take 128-row tiles in place of 256-row ones (host), and on the GPU
those against the fp64 oracle, with a last tile of a head that is nearly empty or nearly full, one round and several."""
import numpy as np
import pytest

import paper_2403_16863_amd as A
from paper_2403_16863_amd import inputs as I

ROWS128, D128 = 1, 36


@pytest.mark.parametrize("heads,N,causal,want", [
    (96, 512, False, D128), (96, 513, False, ROWS128), (96, 1024, False, ROWS128), (96, 1025, False, D128),
    (128, 768, False, ROWS128), (128, 769, False, D128), (128, 1024, False, D128), (128, 1025, False, ROWS128), (128, 1152, False, ROWS128),
    (128, 1153, False, D128), (64, 1024, False, D128), (64, 1025, False, ROWS128), (24, 3790, False, D128), (257, 128, False, D128), (33, 1000, False, D128),
    (128, 896, True, ROWS128), (128, 897, True, D128), (128, 1024, True, D128), (128, 1025, True, ROWS128), (96, 1152, True, ROWS128),
    (96, 1153, True, D128), (32, 2560, True, ROWS128), (32, 2561, True, D128), (64, 4096, True, D128), (32, 16384, True, D128),
    (300, 256, True, D128), (1 << 20, 2048, True, D128),
    # heads that XCDs share, under a mask: only far ahead, or with few keys
    (43, 2059, True, D128), (43, 2362, True, D128), (55, 1597, True, D128), (90, 1811, True, D128), (75, 1541, True, D128), (87, 1004, True, D128),
    (86, 806, True, ROWS128), (17, 4256, True, ROWS128), (127, 537, True, ROWS128), (119, 639, True, ROWS128), (119, 640, True, D128), (64, 1373, True, ROWS128),
])
def test_the_choice(heads, N, causal, want):
    for dtype in (A.ATTN_F16, A.ATTN_BF16):
        assert A.attn_choose_variant(1, heads, N, 128, dtype, causal) == want


CASES = [(2, 48, 599, False, I.BF16), (8, 16, 257, False, I.F16), (4, 32, 642, False, I.F16), (4, 32, 561, True, I.BF16), (2, 48, 846, True, I.F16), (1, 32, 2500, True, I.BF16)]


@pytest.mark.gpu
@pytest.mark.parametrize("B,H,N,causal,dtype", CASES)
def test_against_the_oracle(B, H, N, causal, dtype):
    from gpu_util import check, run_gpu
    from oracle import ref
    w = I.Workload("rows128", B, H, N, 128, causal, dtype)
    assert A.attn_choose_variant(B, H, N, 128, dtype, causal) == ROWS128
    print(f"case {w.label}", flush=True)
    qb, kb, vb = I.make_qkv(w, seed=N)
    O, l = run_gpu(qb, kb, vb, causal, w.scale, dtype)
    assert np.isfinite(O).all() and np.isfinite(l).all()
    # a row of every 64-row stretch of every head, both ends of the first and the last
    rows = {bh * N + min(N - 1, 64 * t + (7 * t + 3 * bh) % 64) for bh in range(B * H) for t in range(-(-N // 64))}
    rows |= {bh * N + i for bh in (0, B * H - 1) for i in (0, 31, 32, 127, 128, N - 1)}
    rows = np.array(sorted(rows), dtype=np.int64)
    O_ref, l_ref, _ = ref.attn_ref(qb, kb, vb, causal, w.scale, dtype, rows=rows)
    check(O.reshape(-1, 128)[rows], l.reshape(-1)[rows], O_ref, l_ref, dtype, what=w.label)
