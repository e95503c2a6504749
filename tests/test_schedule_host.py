"""Host-side tests of the work-item schedule (no GPU): the function the kernels call to pick
their items is exported through the C ABI and checked here as plain host logic."""
import itertools

import pytest

import paper_2403_16863_amd as A


def items_of(grid, BH, nqt):
    """{workgroup: [(bh, qt), ...]} by walking rounds until a workgroup runs dry."""
    out = {}
    for g in range(grid):
        seq = []
        for rnd in itertools.count():
            it = A.attn_schedule_item(grid, g, BH, nqt, rnd)
            if it is None:
                # once dry, always dry
                assert A.attn_schedule_item(grid, g, BH, nqt, rnd + 1) is None
                break
            seq.append(it)
        out[g] = seq
    return out


@pytest.mark.parametrize("grid,BH,nqt", [
    (256, 64, 16), (256, 32, 64), (512, 128, 16), (256, 64, 4), (8, 8, 1), (16, 8, 5),
    (7, 3, 5), (1, 1, 1), (1, 5, 7), (30, 6, 5), (256, 2, 1), (24, 40, 3), (256, 24, 11), (255, 64, 16),
])
def test_every_item_exactly_once(grid, BH, nqt):
    sched = items_of(grid, BH, nqt)
    seen = [it for seq in sched.values() for it in seq]
    assert len(seen) == BH * nqt
    assert set(seen) == {(b, q) for b in range(BH) for q in range(nqt)}


@pytest.mark.parametrize("grid,BH,nqt", [(256, 64, 16), (256, 32, 64), (512, 128, 16), (64, 16, 8)])
def test_heads_stay_on_their_xcd(grid, BH, nqt):
    # grid and BH multiples of 8: workgroup g runs on XCD g % 8 and only touches heads = g mod 8
    for g, seq in items_of(grid, BH, nqt).items():
        assert all(bh % 8 == g % 8 for bh, _ in seq)


@pytest.mark.parametrize("grid,BH,nqt", [(256, 64, 16), (256, 32, 64), (512, 128, 16), (256, 64, 8)])
def test_balanced_and_local(grid, BH, nqt):
    # causal weight of query tile qt is proportional to qt + 1
    sched = items_of(grid, BH, nqt)
    loads = [sum(qt + 1 for _, qt in seq) for seq in sched.values()]
    assert max(loads) - min(loads) <= 1 + nqt // 8   # serpentine deal: near-equal sums
    # in every round the workgroups of one XCD work on few heads (their K/V share that L2)
    per_xcd = grid // 8
    rounds = max(len(seq) for seq in sched.values())
    for x in range(8):
        for rnd in range(rounds):
            heads = {sched[g][rnd][0] for g in range(x, grid, 8) if rnd < len(sched[g])}
            assert len(heads) <= -(-per_xcd // nqt) + 1


@pytest.mark.parametrize("grid,BH,nqt", [
    (512, 64, 8), (512, 32, 16), (400, 50, 8), (768, 64, 32), (320, 8, 40), (552, 24, 23),   # layers of 256, whole and partial
    (256, 32, 12), (256, 64, 12), (512, 12, 50), (768, 128, 18), (256, 3, 100), (768, 48, 20),  # rounds that are no whole pairs
])
def test_causal_sums_per_compute_unit(grid, BH, nqt):
    """Workgroups g, g + 256 and g + 512 share a compute unit: every item once, and no unit has more than about
    one item above the mean (whole deals) or above a unit's fair share (a single, partial one)."""
    sched = items_of(grid, BH, nqt)
    seen = [it for seq in sched.values() for it in seq]
    assert len(seen) == len(set(seen)) == BH * nqt
    units = [0] * 256
    for g, seq in sched.items():
        units[g % 256] += sum(qt + 1 for _, qt in seq)
    assert max(units) <= sum(units) / min(256, grid) + nqt


def test_rounds_by_weight_go_from_heavy_to_light():
    """384 items on 256 workgroups: the second, partial round holds the lightest third."""
    sched = items_of(256, 32, 12)
    assert min(seq[0][1] for seq in sched.values()) >= max(seq[1][1] for seq in sched.values() if len(seq) > 1)


@pytest.mark.parametrize("causal", [False, True], ids=["full", "causal"])
@pytest.mark.parametrize("grid,BH,nqt", [
    (300, 5, 60), (304, 8, 38), (512, 16, 32), (776, 9, 57), (776, 8, 96), (776, 3, 171), (769, 1, 769), (776, 8, 97), (1008, 16, 63),  # layers, and more
    (256, 32, 12), (256, 64, 16), (512, 64, 16), (512, 12, 50), (768, 128, 18), (768, 48, 20), (256, 3, 100), (255, 64, 16), (8, 8, 1),
])
def test_either_mask_names_every_item_once(grid, BH, nqt, causal):
    """The persistent deal, over grids with a second layer, with more workgroups than items, of more than three layers,
    and of several rounds.  Without a mask the items of a head follow each other."""
    import ctypes
    L = A.binding.lib()
    bh, qt, seen, rounds = ctypes.c_int(0), ctypes.c_int(0), [], 0
    while True:
        this = []
        for g in range(grid):
            rc = L.attn_schedule_item_of(grid, g, BH, nqt, rounds, int(causal), ctypes.byref(bh), ctypes.byref(qt))
            assert rc in (0, 1)
            if rc:
                this.append((bh.value, qt.value))
                if causal:
                    assert A.attn_schedule_item(grid, g, BH, nqt, rounds) == this[-1]
        if not this:
            break
        if not causal:                                  # the items of a round are those of as few heads as hold them
            by_xcd = grid % 8 == 0 and BH % 8 == 0
            heads = {b for b, _ in this}
            assert len(heads) <= (8 if by_xcd else 1) * (-(-len(this) // (nqt * (8 if by_xcd else 1))) + 1)
        seen += this
        rounds += 1
    assert len(seen) == BH * nqt and set(seen) == {(b, q) for b in range(BH) for q in range(nqt)}
    assert rounds == -(-BH * nqt // grid)


def test_the_split_pads_its_grid_between_two_and_three_layers():
    v = 37
    for n, want in ((512, 512), (513, 776), (768, 776), (769, 769), (300, 300)):
        assert A.attn_schedule_grid(v, 256, 1, 1, 32 * n) == want


def test_grids_beyond_the_thread_count_of_a_launch_are_refused():
    """One workgroup per item: 2^32 threads are reached with 2^23 items of eight waves, 2^24 of four.  (Fake
    pointers: the check comes before the launch.)"""
    from paper_2403_16863_amd import binding
    L = binding.lib()
    split = [v for v in range(A.attn_num_variants()) if "pipe=0" in A.attn_variant_desc(v) and "ldpos=1" in A.attn_variant_desc(v)]
    assert len(split) == 2
    for v in split:
        most = (2 ** 32 - 1) // (64 * int(A.attn_variant_desc(v).split("nw=")[1].split()[0]))
        assert A.attn_schedule_grid(v, 256, 1, most, 1) == most
        with pytest.raises(A.AttnError) as e:
            A.attn_schedule_grid(v, 256, 1, most + 1, 1)
        assert e.value.code == A.binding.ATTN_EUNSUPPORTED
        q, k, v_, o, lse = (n << 40 for n in range(1, 6))
        assert L.attn_fwd_variant(q, k, v_, o, lse, 1, most + 1, 1, 64, 0, 1.0, 0, None, v) == A.binding.ATTN_EUNSUPPORTED


def test_grid_size():
    v = A.attn_default_variant(4096, 128, A.ATTN_BF16, True)
    assert A.attn_schedule_grid(v, 256, 2, 32, 4096) == 256           # one persistent workgroup per CU
    assert A.attn_schedule_grid(v, 256, 1, 2, 128) == 2               # never more than items
    assert A.attn_schedule_grid(v, 256, 1, 8, 256) == 8
    v64 = A.attn_default_variant(1024, 64, A.ATTN_F16, True)
    g = A.attn_schedule_grid(v64, 256, 4, 16, 1024)
    assert 0 < g <= 512 and g % 8 == 0
    with pytest.raises(A.AttnError):
        A.attn_schedule_grid(v, 0, 1, 1, 1)
    with pytest.raises(A.AttnError):
        A.attn_schedule_item(4, 4, 1, 1, 0)


@pytest.mark.parametrize("grid,BH,nqt", [(192, 6, 32), (7, 7, 1), (9, 3, 3), (776, 36, 20), (1030, 10, 103), (12, 2, 6), (1002, 6, 167), (1204, 4, 301)])
def test_short_launches_keep_a_head_on_few_xcds(grid, BH, nqt):
    """One workgroup per item: without a mask every XCD has a run of the items in head-major order, with one the key
    split's deal (bit 1) gives groups of XCDs heads of their own; every item once either way."""
    import ctypes
    L = A.binding.lib()
    bh, qt = ctypes.c_int(0), ctypes.c_int(0)
    for causal in (2, 3):
        items, ran = {}, []
        for g in range(grid):
            if L.attn_schedule_item_of(grid, g, BH, nqt, 0, causal, ctypes.byref(bh), ctypes.byref(qt)):
                items.setdefault(g % 8, []).append((bh.value, qt.value))
                ran.append((bh.value, qt.value))
            assert L.attn_schedule_item_of(grid, g, BH, nqt, 1, causal, ctypes.byref(bh), ctypes.byref(qt)) == 0
        assert sorted(ran) == [(b, q) for b in range(BH) for q in range(nqt)]
        groups = next(n for n in (8, 4, 2, 1) if grid % n == 0 and BH % n == 0)
        for x, seq in items.items():
            if causal == 3:
                assert all(b % groups == x % groups for b, _ in seq)
            else:
                place = [b * nqt + nqt - 1 - q for b, q in seq]
                assert groups == 8 or place == list(range(place[0], place[0] + len(seq)))


@pytest.mark.parametrize("BH,nqt", [(200, 2), (96, 3), (128, 3), (72, 5), (56, 7), (61, 6), (50, 8), (35, 8)])
def test_a_partial_second_layer_of_short_heads_holds_the_lightest(BH, nqt):
    """One round, workgroups 256 and up share the units of the first 256: no item of theirs weighs more than one of those."""
    sched = items_of(BH * nqt, BH, nqt)
    assert len({it for seq in sched.values() for it in seq}) == BH * nqt
    for x in range(8):
        first = [sched[g][0][1] for g in range(x, 256, 8)]
        second = [sched[g][0][1] for g in range(256 + x, BH * nqt, 8)]
        assert min(first) >= max(second, default=0)


def deal(grid, BH, nqt, causal, resident, mirrored=0):
    """{workgroup: item} of workgroups with one item each, `resident` of them to a unit."""
    import ctypes
    L, kind = A.binding.lib(), causal + 2 * resident + 16 * mirrored
    bh, qt, out = ctypes.c_int(0), ctypes.c_int(0), {}
    for g in range(grid):
        if L.attn_schedule_item_of(grid, g, BH, nqt, 0, kind, ctypes.byref(bh), ctypes.byref(qt)):
            out[g] = (bh.value, qt.value)
        assert L.attn_schedule_item_of(grid, g, BH, nqt, 1, kind, ctypes.byref(bh), ctypes.byref(qt)) == 0
    return out


@pytest.mark.parametrize("causal", [0, 1], ids=["full", "causal"])
@pytest.mark.parametrize("BH,nqt", [(6, 32), (5, 63), (10, 83), (18, 40), (8, 97), (36, 20)])
def test_what_each_variant_deals(BH, nqt, causal):
    """The order that a variant launches: the key split and the wave groups with what a unit holds of their workgroups, the
    persistent ones as attn_schedule_item names it (under a mask)."""
    from test_gpu_key_split import launched_item
    for v in range(A.attn_num_variants()):
        knobs = dict(kv.split("=") for kv in A.attn_variant_desc(v).split())
        splits = knobs["pipe"] == "0" and knobs["ldpos"] != "0"
        if not splits and v % 9:
            continue
        grid = A.attn_schedule_grid(v, 256, 1, BH, nqt * int(knobs["bm"]))
        for d in (64, 128):
            got = {g: launched_item(v, d, causal, grid, g, BH, nqt, 0) for g in range(grid)}
            if splits:
                resident = 1 if knobs["nw"] == "8" and d == 128 else 2
                mirrored = 4 if knobs["ldpos"] == "1" and knobs["nw"] == "4" else 0
                assert {g: it for g, it in got.items() if it} == deal(grid, BH, nqt, causal, resident, mirrored)
            elif causal:
                assert got == {g: A.attn_schedule_item(grid, g, BH, nqt, 0) for g in range(grid)}


@pytest.mark.parametrize("grid,BH,nqt,resident", [
    (315, 5, 63, 1), (257, 1, 257, 1), (288, 18, 16, 1), (320, 10, 32, 1), (264, 8, 33, 1), (776, 36, 20, 1), (776, 36, 20, 2), (1030, 10, 103, 2), (513, 1, 513, 2),
])
def test_what_does_not_start_at_once_is_the_lightest(grid, BH, nqt, resident):
    """Causal, more items than the units hold: in the order in which an XCD's workgroups start the weight never rises."""
    items = deal(grid, BH, nqt, 1, resident)
    assert len(set(items.values())) == BH * nqt
    for x in range(8):
        weights = [items[g][1] for g in range(x, grid, 8) if g in items]
        assert weights == sorted(weights, reverse=True)


@pytest.mark.parametrize("grid,BH,nqt,resident", [(256, 4, 64, 1), (512, 4, 128, 2), (512, 16, 32, 2), (300, 5, 60, 2)])
def test_what_starts_at_once_is_dealt_in_layers(grid, BH, nqt, resident):
    """A unit's two workgroups hold items of one weight sum, the heads of a round stay together."""
    items = deal(grid, BH, nqt, 1, resident)
    heads = next(n for n in (8, 4, 2, 1) if grid % n == 0 and BH % n == 0)
    for layer in range(0, grid, 256):
        for x in range(heads):
            group = [items[g] for g in range(layer + x, min(grid, layer + 256), heads)]
            assert len({b for b, _ in group}) <= -(-len(group) // nqt) + 1


@pytest.mark.parametrize("grid,BH,nqt", [(830, 10, 83), (1008, 18, 56), (864, 9, 96), (1024, 16, 64), (776, 12, 63)])
def test_four_waves_on_a_unit_have_even_sums(grid, BH, nqt):
    """Key split on four waves, d = 64, 513 to 1024 items: all start at once, four to a unit (g, g + 256, ...); no unit has
    more than a fifth of the heaviest item above the mean (dealt forward only: half of it)."""
    items = deal(grid, BH, nqt, 1, 2, 4)
    assert len(set(items.values())) == BH * nqt
    units = [[items[g][1] + 1 for g in range(u, grid, 256) if g in items] for u in range(256)]
    assert max(map(sum, units)) <= sum(map(sum, units)) / 256 + nqt / 5


@pytest.mark.parametrize("resident,mirrored", [(1, 0), (2, 0), (2, 4)])
@pytest.mark.parametrize("causal", [0, 1], ids=["full", "causal"])
def test_one_item_per_workgroup_names_every_item_once(causal, resident, mirrored):
    """Over heads that divide by 8, 4, 2 and nothing and any number of tiles, with the padding to 776 workgroups."""
    for BH in (*range(1, 18), 20, 24, 33, 36, 64):
        for nqt in (1, 2, 3, 4, 5, 7, 8, 9, 16, 17, 31, 40):
            total = BH * nqt
            grid = 776 if 512 < total <= 768 else total
            assert sorted(deal(grid, BH, nqt, causal, resident, mirrored).values()) == [(b, q) for b in range(BH) for q in range(nqt)]
