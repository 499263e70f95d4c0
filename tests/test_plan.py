"""Host checks of the rules that pick the kernels of a call and size its workspace (csrc/plan.h)."""
import ctypes
import random

import pytest

from paper_2011_09208_amd import buildlib
from tests import plan_rules
from tests.plan_rules import BLOCKS, FORWARD, LISTS, PROBS, SMALL, STEP, TILES, TOP1


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return plan_rules.load(str(tmp_path_factory.mktemp("plan")))


@pytest.fixture(scope="module")
def ws():
    if buildlib.is_stale():
        buildlib.build()
    from paper_2011_09208_amd import binding
    return binding


def drawn(n, seed, max_b=70000, max_d=4096, max_c=150000):
    """Sizes spread over their logarithms, every other batch and width at or beside the edge of a tile."""
    rng = random.Random(seed)
    for _ in range(n):
        B, C = (int(m ** rng.random()) for m in (max_b, max_c))
        D = 64 * int((max_d // 64) ** rng.random())
        if rng.random() < 0.5:
            B = max(1, (B + 32) // 64 * 64 + rng.choice((-1, 0, 1)))
        if rng.random() < 0.5:
            C = max(1, (C + 32) // 64 * 64 + rng.choice((-1, 0, 1)))
        yield B, D, C


def test_the_rules_tested_here_are_the_librarys(rules, ws):
    for B, D, C in drawn(2000, seed=1):
        assert rules.fwd_bytes_(B, D, C) == ws.fwd_workspace_bytes(B, D, C), (B, D, C)
        assert rules.bwd_bytes_(B, D, C) == ws.bwd_workspace_bytes(B, D, C), (B, D, C)


@pytest.mark.parametrize("B,D,C,want", [(300, 2048, 12000, 2 * 128 * 512 * 4), (257, 192, 8441, 2 * 128 * 512 * 4),
                                        (100, 2048, 20000, 2 * 256 * 256 * 4), (85, 192, 30922, 2 * 256 * 256 * 4)])
def test_forward_query_holds_the_lists_where_the_arg_max_takes_blocks(rules, ws, B, D, C, want):
    assert rules.way_(B, D, C, FORWARD) == LISTS and ws.fwd_workspace_bytes(B, D, C) == want


def test_forward_query_is_what_the_calls_compare_with(rules, ws):
    """The forward call and the arg-max take their own kernels with a workspace as large as the query, and the former size, a pair
    per class tile of 256, is never more than that.  Where the former size fits the built-in scratch, so does what the call wants."""
    lists = 0
    for B, D, C in [*drawn(30000, seed=2), (2 ** 31 - 1, 64, 2 ** 31 - 1), (1, 64, 2 ** 31 - 1), (20, 64, 2 ** 31 - 1), (2 ** 31 - 1, 64, 1)]:
        step, top1, least = rules.way_bytes_(B, D, C, FORWARD), rules.way_bytes_(B, D, C, TOP1), rules.least_fwd_bytes_(B, C)
        assert least == 2 * ((C + 255) // 256) * ((B + 255) // 256 * 256) * 4
        assert ws.fwd_workspace_bytes(B, D, C) == max(step, top1, least), (B, D, C)
        if least <= ws.STATIC_SCRATCH_BYTES:
            assert step <= ws.STATIC_SCRATCH_BYTES, (B, D, C)
        lists += rules.way_(B, D, C, FORWARD) == LISTS
    assert lists > 3000


def test_quotients_of_the_list_kernels(rules):
    """By 1 to 1024 ranges, four times as many, and up to three batch tiles: every edge of a quotient below the bound n * d < 2^32."""
    rng = random.Random(3)
    for d in [*range(1, 1025), *range(1028, 4097, 4)]:
        top = (2 ** 32 - 1) // d
        for q in {1, 2, 3, top // d, *(rng.randint(0, top // d) for _ in range(20))}:
            for n in (q * d - 1, q * d, q * d + d - 1):
                if 0 <= n <= top:
                    assert rules.quotient_(n, d) == n // d, (n, d)


@pytest.mark.parametrize("B,D,C,ranges", [(50000, 128, 600, 1), (65536, 512, 1000, 1), (20000, 128, 2000, 3), (600, 640, 43553, 85)])
def test_whole_tiles_of_a_list_are_a_range_apart(rules, B, D, C, ranges):
    assert rules.way_(B, D, C, STEP) == LISTS and rules.ranges_(D, C, (B + 255) // 256) == ranges
    for ct in range((C + 255) // 256):
        assert rules.list_quotient_(ct, D, C, (B + 255) // 256) == ct // ranges


def test_every_kind_of_tile_walks_the_features_in_one_direction(rules):
    """A shard's calls may run a logit in 64 x 64 tiles (always ascending), in a list (which alternates its whole tiles) or in a
    wide tile, which asks the rule: the rule must say what the others do.  Small batches have an order of their own."""
    seen = set()
    for B, D, C in [*drawn(20000, seed=4), (64, 192, 140000), (17, 128, 150000)]:
        ways = {use: rules.way_(B, D, C, use) for use in (STEP, PROBS, TOP1)}
        nBT, nCT = (B + 255) // 256, (C + 255) // 256
        tiles = [(ct, bt) for ct in {0, 1, 2, 31, 32, 33, nCT // 2, nCT - 1} for bt in {0, 3, 4, nBT - 1} if 0 <= ct < nCT and bt < nBT]
        got = {t: rules.descending_(B, D, C, *t) for t in tiles}
        if BLOCKS in ways.values():
            assert not any(got.values()), (B, D, C, ways)
        elif ways[STEP] == LISTS:
            ranges = rules.ranges_(D, C, nBT)
            full = 2 * ((C + 63) // 64) // (8 * ranges)
            assert got == {(ct, bt): int(ct < full * ranges and ct // ranges % 2 == 1) for ct, bt in tiles}, (B, D, C)
        elif ways[STEP] == TILES and nBT * nCT > 256:
            assert got == {(ct, bt): (ct * nBT // 32 if nBT <= 4 else ct // 8 ^ bt // 4) % 2 for ct, bt in tiles}, (B, D, C)
        else:
            assert not any(got.values()), (B, D, C, ways)
        seen.add(tuple(ways.values()))
    assert {(BLOCKS, BLOCKS, TILES), (LISTS, TILES, TILES), (LISTS, BLOCKS, BLOCKS), (TILES, TILES, TILES), (SMALL, SMALL, SMALL)} <= seen


def test_splits_of_dx_are_the_cheapest(rules):
    """The search skips numbers of splits; trying each of them finds nothing better, and nothing as good that comes earlier."""
    out = (ctypes.c_int * 4)()
    for B, D, C in [*drawn(1500, seed=5, max_b=20000), *((1, 64, 64 * t) for t in range(1, 400)), (32, 64, 30000), (64, 64, 100000), (1, 64, 1), (1, 64, 2 ** 31 - 1),
                    (64, 2048, 65536), (64, 2048, 65537)]:
        rules.dx_splits_(B, D, C, out)
        total, best = (C + 63) // 64, None
        turns_of_the_sum = -(-B * (D // 4) // (128 * 512))
        for small in (0,) if 2 * C * D > 2 ** 28 and 32 * (-D % 256) <= D + -D % 256 else (0, 1):
            tiles = D // 64 * -(-B // 64) if small else -(-D // 256) * -(-B // 256)
            room = 512 if small else 256
            for want in range(1, min(max(1, -(-room // tiles)), total) + 1):
                steps = -(-total // want)
                splits, turns = -(-total // steps), -(-tiles * -(-total // steps) // 256)
                cost = turns * 320 * steps + 1500 if small else turns * (1300 * steps + 6000)
                cost += splits * (8 * B * D // 4500 + turns_of_the_sum * 1000 // 16) - (4000 if small and splits == 1 and out[3] else 0)
                if best is None or cost < best[0]:
                    best = (cost, small, splits, steps)
        assert (out[0], out[1], out[2]) == best[1:], (B, D, C)
        assert (out[1] - 1) * out[2] < total <= out[1] * out[2]


def test_dx_of_a_large_w_and_padded_features_runs_in_small_tiles(rules):
    """W beyond the Infinity Cache: wide tiles, unless more than 1 / 32 of them is padding of the features."""
    out = (ctypes.c_int * 4)()
    for B in (24, 64):
        for D, small in [(1024, 0), (1088, 1), (1280, 0), (1600, 1), (1728, 1), (1920, 1), (1984, 0), (2048, 0), (3008, 0)]:
            for megabytes in (275, 430):
                rules.dx_splits_(B, D, megabytes * 500000 // D, out)
                assert out[0] == small, (B, D, megabytes)


def test_short_lists_have_a_compute_unit_of_their_own(rules):
    """More than 256 tiles: several lists on a compute unit are of 12 units of 32 classes (a tile and a half) or more."""
    for B, D, C in [(1408, 64, 13471), (1408, 256, 24271), (3261, 64, 8679), (5409, 128, 2909), (14734, 192, 3268), (38406, 64, 1611)]:
        assert rules.way_(B, D, C, STEP) == TILES
    for B, D, C in drawn(10000, seed=6):
        nBT, nCT = (B + 255) // 256, (C + 255) // 256
        ranges = rules.ranges_(D, C, nBT)
        if rules.way_(B, D, C, STEP) == LISTS and nBT * nCT > 256 < ranges * nBT:
            assert 2 * ((C + 63) // 64) >= 12 * ranges, (B, D, C)


def test_the_forward_call_of_a_short_contraction_runs_a_single_round_on_tiles(rules):
    for B, D, C, way in [(94, 64, 29001, TILES), (94, 128, 25601, TILES), (94, 128, 25600, LISTS), (94, 192, 29001, LISTS), (2303, 64, 8376, TILES),
                         (4363, 64, 6004, LISTS), (1280, 128, 16384, TILES), (1281, 128, 14000, LISTS)]:
        assert rules.way_(B, D, C, STEP) == LISTS and rules.way_(B, D, C, FORWARD) == way, (B, D, C)
    for B, D, C in drawn(10000, seed=7):
        step, forward = rules.way_(B, D, C, STEP), rules.way_(B, D, C, FORWARD)
        assert forward == step or (step, forward) == (LISTS, TILES)


def test_shapes_of_the_list_tests_run_lists(rules):
    """Which of the shapes of test_gpu_list.py (a whole shard) run lists, both ways or dz alone: their tests must not lose them unnoticed."""
    from tests.test_gpu_list import SHAPES
    tiles = {(700, 576, 22081), (1000, 576, 35072), (33000, 64, 500)}
    dz_alone = {(70, 64, 16600), (257, 64, 8441), (1700, 64, 2600), (300, 128, 33024), (1100, 128, 5377)}
    for shape in SHAPES:
        step, forward = rules.way_(*shape, STEP), rules.way_(*shape, FORWARD)
        assert step == (TILES if shape in tiles else LISTS), shape
        assert forward == (TILES if shape in tiles | dz_alone else LISTS), shape
    assert rules.way_(257, 192, 8441, FORWARD) == LISTS


@pytest.mark.parametrize("B,D,tiles,way", [(64, 192, 768, BLOCKS), (64, 192, 769, TILES), (33, 64, 1024, TILES), (64, 192, 1025, BLOCKS), (64, 256, 1024, BLOCKS),
                                           (128, 64, 768, BLOCKS), (128, 64, 770, TILES), (128, 128, 1024, BLOCKS), (128, 128, 1026, TILES)])
def test_arg_max_of_short_contractions(rules, B, D, tiles, way):
    C = 64 * (tiles // ((B + 63) // 64))
    assert rules.way_(B, D, C, TOP1) == way
    assert rules.way_(B, D, C, PROBS) == (BLOCKS if tiles <= 1024 or B <= 64 else TILES)


def test_shapes_of_the_guard_band_tests(rules):
    """The kernels that the tags of test_gpu_guards.py name (the logits; the others are about dW)."""
    from tests.test_gpu_guards import SHAPES
    want = {"64 x 64 tiles": (BLOCKS, BLOCKS), "thin tiles only": (TILES, TILES), "full tiles only": (TILES, TILES),
            "forward on full and thin tiles, dz in lists": (LISTS, TILES), "full and thin tiles": (TILES, TILES),
            "forward on full and thin tiles, dz in lists, five batch tiles": (LISTS, TILES), "lists, five batch tiles": (LISTS, LISTS), "lists, nine k-steps": (LISTS, LISTS), "two rows": (SMALL, SMALL),
            "16 rows": (SMALL, SMALL), "20 rows": (SMALL, SMALL), "64 x 64 tiles, 64 rows": (BLOCKS, BLOCKS),
            "64 x 64 tiles, 61 rows": (BLOCKS, BLOCKS)}
    tiles = {"thin tiles only": range(1, 65), "full tiles only": range(65, 257), "full and thin tiles": range(257, 321),
             "forward on full and thin tiles, dz in lists": range(257, 321),
             "forward on full and thin tiles, dz in lists, five batch tiles": range(257, 321)}
    shapes = {s[0]: s[1:] for s in SHAPES}
    for tag, ways in want.items():
        B, D, C = shapes[tag]
        assert (rules.way_(B, D, C, STEP), rules.way_(B, D, C, FORWARD)) == ways, tag
        if tag in tiles:
            assert (B + 255) // 256 * ((C + 255) // 256) in tiles[tag], tag


def test_shapes_of_the_recompute_tests(rules):
    from tests.test_gpu_parity import RECOMPUTE_SHAPES
    want = {"64x64-tiles": (BLOCKS, BLOCKS, BLOCKS), "mixed-tiles": (TILES, TILES, TILES), "thin-tiles": (TILES, BLOCKS, BLOCKS),
            "lists-of-rests": (LISTS, BLOCKS, BLOCKS), "lists-of-whole-tiles": (LISTS, TILES, TILES), "16-rows": (SMALL,) * 3,
            "32-rows": (BLOCKS,) * 3, "32-rows-small-batch": (SMALL,) * 3, "64-rows": (BLOCKS,) * 3}
    for name, shape in RECOMPUTE_SHAPES.items():
        assert tuple(rules.way_(*shape, use) for use in (STEP, PROBS, TOP1)) == want[name], name
        assert rules.way_(*shape, FORWARD) == want[name][0], name


def test_shapes_of_the_dx_tests(rules):
    from tests.test_gpu_dx_splits import SHAPES
    out, got = (ctypes.c_int * 4)(), set()
    for B, D, widths in SHAPES:
        for C in widths:
            rules.dx_splits_(B, D, C, out)
            tiles = D // 64 * ((B + 63) // 64) if out[0] else (D + 255) // 256 * ((B + 255) // 256)
            got.add((out[0], tiles, out[1], out[2], (C + 63) // 64 - (out[1] - 1) * out[2]))
    assert {(0, 20, 9, 16, 13), (0, 44, 4, 16, 13), (0, 72, 2, 20, 20), (0, 32, 5, 16, 15), (1, 1, 18, 4, 3), (1, 4, 29, 7, 4),
            (1, 3, 14, 3, 2), (1, 33, 1, 21, 21), (1, 324, 1, 20, 20), (1, 312, 2, 21, 20), (1, 288, 1, 3, 3), (1, 10, 7, 3, 3)} <= got
