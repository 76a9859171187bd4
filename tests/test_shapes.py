"""Which variant the rules of the library choose: for the calls that the parity tests make of them, so that every
variant meets the oracle and every test runs what it names."""
import test_gpu_parity as gp
from shapes import COMMON, ROWS, STORE, eq_pairs, few, grid, infer, onehot_bytes, setup, split_early, staged

ALL_INFER = {"ahead1", "ahead2", "ahead4", "infer1", "infer2", "infer4"}


def one(cases):
    return {(binary,) + infer(NI, H, d, not binary) for binary, NI, H, d in cases}


def asked(cases):
    return {(binary,) + infer(NI, H, d, not binary, tile=how) for how, binary, NI, H, d in cases}


def forest(cases):
    return {(binary,) + infer(NI, H, d, not binary, ntrees=nt) for binary, nt, NI, H, d in cases}


def test_inference_cases_run_what_they_name():
    single = one(gp.SINGLE_WAVEFRONT_TILES)
    assert {k for _, k, _ in single} == {"infer1"} and {n for _, _, n in single} == {2, 3, 4}, single
    ahead = one(gp.AHEAD_TILES)
    assert {(b, k) for b, k, _ in ahead} == {(b, k) for b in (False, True) for k in ("ahead1", "ahead2", "ahead4")}, ahead
    few_inst = forest(gp.FOREST_FEW)
    assert {k for _, k, _ in few_inst} == {"ahead1"} and {n for _, _, n in few_inst} == {1, 2, 3, 4}, few_inst
    small = asked(gp.SMALL_FORCED_TILES)
    assert {k for _, k, _ in small} == {"ahead1", "ahead2", "infer1", "infer2"}, small
    wide = asked(gp.WIDE_FORCED_TILES)
    assert {(b, k) for b, k, _ in wide} == {(b, k) for b in (False, True) for k in ("infer2", "infer4")}, wide
    groups = forest(gp.ONE_OR_TWO_GROUPS_FORESTS)
    assert groups == {(b, "infer1", n) for b in (False, True) for n in (1, 2)}, groups
    assert asked(gp.ONE_OR_TWO_GROUPS_TILES) == {(b, "infer1", 2) for b in (False, True)}


def test_every_inference_variant_meets_the_oracle():
    """Both modes of every kernel; k_infer in single wavefronts with staged sums and without."""
    seen = set()
    for b, k, n in (one(gp.SINGLE_WAVEFRONT_TILES + gp.AHEAD_TILES) | asked(gp.SMALL_FORCED_TILES + gp.WIDE_FORCED_TILES + gp.ONE_OR_TWO_GROUPS_TILES)
                    | forest(gp.FOREST_FEW + gp.ONE_OR_TWO_GROUPS_FORESTS)):
        seen.add((b, k, k == "infer1" and staged(n, not b)))
    assert seen == {(b, k, False) for b in (False, True) for k in ALL_INFER} | {(True, "infer1", True)}, seen
    # staged sums only where they measured faster (see group_sums)
    assert [staged(n, thr) for thr in (False, True) for n in (1, 2, 3)] == [True, False, False, False, False, False]


def test_grid_variants_meet_the_oracle():
    """The grids with issue priorities: two sums level by level, the others at the full sizes of the census table (own rows) and of
    the level on 10^6 samples (a tree level, the leaf one-hot)."""
    n, d = gp.OWN_ROWS_ALONE
    assert grid(ROWS, d, n)["alone"] and grid(ROWS, d, n)["ranges"] == grid(COMMON, d, n)["ranges"]
    _, N, H, d = gp.LEVELWISE_LARGE
    assert not grid(COMMON, 1 << (H - 1), N, sums=2)["alone"]
    assert not grid(ROWS, 294, 48842)["alone"]
    assert not grid(COMMON, 64, 1000000)["alone"]
    assert not grid(STORE, 128, 48842, tile_sums=False)["alone"] and not grid(STORE, 64, 48842, tile_sums=True)["alone"]
    assert grid(STORE, 128, 1000000, tile_sums=True)["alone"] and not grid(STORE, 256, 1000000)["alone"]


def test_grids_of_three_wavefronts_meet_the_oracle():
    """Shared arrays at sizes of their own; the leaf one-hot, with its sums and without, at the full size of the census table.  Own rows and two sums never take three (see column_ranges)."""
    for w, n in gp.OAA_THREE_WAVEFRONTS:
        assert grid(COMMON, w, n)["waves"] == 3, (w, n)
    assert [grid(STORE, 64, 48842, tile_sums=True)[k] for k in ("waves", "alone")] == [3, False]
    assert [grid(STORE, 128, 48842)[k] for k in ("waves", "alone")] == [3, False]
    assert [grid(STORE, 128, 1000000, tile_sums=True)[k] for k in ("waves", "alone")] == [2, True]
    for w, n in ((5, 30), (64, 48842), (300, 200003)):
        assert grid(ROWS, w, n)["waves"] == grid(COMMON, w, n, sums=2)["waves"] == 2, (w, n)
    assert [grid(COMMON, w, n)["waves"] for w, n in ((64, 48842), (28, 89221), (733, 8477), (939, 4061))] == [2] * 4     # measured faster
    assert [grid(COMMON, w, n)["waves"] for w, n in ((49, 49820), (25, 100666), (18, 127049), (70, 50207), (1044, 9027), (3492, 3152))] == [2] * 6
    assert [grid(COMMON, w, n)["waves"] for w, n in ((390, 25221), (30, 121599), (54, 73408), (1463, 12735), (2480, 15069), (2920, 5980))] == [3] * 6


def test_count_few_cases_run_what_they_name():
    for N, d, K, H in gp.COUNT_FEW_NARROW:
        assert all(few(1 << h, N, d * K + K) == (h <= 3) for h in range(H)), (N, d, K)
    for N, d, K, H in gp.COUNT_FEW_WIDE:
        assert not any(few(1 << h, N, d * K + K) for h in range(H)), (N, d, K)


def test_onehot_takes_the_faster_route():
    """One launch or two (see onehot_bytes): on the side that measured faster, and the parity test's levels on both."""
    for np_, d in ((64, 64), (256, 64), (512, 20), (32, 300), (16, 2000), (8, 4000), (4, 4096)):
        assert onehot_bytes(np_, d), (np_, d)
    for np_, d in ((1024, 20), (512, 64), (128, 300), (1024, 300), (32, 2000), (1, 10000), (32, 10000)):
        assert not onehot_bytes(np_, d), (np_, d)
    for N, d, H in gp.PRODUCTS_WORDS:
        assert not onehot_bytes(1 << (H - 1), d) and (d > 4096 or onehot_bytes(1 << (H - 2), d)), (N, d, H)


def test_node_split_loads_on_the_faster_side():
    """Before the block function or after it (see split_early): on the side that measured faster; both variants meet the oracle."""
    for nodes, N, ncol in ((1, 267, 46), (16, 267, 46), (512, 5000, 244), (256, 5000, 590), (16, 20000, 130)):
        assert split_early(nodes, N, ncol), (nodes, N, ncol)
    for nodes, N, ncol in ((1, 48842, 306), (64, 48842, 590), (4096, 3000, 123), (2048, 20000, 130)):
        assert not split_early(nodes, N, ncol), (nodes, N, ncol)
    for N, d, K, H in gp.SPLIT_LATE:
        assert not split_early(1 << (H - 1), N, d * K + K, 6) and split_early(1 << (H - 2), N, d * K + K, 6), (N, d, K, H)


def test_equality_sizes_lie_on_both_sides():
    assert [eq_pairs(n) for n in gp.EQUALITY_PAIRS] == [False] + [True] * (len(gp.EQUALITY_PAIRS) - 1)
    n0 = next(n for n in gp.EQUALITY_PAIRS if eq_pairs(n))
    assert not eq_pairs(n0 - 1) and gp.EQUALITY_PAIRS[0] == n0 - 1
    assert {n % 40 for n in gp.EQUALITY_PAIRS[1:]} >= {0, 1, 19, 21, 39}


def test_setup_shapes_run_what_they_name():
    """Both storage forms x both class variants with parts of several features; parts of 32; workgroups with a second item in both forms."""
    seen = [(setup(*s), s[1], s[2]) for s in gp.SETUP_SPLITS]
    assert {(s["comps"], K > 4) for s, d, K in seen if s["features"] >= 17} == {(c, k) for c in (False, True) for k in (False, True)}
    assert [(s["features"], d) for s, d, K in seen] == [(32, 32), (17, 33), (32, 64), (22, 65), (32, 32), (32, 64), (32, 64)]
    assert {(s["comps"], K > 4) for s, d, K in seen if s["items"] > s["groups"] and d > s["features"]} == {(True, False), (False, True)}


def test_many_columns_fill_the_chip():
    """More than half of the SIMDs' worth of tiles: one range only where the columns are few (see column_ranges)."""
    for n in (100003, 140244, 168657):
        assert grid(COMMON, 32, n)["ranges"] >= 2 and grid(COMMON, 3, n)["ranges"] == 1, n
    assert grid(ROWS, 20, 140244)["ranges"] == grid(ROWS, 17, 168657)["ranges"] == 2
    assert [grid(COMMON, w, 360000)["alone"] for w in (2, 3, 6)] == [True, True, False] and not grid(COMMON, 2, 534134)["alone"]
    for n, w, ranges in ((445, 669, 335), (3604, 57, 29), (6495, 248, 25)):        # few rows: a wavefront per SIMD
        assert grid(COMMON, w, n)["ranges"] == ranges and grid(COMMON, w, n)["alone"], n


def test_two_columns_take_the_faster_split():
    """Two columns in one range, or in two with the launch that completes the sums: on the side that measured faster (see
    column_ranges), for few rows and for many."""
    for n in (13, 267, 3000, 10000):
        assert grid(ROWS, 2, n)["ranges"] == 2 and grid(COMMON, 2, n, sums=2)["ranges"] == 2, n
        assert grid(COMMON, 2, n)["ranges"] == 1, n
    assert grid(COMMON, 3, 45753)["ranges"] == 1 and grid(COMMON, 4, 30000)["ranges"] == 4
    assert grid(ROWS, 2, 30000)["ranges"] == 1 and grid(COMMON, 2, 30000, sums=2)["ranges"] == 2
    for n in (60000, 170000):
        assert grid(ROWS, 2, n)["ranges"] == grid(COMMON, 2, n, sums=2)["ranges"] == grid(COMMON, 2, n)["ranges"] == 1, n


def test_lone_label_runs_ahead():
    """Trees of depth 0: the kernel for few instances wherever it takes them (see infer_shape)."""
    for n in (1, 137, 2699, 12110, 30000):
        for thr in (False, True):
            assert infer(n, 0, 2, thr)[0] == "ahead1", n
    assert infer(60386, 0, 7, False)[0] == "infer1"
    assert [infer(49, 0, 2, False, tile)[0] for tile in (16, 32, 64)] == ["ahead1", "ahead1", "ahead2"]


def test_asked_tiles_of_wide_rows():
    """Tiles asked for: ten columns a step up to 249, at least 21 from 250 on (see infer_shape)."""
    for thr in (False, True):
        assert [infer(208758, 3, d, thr, 32)[0] for d in (100, 200, 373, 600)] == ["infer2", "infer2", "infer4", "infer4"]
        assert [infer(208758, 3, d, thr, 16)[0] for d in (100, 200, 373, 600)] == ["infer1", "infer1", "infer2", "infer2"]
        assert [infer(208758, 3, d, thr, 64)[0] for d in (20, 100, 373)] == ["infer2", "infer4", "infer4"]
        assert [infer(208758, 3, d, thr, 32)[0] for d in (20, 30, 47)] == ["infer1"] * 3      # narrow rows: the fewest that hold the tile
        assert [infer(208758, 12, d, thr, 32)[0] for d in (20, 30, 64)] == ["infer1", "infer2", "infer2"]
        assert infer(25000, 3, 300, thr, 32)[0] == "infer2" and infer(25000, 3, 300, thr, 16)[0] == "infer1"
