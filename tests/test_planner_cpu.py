"""The planner's tables and workspace, without a GPU."""
import pytest

from tests.planner import plan

N_MAX = 2 ** 31 - 1     # elements, rows or columns the boundary admits per tensor


@pytest.mark.parametrize("rows,cols", [(N_MAX, 1), (1, N_MAX), (N_MAX - 40, 1), (1, N_MAX - 254), (2 ** 30 - 1, 2), (3, N_MAX // 3)])
def test_block_counts_at_the_size_limit(rows, cols):
    # the counts are ceilings of sizes up to 2^31 - 1: m + 255 does not fit 32 signed bits
    r = plan([(rows, cols)])
    t = r["tensors"][0]
    up = lambda a, b: -(-a // b)
    assert (t["nrt"], t["nct"]) == (up(rows, t["TR"]), up(cols, 256)) and t["TR"] <= 1024
    assert (t["nrblk"], t["ncblk"]) == (up(rows, 256), up(cols, 256))
    assert r["n_tiles"] == t["nrt"] * t["nct"] and r["n_rcitems"] == t["nrblk"] + t["ncblk"]
    pad4 = lambda a: up(a, 4) * 4
    size = [t["nct"] * rows, t["nrt"] * cols, 3 * pad4(rows), 3 * pad4(cols), 12 * r["n_rcitems"], 20 * r["n_tiles"], 32, 32]
    at = t["regions"]
    for k, s in enumerate(size):   # regions in order, none overlapping the next
        assert at[k] + s <= at[k + 1]
    assert at[-1] < r["ws_floats"] < 2 ** 36
    assert t["state_bytes"] == 4 * (4 * pad4(rows * cols) + 3 * pad4(rows) + 3 * pad4(cols))


def test_only_the_kernels_that_read_apply_tiles_get_them():
    # VeLO's kernels walk the statistics tiles: no table of apply tiles to upload or to count against lopt_step_static's array
    shapes = [(5504, 2048)] * 4 + [(1, 300)] * 50
    velo, fc = plan(shapes, kind="velo"), plan(shapes)
    assert velo["n_atiles"] == 0 and fc["n_atiles"] > 0
    assert fc["table_bytes"] - velo["table_bytes"] >= 16 * fc["n_atiles"]


@pytest.mark.parametrize("hidden,groups", [(32, 3), (16, 1), (8, 1), (4, 1)])
def test_apply_tiles_shorten_once_per_launch(hidden, groups):
    # 134 M elements: three tensor groups, but only the strip kernel (width 32) is launched once per group; every launch has
    # tiles of full height, then half, then a quarter
    runs = [h for h, _ in plan([(8192, 4096)] * 4, hidden=hidden)["atile_runs"]]
    assert runs == [128, 64, 32] * groups


@pytest.mark.parametrize("count,groups", [(1, 1), (3, 4), (7, 4), (9, 8), (20, 8)])
def test_tensor_groups_of_long_lists(count, groups):
    # tensors of 64 M elements, 8192 x 8192: a single one is not cut, 512 M elements and more go in eight groups
    assert [h for h, _ in plan([(8192, 8192)] * count)["atile_runs"]] == [128, 64, 32] * min(groups, count)


@pytest.mark.parametrize("hidden,per_cu,least", [(32, 2, 2), (16, 4, 2), (8, 3, 8), (4, 4, 8)])
@pytest.mark.parametrize("shapes", [[(256, 256), (1, 256), (64, 256)], [(1000, 1000)], [(1700, 1400)], [(40, 30)]])
def test_short_lists_are_one_round_of_equal_tiles(hidden, per_cu, least, shapes):
    # two tiles per CU if 32 rows suffice, otherwise as many as the kernel has workgroups there (otherwise graded heights); no
    # tile lower than one trip of the two wavefronts that share a column segment
    r = plan(shapes, hidden=hidden)
    tiles = lambda ar: sum(-(-m // ar) * -(-n // 128) for m, n in shapes)
    heights = [ar for ar in (2, 4, 6, 8, 12, 16, 20, 24, 32) if ar >= least]
    want = [ar for k in (2, per_cu) for ar in heights if tiles(ar) <= 256 * k]
    if not want:
        assert hidden == 32 and shapes == [(1700, 1400)]   # 594 tiles of 32 rows
        return
    top = max(h for h, _ in r["atile_runs"])
    assert top == min(want[0], max(m for m, _ in shapes)) and r["n_atiles"] == tiles(want[0])


SUBLIST = [(8216, 549), (9, 1024), (2059, 48), (528, 36), (144, 8211)]   # tests/test_gpu_optim_wrapper.py steps it without the third


def test_a_part_of_a_list_may_need_more_workspace_than_the_whole():
    # what a caller that steps parts of a list has to provide for: the shorter list falls below the tile count from which tiles
    # keep their full height
    whole, part = plan(SUBLIST), plan(SUBLIST[:2] + SUBLIST[3:])
    assert part["tensors"][0]["TR"] < whole["tensors"][0]["TR"] and part["ws_floats"] > 1.5 * whole["ws_floats"]


# Lists of the GPU tests whose point is the shape of the tiles they get, and what the planner makes of them.
NARROW = [(2100, 129), (1301, 192), (131149, 17), (700, 65), (9, 40)]
UNALIGNED = [(70007, 5), (12005, 61), (8003, 125), (5003, 190), (2001, 449), (1003, 257), (515, 65), (70003, 3)]


@pytest.mark.parametrize("hidden,resident", [(4, 1024), (8, 768), (16, 1024)])
def test_the_narrow_width_list_reaches_full_tiles_and_second_tiles_of_a_workgroup(hidden, resident):
    r = plan(NARROW, hidden=hidden)
    # 128 rows: four and eight trips of the two and four wavefronts that share a segment at widths 4 and 8; ragged last rows
    assert [h for h, _ in r["atile_runs"]] == [128, 52, 128, 21, 128, 64, 32, 13, 32, 28, 9]
    assert r["n_atiles"] > 1.5 * resident


def test_the_unaligned_list_reaches_tiles_of_ordinary_height_and_every_number_of_segments():
    r = plan(UNALIGNED, kind="velo", lstm_hidden=32, n_bank=8)
    assert [t["TR"] for t in r["tensors"]] == [320, 64, 64, 64, 64, 64, 64, 320]
    # 64-column segments of a tensor's last tile
    seg = {-(-(n - 256 * ((n - 1) // 256)) // 64) for _, n in UNALIGNED}
    assert seg == {1, 2, 3, 4} and all(m % 16 and n % 4 for m, n in UNALIGNED)


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_short_lists_are_not_cut_into_tensor_groups(kind):
    # the groups of a caller's own, which such lists only lose by, leave the plan of a short list as it is; a tensor of more than
    # 6144 rows makes a list of the other form
    for shapes, short in (([(4096, 2560)] * 4 + [(2560,)] * 4, 1), ([(6145, 1707)] * 4 + [(2560,)] * 4, 0), ([(300, 257), (5,), (64, 256)], 1)):
        r, one = plan(shapes, kind=kind, groups=3), plan(shapes, kind=kind, groups=1)
        assert r["short_list"] == one["short_list"] == short
        assert (r["groups"], one["groups"]) == (1 if short else 3, 1)
        if short:
            assert r == one


@pytest.mark.parametrize("kind,hidden", [("small_fc_lopt", 32), ("small_fc_lopt", 16), ("velo", 4)])
def test_which_tiles_the_statistics_pass_leaves_in_the_cache(kind, hidden):
    # up to 15.5 M elements (11 M off the 16-byte grid) all, beyond it those of the first 10 M (where the apply pass begins, so the pass goes backwards), for the
    # narrow widths none; rows off the 16-byte grid all, under VeLO from 13 M on those of the first 10 M
    velo, everything = kind == "velo", 2 ** 31 - 1
    for count in (1, 8, 12, 13, 15, 16, 40, 63):
        r = plan([(1024, 1024)] * count, kind=kind, hidden=hidden)
        first = r["n_tiles"] * 10 // count if count > 10 else r["n_tiles"]
        assert r["short_list"] == 1 and r["backwards"] == (count >= 16)
        assert r["keep"] == (everything if count < 16 else first if velo or hidden == 32 else 0)
        assert r["keep_off"] == (first if velo and count >= 13 else everything)
    assert [plan([(1024, 1025)] * count, kind=kind, hidden=hidden)["backwards"] for count in (10, 11, 14)] == [0, 1, 1]
    r = plan([(1024, 1024)] * 64, kind=kind, hidden=hidden)
    assert r["short_list"] == 0 and r["backwards"] == velo and r["keep"] == (r["n_tiles"] * 10 // 64 if velo else 0)


M = 1 << 20


@pytest.mark.parametrize("kind,hidden", [("small_fc_lopt", 32), ("small_fc_lopt", 16), ("velo", 4)])
@pytest.mark.parametrize("cols", [1024, 1000, 1025])
def test_which_loads_the_passes_take_by_size(kind, hidden, cols):
    # matrices, and a vector that brings the list to one element below each line or onto it. Strip kernel, off the 128-byte grid:
    # ordinary loads but from 7 to 13 M, on it up to 5.5 M. Other apply kernels, rows off the 16-byte grid: nontemporal from 6 (7) to 21
    # (18) M. Statistics of short lists, rows on the 16-byte but off the 128-byte grid: ordinary under VeLO and otherwise from 1.5 to 13 M.
    velo = kind == "velo"
    for line in (3 * M // 2, 11 * M // 2, 6 * M, 7 * M, 13 * M, 18 * M, 21 * M):
        for above in (0, 1):
            total = line - 1 + above
            rows, rest = divmod(total, cols)
            shapes = [s for s in [(1024, cols)] * (rows // 1024) + [(rows % 1024, cols), (1, rest)] if 0 not in s]
            assert sum(a * b for a, b in shapes) == total
            r = plan(shapes, kind=kind, hidden=hidden)
            assert r["short_list"] == 1 and r["n_rcitems"] == 0 and r["n_rcshort"] > 0
            assert r["keep_line"] == (velo or 3 * M // 2 <= total < 13 * M)
            assert r["off_grid_nt"] == ((6 if velo else 7) * M <= total < (21 if velo else 18) * M)
            if kind == "small_fc_lopt" and hidden == 32:
                ordinary = total < 7 * M or total >= 13 * M if cols != 1024 else total < 11 * M // 2
                assert r["strip_ordinary"] == (ordinary and not r["fold_finalize"])


def test_loads_of_long_lists_and_of_mixed_ones():
    big, odd = (8192, 8192), (8191, 6001)
    for kind in ("small_fc_lopt", "velo"):
        r = plan([big, odd], kind=kind)
        assert (r["short_list"], r["keep_line"], r["off_grid_nt"]) == (0, 0, 0)
        assert r["keep_off"] < r["n_tiles"] if kind == "velo" else r["keep_off"] == 2 ** 31 - 1
    # the strip kernel's loads go by the larger part of the list
    assert [plan(s)["strip_ordinary"] for s in ([big, odd], [big, odd, odd], [odd], [big])] == [0, 1, 1, 0]


def test_lists_that_fold_the_finalize_have_one_kind_of_strip_load():
    # their launch has no instantiation with ordinary loads: the plan says so
    for shapes, folds in (([(256, 256), (256,), (64, 256)], 1), ([(1000, 1000)], 1), ([(1200, 1200)], 1), ([(1700, 1400)], 0)):
        r = plan(shapes)
        assert (r["fold_finalize"], r["strip_ordinary"]) == (folds, 1 - folds)


@pytest.mark.parametrize("kind", ["small_fc_lopt", "velo"])
def test_lists_of_many_tiles_of_few_rows_are_no_short_lists(kind):
    short = lambda shapes: plan(shapes, kind=kind)["short_list"]
    assert [short([(768,)] * n) for n in (341, 342)] == [1, 0]          # three column tiles each
    assert [short([(15, 100)] * n) for n in (1024, 1025)] == [1, 0]
    assert short([(16, 100)] * 1500) == 1 and short([(64, 64)] * 1500 + [(20,)] * 1024) == 1
    assert short([(64, 64)] * 1500 + [(20,)] * 1025) == 0


@pytest.mark.parametrize("lstm_hidden,most", [(512, 96), (680, 96), (681, 80), (768, 80), (1024, 48), (9, 96)])
def test_the_recurrent_product_is_formed_ahead_where_it_leaves_room_for_the_sums(lstm_hidden, most):
    # up to 96 tensors and fewer than 512 workgroups of 16 tensors x 8 units
    ahead = lambda n: plan([(20, 20)] * n, kind="velo", lstm_hidden=lstm_hidden)["lstm_ahead"]
    assert [ahead(n) for n in (1, most, most + 1)] == [1, 1, 0]


@pytest.mark.parametrize("kind,line", [("small_fc_lopt", 1024), ("velo", 512)])
def test_column_sums_of_short_lists_are_doubles_of_64_or_128_rows(kind, line):
    for rows, tall in ((64, 64), (65, 64), (line, 64), (line + 1, 128), (6144, 128)):
        r = plan([(rows, 300)], kind=kind)
        sums = -(-rows // tall)
        assert r["short_list"] == 1 and r["n_rctiles"] == 2 * sums
        at = r["tensors"][0]["regions"]
        assert at[1] % 2 == 0 and 2 * sums * 300 <= at[2] - at[1] < 2 * sums * 300 + 64


def test_a_short_list_stays_within_the_fixed_scratch():
    # wide matrices of few rows whose workspace fits lopt_step_static's 64 MiB: with copies of c_k and column sums in double it would
    # not (69 MiB)
    wide = [(16, 20000)] * 110
    r, s = plan(wide, hidden=4), plan(wide[:60], hidden=4)
    assert r["short_list"] == 0 and r["n_rcitems"] > 0
    assert s["short_list"] == 1 and s["n_rcitems"] == 0 and 4 * s["ws_floats"] <= 48 << 20   # small enough for the copies
    assert 4 * s["ws_floats"] * 110 / 60 > 64 << 20 and 4 * r["ws_floats"] < 48 << 20
