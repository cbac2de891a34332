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
