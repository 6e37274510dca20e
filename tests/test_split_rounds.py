"""Plans of the streaming kernel (host only): numbers of column-space splits where the matrix cores bound a launch (items fill
whole rounds of the chip, fp32 chains of sums and the workspaces that callers provide stay within what they were), and
which of its two builds runs."""
import re

import pytest

from paper_2510_14891_amd import binding as mt


def describe(dims, R, k, sbytes):
    return {a: b for a, b in re.findall(r"(\w+)=(-?\d+)", mt.mttkrp_plan_describe(dims, R, k, sbytes).split("|")[-1])}


def test_first_mode_takes_a_round_fewer_where_memory_forbids_the_nearest():
    p = describe([129, 129, 129, 12], 500, 0, 8)
    assert int(p["items"]) <= 2048 and int(p["items"]) > 1900


# At low rank, HBM bounds the launch and shorter items win.  The nearest number of rounds is beyond the cap on memory for these
# calls, and a round fewer (4080, 6072 and 8192 items of 33 to 45 steps) is within it.
@pytest.mark.parametrize("dims,R,items,steps", [([160, 163, 10, 65], 9, 6500, 21), ([1440, 39, 1206], 14, 7360, 37), ([96, 24, 16, 1425], 6, 11400, 24)])
def test_first_mode_at_low_rank_keeps_its_items(dims, R, items, steps):
    p = describe(dims, R, 0, 8)
    assert p["col_blocks"] == "1" and p["paired_rows"] == "0"
    assert int(p["items"]) == items and int(p["steps_per_item"]) == steps, p


@pytest.mark.parametrize("dims,R,k", [([65, 66, 36, 24], 36, 3), ([16, 16, 16, 16, 24, 8], 85, 5), ([16, 8, 16, 8, 16, 16], 52, 3)])
def test_other_modes_leave_little_of_the_last_item_of_a_simd_idle(dims, R, k):
    items = int(describe(dims, R, k, 8)["items"])
    assert items / (1024.0 * -(-items // 1024)) > 0.85


@pytest.mark.parametrize("dims,R", [([27, 21, 15, 12, 31], 2038), ([10, 6, 15, 2, 9, 6, 39], 959), ([3, 28, 12, 10, 1, 7, 49], 842),
                                    ([1, 13, 55, 12, 2, 152, 30], 263), ([16, 36, 14, 108, 2, 10], 398)])
def test_sweeps_near_their_limit_stay_supported(dims, R):
    n = 4
    for d in dims:
        n *= d
    assert 0 < mt.mttkrp_dense_all_modes_shared_bytes(dims, R, 4) <= max(64 << 20, n // 8)


@pytest.mark.parametrize("dims,R,sbytes", [([1000000, 20, 20], 32, 4), ([400000, 7, 6], 40, 8)])
def test_one_range_of_the_column_space_leaves_no_wavefront_idle(dims, R, sbytes):
    p = describe(dims, R, 0, sbytes)
    assert p["outer_splits"] == p["inner_splits"] == "1" and p["items"] == p["row_blocks"], p


# (one column block in fp32: the run keeps X's addresses in 64-bit pointers of the lanes)
@pytest.mark.parametrize("dims,R,k,sbytes,rows,cols", [([200000, 16, 140, 30], 16, 2, 4, 64, 1), ([200000, 16, 140, 128], 10, 2, 4, 64, 1)])
def test_runs_of_lane_pointers_take_any_stride(dims, R, k, sbytes, rows, cols):
    p = describe(dims, R, k, sbytes)
    assert p["rows_per_wave"] == str(rows) and p["col_blocks"] == str(cols) and p["inner_mode"] == "3"
    assert 3 * dims[0] * dims[1] * dims[2] * sbytes > 2 ** 32
    assert int(p["steps_per_item"]) >= 32 and p["deep"] == "1", p


# (stride of the inner mode times four columns: below and beyond 2^32 bytes; extents of one kind otherwise)
@pytest.mark.parametrize("dims,R,k,sbytes,deep", [([100000, 16, 80, 32], 32, 2, 8, 1), ([100000, 16, 120, 32], 32, 2, 8, 0),
                                                  ([100000, 16, 120, 32], 32, 2, 4, 1), ([200000, 16, 140, 30], 64, 2, 4, 0),
                                                  ([200000, 16, 100, 30], 64, 2, 4, 1)])
def test_the_run_is_built_in_only_where_its_offsets_fit(dims, R, k, sbytes, deep):
    p = describe(dims, R, k, sbytes)
    inner = int(p["inner_mode"])
    stride = 1
    for d in dims[:inner]:
        stride *= d
    assert ((3 * stride + 64) * sbytes < 2 ** 32) == bool(deep)
    assert int(p["steps_per_item"]) >= 32 and int(p["deep"]) == deep, p
