"""Host-side launch-shape logic (es_spmm_launch_info): runs without a GPU.
Checks the invariants the kernels rely on before anything is launched."""
import itertools

import pytest

import paper_2104_10716_amd as es


SHAPES = [(1, 0), (7, 20), (2708, 13518), (170_000, 2_370_240), (233_000, 113_134_823),
          (2_450_000, 119_569_270)]
WIDTHS = [1, 2, 3, 4, 5, 16, 17, 41, 48, 64, 100, 128, 130, 256, 512, 602, 1024, 1028, 5000]


def _check(info, N, F, backward):
    G, CH, V = info["lanes_per_row"], info["chunks_per_lane"], info["vector_width"]
    R, E = info["rows_per_wave"], info["edge_slots"]
    assert V in (1, 4) and CH in (1, 2, 4) and G in (4, 8, 16, 32, 64)
    if info["flattened"]:
        assert R * G in (64, 128) and E * G == 64         # E or 2E rows per wave in the workgroup's run ...
        assert 4 * R <= 64                                # ... of which a lane of a wave describes one
    else:
        assert R * G * E == 64 and E >= 1                 # a wave is R rows x E slots x G lanes
    assert info["loads_in_flight"] * CH == 8
    assert info["tile_slots_per_row"] * R == es.es_spmm_tile_slots(1)
    assert G * CH * V * info["grid_y"] >= F               # every column is covered ...
    assert G * CH * V * (info["grid_y"] - 1) < F          # ... by no more column blocks than needed
    rows_per_workgroup = 4 * R
    row_groups = info["grid_x"] - info["long_row_workgroups"]
    if info["column_ranges"] == 8 and not info["flattened"]:   # a wave serves 4 rows; two sweeps per launch
        rows_per_workgroup *= 4
        assert info["long_row_workgroups"] == row_groups
    assert row_groups % 8 == 0                            # one equal share per XCD
    assert row_groups * rows_per_workgroup >= N
    assert (row_groups - 8) * rows_per_workgroup < N      # no more workgroups than needed, up to one per XCD
    assert info["long_row_workgroups"] % 8 == 0
    assert info["long_row_threshold"] >= 64
    if backward:
        assert V == 1 and info["aligned"] == 0
    if V == 4 and not info["aligned"]:
        assert F >= 4


@pytest.mark.parametrize("backward", [False, True])
def test_shape_invariants_over_sizes_and_widths(backward):
    for (N, nnz), F, mode, W in itertools.product(SHAPES, WIDTHS, ("full", "bucket", "fastrand"),
                                                  (1, 16, 128, 2304)):
        for aligned in (True, False):
            info = es.es_spmm_launch_info(N, nnz, F, W, mode, aligned16=aligned, backward=backward)
            _check(info, N, F, backward)
            if not backward:
                expect_aligned = aligned and F % 4 == 0
                assert info["aligned"] == int(expect_aligned)
                assert info["vector_width"] == (4 if F >= 4 else 1)


def test_long_rows_are_only_possible_when_the_long_part_is_launched():
    for (N, nnz), F in itertools.product(SHAPES, (16, 64, 128, 41)):
        full = es.es_spmm_launch_info(N, nnz, F, 0, "full", opts=dict(column_partition=-1))
        assert full["long_row_workgroups"] > 0            # nnz is only a hint: never gated by it
        assert full["column_ranges"] == 1
        auto = es.es_spmm_launch_info(N, nnz, F, 0, "full")
        # the column-partitioned product sweeps its rows twice per launch (long pieces first)
        if auto["column_ranges"] == 8 and not auto["flattened"]:
            assert auto["long_row_workgroups"] * 2 == auto["grid_x"]
        for W in (1, 16, 128, 512):
            s = es.es_spmm_launch_info(N, nnz, F, W, "fastrand")
            assert s["long_row_threshold"] >= 512 and s["long_row_workgroups"] == 0
        big = es.es_spmm_launch_info(N, nnz, F, 2304, "bucket")
        assert (big["long_row_workgroups"] > 0) == (2304 > big["long_row_threshold"])


def test_rows_up_to_about_four_times_the_mean_are_not_split():
    """Exact product and its transpose: the threshold is at least 64 and at least
    four times the mean, rounded down to a multiple of 64."""
    for N, mean, F, backward in itertools.product((300, 3000, 40_000, 2_450_000), (1, 15, 16, 20, 31, 32, 300, 1000),
                                                  (16, 41, 64, 128, 602), (False, True)):
        if N * mean >= 2 ** 31 or mean > N:
            continue
        info = es.es_spmm_launch_info(N, N * mean, F, 0, "full", backward=backward, opts=dict(column_partition=-1))
        assert info["long_row_threshold"] >= max(64, 4 * mean // 64 * 64), (N, mean, F, backward)


def test_options_are_honoured_and_clamped():
    base = es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket")
    info = es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket", opts=dict(rows_per_wave=64))
    assert info["lanes_per_row"] == 16 and info["rows_per_wave"] == 4      # lowered to fit G
    assert es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket", opts=dict(rows_per_wave=1))["rows_per_wave"] == 1
    info = es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket", opts=dict(long_row_threshold=7))
    assert info["long_row_threshold"] == 7 and info["long_row_workgroups"] > 0
    # options travel with the call: the next call without them sees the heuristic again
    assert es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket") == base
    assert base["long_row_workgroups"] == 0
    # an all-zero struct is the same as no struct
    assert es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket", opts={}) == base
    for bad in (dict(rows_per_wave=3), dict(rows_per_wave=-1), dict(lanes_per_row=12), dict(lanes_per_row=-2),
                dict(long_row_threshold=-4), dict(column_partition=-2)):
        with pytest.raises(es.EsSpmmError):
            es.es_spmm_launch_info(1000, 5000, 64, 8, "bucket", opts=bad)


def test_option_grid_keeps_the_shape_invariants():
    for (N, nnz), F, mode in itertools.product(SHAPES[1:], (3, 16, 41, 64, 128, 256, 602), ("full", "fastrand")):
        for rpw, lanes, thr in itertools.product((0, 1, 8, 64), (0, -1, 4, 8, 32, 64), (0, 1, 100)):
            opts = dict(rows_per_wave=rpw, lanes_per_row=lanes, long_row_threshold=thr)
            for backward in (False, True):
                info = es.es_spmm_launch_info(N, nnz, F, 64, mode, backward=backward, opts=opts)
                assert info["long_row_threshold"] >= (thr if thr else 64)
                if thr and info["column_ranges"] == 1:
                    assert info["long_row_threshold"] == thr
                G, CH, V = info["lanes_per_row"], info["chunks_per_lane"], info["vector_width"]
                assert info["rows_per_wave"] * G * info["edge_slots"] == (64 * info["rows_per_wave"] if info["flattened"] else 64)
                assert G * CH * V * info["grid_y"] >= F
                groups = 4 if info["column_ranges"] == 8 and not info["flattened"] else 1
                assert (info["grid_x"] - info["long_row_workgroups"]) * 4 * info["rows_per_wave"] * groups >= N


def test_column_slicing_option_only_narrows():
    base = es.es_spmm_launch_info(1000, 9000, 128, 8, "bucket", opts=dict(lanes_per_row=-1))
    assert base["lanes_per_row"] == 32 and base["grid_y"] == 1
    sliced = es.es_spmm_launch_info(1000, 9000, 128, 8, "bucket", opts=dict(lanes_per_row=8))
    assert sliced["lanes_per_row"] == 8 and sliced["chunks_per_lane"] == 1 and sliced["grid_y"] == 4
    _check(sliced, 1000, 128, False)
    wide = es.es_spmm_launch_info(1000, 9000, 16, 8, "bucket", opts=dict(lanes_per_row=8))
    assert wide["lanes_per_row"] == 4 and wide["grid_y"] == 1           # already narrower than 8 lanes
    bwd = es.es_spmm_launch_info(1000, 9000, 128, 8, "bucket", backward=True, opts=dict(lanes_per_row=8))
    assert bwd["lanes_per_row"] == 64                                   # the transposed product ignores it


def test_column_partition_choice():
    """Dense graph whose eighth of X is near an L2: partitioned for the exact
    product and for wide FastRand, never for Bucket, never for sparse graphs or
    for tables far beyond the L2s; the option forces it either way."""
    dense = (233_000, 113_134_823)
    assert es.es_spmm_launch_info(*dense, 64, 0, "full")["column_ranges"] == 8
    assert es.es_spmm_launch_info(*dense, 64, 256, "fastrand")["column_ranges"] == 1      # only on request
    assert es.es_spmm_launch_info(*dense, 64, 256, "fastrand", opts=dict(column_partition=1))["column_ranges"] == 8
    assert es.es_spmm_launch_info(*dense, 64, 256, "bucket")["column_ranges"] == 1
    assert es.es_spmm_launch_info(*dense, 64, 256, "bucket", opts=dict(column_partition=1))["column_ranges"] == 1
    assert es.es_spmm_launch_info(*dense, 64, 0, "full", opts=dict(column_partition=-1))["column_ranges"] == 1
    assert es.es_spmm_launch_info(170_000, 2_370_240, 128, 0, "full")["column_ranges"] == 1      # 14 per row
    assert es.es_spmm_launch_info(2_450_000, 119_569_270, 128, 0, "full")["column_ranges"] == 1  # X far too big
    forced = es.es_spmm_launch_info(170_000, 2_370_240, 128, 0, "full", opts=dict(column_partition=1, kernel=1))
    assert forced["column_ranges"] == 8 and forced["long_row_workgroups"] * 2 == forced["grid_x"]
    assert forced["long_row_workgroups"] % 8 == 0 and forced["lanes_per_row"] == 16
    forced = es.es_spmm_launch_info(170_000, 2_370_240, 128, 0, "full", opts=dict(column_partition=1))
    assert forced["column_ranges"] == 8 and forced["flattened"] == 1 and forced["lanes_per_row"] == 8
    assert es.es_spmm_launch_info(100, 5000, 64, 0, "full", opts=dict(column_partition=1))["column_ranges"] == 1
    assert es.es_spmm_launch_info(*dense, 64, 0, "full", backward=True)["column_ranges"] == 1


@pytest.mark.parametrize("N,mean,F,aligned,ranges,lanes", [
    # row form: rows of 256 entries on, and a product of mean and X of 4e9 bytes on
    (62_500, 150, 64, True, 1, 16), (62_501, 255, 64, True, 1, 16), (62_501, 256, 64, True, 8, 16), (70_000, 300, 41, False, 1, 16),
    (62_500, 255, 64, True, 1, 16), (32_000, 488, 64, True, 1, 16), (32_000, 489, 64, True, 8, 16), (70_000, 490, 41, False, 8, 16),
    # ... not for rows of one line, nor for wide rows that tile none on large tables
    (125_000, 490, 32, True, 1, 8), (125_000, 490, 36, True, 8, 16), (125_000, 300, 205, False, 8, 16), (125_001, 490, 205, False, 1, 64),
    (62_500, 490, 32, True, 1, 8), (125_000, 490, 24, False, 1, 8), (125_000, 490, 25, False, 8, 8),
    # ... wide aligned rows: 216 entries and 4.5e9 bytes on
    (70_000, 215, 128, True, 1, 32), (70_000, 216, 128, True, 8, 16), (40_000, 219, 128, True, 1, 32), (40_000, 220, 128, True, 8, 16),
    (62_500, 255, 96, True, 1, 32), (62_500, 255, 160, True, 1, 64), (70_000, 216, 300, True, 8, 16), (70_000, 255, 301, False, 1, 64),
    # flattened kernel: a product of 3.6e9 bytes on where rows tile lines, always where they do not, 4.1e9 and 19 MB up to F = 16
    (187_000, 150, 32, True, 1, 8), (188_000, 150, 32, True, 8, 8), (126_000, 300, 32, True, 8, 8), (350_000, 150, 16, True, 8, 4),
    (140_000, 200, 32, True, 1, 8), (142_000, 200, 32, True, 8, 8), (126_000, 128, 28, True, 8, 8), (126_000, 128, 36, True, 8, 16),
    (148_000, 300, 16, True, 1, 4), (149_000, 300, 16, True, 8, 4), (160_000, 200, 16, True, 1, 4), (161_000, 200, 16, True, 8, 4),
    (233_000, 127, 64, True, 1, 16), (233_000, 128, 64, True, 8, 8), (180_000, 300, 100, True, 8, 16)])
def test_column_range_rule(N, mean, F, aligned, ranges, lanes):
    info = es.es_spmm_launch_info(N, N * mean, F, 0, "full", aligned16=aligned)
    assert (info["column_ranges"], info["lanes_per_row"]) == (ranges, lanes)


@pytest.mark.parametrize("N,mean,F,lanes", [
    # exact product, whole rows: 32-column slices from 40 k to 140 k rows, else 64-column ones where they tile the row
    (58_593, 40, 64, 16), (58_594, 40, 64, 8), (58_594, 31, 64, 16), (58_594, 149, 64, 8), (58_594, 150, 64, 16), (140_000, 40, 64, 8),
    (29_296, 40, 128, 32), (29_297, 40, 128, 16), (39_999, 40, 128, 16), (40_000, 40, 128, 8), (40_000, 199, 128, 8), (40_000, 200, 128, 32),
    (140_001, 40, 128, 16), (100_000, 31, 128, 16), (100_000, 10, 128, 16), (100_000, 9, 128, 32), (99_999, 31, 128, 32), (488_282, 31, 128, 32),
    (39_999, 40, 96, 32), (40_000, 40, 96, 8), (140_001, 40, 96, 32), (100_000, 40, 100, 32), (100_000, 40, 48, 16), (500_000, 40, 128, 16)])
def test_exact_slices_of_middling_tables(N, mean, F, lanes):
    info = es.es_spmm_launch_info(N, N * mean, F, 0, "full")
    assert info["column_ranges"] == 1 and info["lanes_per_row"] == lanes
    assert es.es_spmm_launch_info(N, N * mean, F, 0, "full", opts=dict(kernel=1))["lanes_per_row"] >= 16
    assert es.es_spmm_launch_info(N, N * mean, F, 0, "full", aligned16=False)["flattened"] == 0


@pytest.mark.parametrize("N,mean,F,lanes,flattened", [
    # F = 64 takes 16 lanes on the row kernel and in 64-column slices alike: which of the two runs is asked for too
    (58_593, 40, 64, 16, 0), (58_594, 31, 64, 16, 0), (58_594, 32, 64, 8, 1), (58_594, 150, 64, 16, 0), (99_999, 31, 64, 16, 0),
    (100_000, 15, 64, 16, 0), (100_000, 16, 64, 8, 1), (200_000, 15, 64, 16, 0), (200_000, 16, 64, 8, 1), (200_000, 127, 64, 8, 1),
    (200_001, 63, 64, 16, 0), (200_001, 64, 64, 16, 0), (200_001, 79, 64, 16, 0), (200_001, 80, 64, 16, 1),
    (39_999, 32, 192, 16, 1), (40_000, 32, 192, 8, 1), (99_999, 31, 192, 64, 0), (100_000, 15, 192, 64, 0), (100_000, 16, 192, 8, 1),
    (200_000, 16, 192, 8, 1), (200_001, 63, 192, 64, 0), (200_001, 64, 192, 8, 1), (260_416, 64, 192, 8, 1), (260_417, 64, 192, 64, 0),
    (29_296, 40, 128, 32, 0), (29_297, 40, 128, 16, 1), (40_000, 40, 128, 8, 1), (140_001, 40, 128, 16, 1), (100_000, 9, 128, 32, 0),
    (99_999, 31, 256, 64, 0), (100_000, 10, 256, 16, 1), (140_001, 40, 320, 16, 1), (140_001, 40, 96, 32, 0)])
def test_exact_slices_and_the_kernel_that_runs_them(N, mean, F, lanes, flattened):
    info = es.es_spmm_launch_info(N, N * mean, F, 0, "full")
    assert (info["column_ranges"], info["lanes_per_row"], info["flattened"]) == (1, lanes, flattened)


def test_flattened_kernel_choice():
    """Without options the flattened kernel runs where narrow column slices pay:
    the partitioned product once a 64-column share outgrows an L2, and tables of
    0.3 GB and more with F >= 128; the row kernel everywhere else."""
    big = es.es_spmm_launch_info(2_450_000, 119_569_270, 128, 32, "fastrand")
    assert big["flattened"] == 1 and big["lanes_per_row"] == 8 and big["grid_y"] == 4 and big["rows_per_wave"] == 16
    exact = es.es_spmm_launch_info(2_450_000, 119_569_270, 128, 0, "full")
    assert exact["flattened"] == 1 and exact["rows_per_wave"] == 8            # one row per slot: evens the waves out
    row = es.es_spmm_launch_info(2_450_000, 119_569_270, 128, 32, "fastrand", opts=dict(kernel=1))
    assert row["flattened"] == 0 and row["lanes_per_row"] == 16
    dense = es.es_spmm_launch_info(233_000, 113_134_823, 64, 0, "full")
    assert dense["flattened"] == 1 and dense["column_ranges"] == 8 and dense["lanes_per_row"] == 8
    small = es.es_spmm_launch_info(58_250, 27_659_516, 64, 0, "full")
    assert small["flattened"] == 0 and small["column_ranges"] == 8 and small["lanes_per_row"] == 16
    assert es.es_spmm_launch_info(233_000, 113_134_823, 64, 64, "fastrand")["flattened"] == 0
    assert es.es_spmm_launch_info(233_000, 113_134_823, 256, 64, "fastrand")["flattened"] == 0   # 0.24 GB table
    assert es.es_spmm_launch_info(170_000, 2_370_240, 128, 16, "bucket")["flattened"] == 0
    assert es.es_spmm_launch_info(2_450_000, 119_569_270, 128, 32, "fastrand", backward=True)["flattened"] == 0
    # rows that do not tile 128-byte lines (F = 41, stride 41) keep the row kernel on whole rows
    odd = es.es_spmm_launch_info(233_000, 113_134_823, 41, 0, "full", aligned16=False)
    assert odd["flattened"] == 0 and odd["column_ranges"] == 8 and odd["lanes_per_row"] == 16


def test_flattened_kernel_option():
    for F, G in ((16, 4), (64, 16), (128, 32), (256, 64), (602, 64), (41, 16)):
        info = es.es_spmm_launch_info(100_000, 1_000_000, F, 16, "fastrand", aligned16=(F % 4 == 0),
                                      opts=dict(kernel=2, lanes_per_row=-1))
        assert info["flattened"] == 1 and info["lanes_per_row"] == G and info["chunks_per_lane"] == 1
        assert info["rows_per_wave"] == min(128 // G, 16) and info["edge_slots"] == 64 // G   # sampled: two rows per slot
        assert info["grid_y"] == -(-F // (4 * G))
        _check(info, 100_000, F, False)
    assert es.es_spmm_launch_info(1000, 5000, 3, 2, "bucket", opts=dict(kernel=2))["flattened"] == 0    # F < 4
    assert es.es_spmm_launch_info(1000, 5000, 64, 2, "bucket", backward=True, opts=dict(kernel=2))["flattened"] == 0
    assert es.es_spmm_launch_info(1000, 5000, 64, 2, "bucket", opts=dict(kernel=1))["flattened"] == 0
    part = es.es_spmm_launch_info(10_000, 5_000_000, 64, 0, "full", opts=dict(kernel=2, column_partition=1))
    assert part["flattened"] == 1 and part["column_ranges"] == 8 and part["long_row_workgroups"] == 0
    fr = es.es_spmm_launch_info(10_000, 5_000_000, 64, 9, "fastrand", opts=dict(kernel=2, column_partition=1))
    assert fr["flattened"] == 0 and fr["column_ranges"] == 8                # FastRand pieces: the row form
    with pytest.raises(es.EsSpmmError):
        es.es_spmm_launch_info(1000, 5000, 64, 2, "bucket", opts=dict(kernel=3))


def test_bad_sizes_are_rejected():
    for kw in (dict(N=0), dict(F=0), dict(W=0), dict(mode=5), dict(nnz=-1), dict(ldx=3)):
        a = dict(N=10, nnz=20, F=4, W=2, mode="bucket", ldx=None)
        a.update(kw)
        with pytest.raises(es.EsSpmmError):
            es.es_spmm_launch_info(a["N"], a["nnz"], a["F"], a["W"], a["mode"], ldx=a["ldx"])
    # grids beyond what a launch can carry are refused, not truncated
    with pytest.raises(es.EsSpmmError):
        es.es_spmm_launch_info(2 ** 40, 0, 4, 1, "bucket")
