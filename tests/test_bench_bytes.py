"""The byte counts that bench.py derives from a plan follow the schedule the
library runs: ragged tiles on three passes where they take them, and W rows
that are written, not read, at their first update.
"""
import pytest

import bench
from paper_2110_07670_amd import _lib


@pytest.mark.parametrize("n,prec,ragged", [
    (24, "fp64", "three_pass"), (96, "fp64", "three_pass"), (120, "fp64", "three_pass"),
    (128, "fp64", "four_pass"), (144, "fp64", "four_pass"), (32, "fp32", "four_pass"),
    (40, "fp32", "three_pass"), (96, "fp32", "three_pass"), (120, "fp32", "four_pass"),
    (128, "fp32", "three_pass"), (160, "fp32", "four_pass")])
def test_ragged_tiles(n, prec, ragged):
    plan = _lib.Plan(n, (10.0,) * 3, 37, prec, 0.25)
    block, full = plan.tiling[0], plan.schedule()[0]
    tiles, _ = bench.plan_tiles(plan)
    for bi, bj, _, _, kind in tiles:
        assert kind == (full if (bi, bj) == (block, block) else ragged)


def test_four_pass_schedule():
    plan = _lib.Plan(96, (10.0,) * 3, 37, "fp64", 0.25)
    plan.set_schedule(True)
    assert {t[4] for t in bench.plan_tiles(plan)[0]} == {"four_pass"}


def test_first_rows_are_not_read():
    tiles, npts = bench.tile_plan(128, 16), 96 ** 3
    all_read = bench.algorithmic_bytes("w_accumulate", tiles, npts, 8)
    assert all_read - bench.algorithmic_bytes("w_accumulate", tiles, npts, 8, True, 128) \
        == 128 * 8 * npts


@pytest.mark.parametrize("mode,stage", [(0, "x_poisson"), (1, "x_energy"), (4, "x_energy"),
                                        (2, "yz_fwd"), (3, "yz_inv")])
def test_line_kernels_have_a_stage(mode, stage):
    from paper_2110_07670_amd import profiling
    assert profiling.stage_of("void acex::k_lines<double, 96, %d, 16>(float)" % mode) == stage
