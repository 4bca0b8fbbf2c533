"""The pipelined kernels (ssa_kernel_pl, ssa_kernel_ph) where their parts meet, against the
oracle: trajectories around a wave, events around a batch and around a ring of batches, more
trajectories than lanes with one and two workgroups to a CU, snapshot rows around the LDS
table and many rows of one waiting time, zero guards that a large constant asks for, counts
that cross the exact range, records that wrap, suspended chains.

Counts, events and statuses are equal; the times of the last events agree to the
tolerance that the parity tests state for the format of the clock.
"""
import numpy as np
import pytest

from paper_2605_00479_amd import workloads as wl
from test_gpu_parity import gpu, run_both, run_records   # noqa: F401 (gpu is a fixture)

pytestmark = pytest.mark.gpu

MODES = ["FP64", "MIX_F16_SR", "MIX_F16_RTN", "UNI_F16_SR_NORM", "UNI_BF16_SRA"]


def pipelined(run):
    assert run.info()["block_size"] == 512


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("n", [1, 63, 64, 65, 129])
def test_trajectories_around_a_wave(gpu, orc, mode, n):
    run, _, _ = run_both(gpu, orc, wl.schlogl(), np.array([250], np.int32), n, 0.05, [0.0, 0.02, 0.05], mode, seed=n)
    pipelined(run)


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR", "UNI_BF16_SRA"])
@pytest.mark.parametrize("cap", [1, 2, 3, 4, 5, 7, 8, 9, 31, 32, 33, 40, 64, 129])
def test_event_caps_around_batches(gpu, orc, mode, cap):
    # 8 or fewer events to a batch, at most 16 batches in flight: every trajectory ends on
    # the cap and its lane takes the next
    run, _, st = run_both(gpu, orc, wl.birth_death(), np.array([3], np.int32), 300, 1e4, [1e4], mode, seed=cap,
                          max_events=cap, block_size=512, grid_size=1)
    pipelined(run)
    assert (st["n_events"] == cap).all()


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("grid", [1, 64, 128])
def test_many_short_trajectories(gpu, orc, mode, grid):
    # 4, 256 and 512 workgroups; ends of zero, one and a few events, refills all the time
    n = 1500 if grid == 1 else 40_000
    run, _, _ = run_both(gpu, orc, wl.birth_death(2.0, 1.0), np.array([0], np.int32), n, 1.5, [0.5, 1.0, 1.5],
                         mode, seed=4, block_size=512, grid_size=grid)
    pipelined(run)


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR", "UNI_F16_SR_NORM"])
@pytest.mark.parametrize("rows", [0, 1, 2, 511, 512, 513, 700, 1400])
def test_rows_around_the_table(gpu, orc, mode, rows):
    # some waiting times pass hundreds of rows (a slow network), most none
    snap = np.linspace(0.0, 40.0, rows) if rows > 1 else np.array([40.0][:rows])
    run, _, _ = run_both(gpu, orc, wl.birth_death(0.4, 0.1), np.array([1], np.int32), 200, 40.0, snap, mode,
                         seed=8, block_size=512, grid_size=1)
    pipelined(run)


def catalysed(k):
    """X made at rate 5, lost at rate k with the one catalyst Y (at once, for a large k) and in pairs."""
    return wl._build("catalysed", ["X", "Y"], [
        {"change": {"X": +1}, "k": 5.0},
        {"reactants": {"X": 1, "Y": 1}, "change": {"X": -1}, "k": k},
        {"reactants": {"X": 2}, "change": {"X": -2}, "k": 1.0},
    ])


@pytest.mark.parametrize("mode,k", [("FP64", 1e291), ("FP32", 1e21), ("MIX_BF16_SR", 1e21), ("FP64", 1e3),
                                    ("MIX_F16_SR", 1e4), ("UNI_F16_SR", 1e4)])
def test_guards_that_a_constant_asks_for(gpu, orc, mode, k):
    run, _, _ = run_both(gpu, orc, catalysed(k), np.array([0, 1], np.int32), 200, 10.0, wl.snapshot_grid(10.0, 11),
                         mode, seed=6)
    pipelined(run)


@pytest.mark.parametrize("mode,level", [("MIX_F16_SR", 2048.0), ("UNI_F16_SR", 2048.0), ("MIX_F16_RTN", 2048.0),
                                        ("MIX_BF16_SR", 256.0)])
@pytest.mark.parametrize("grid", [64, 128])
def test_exact_range_crossed_by_some_workgroups(gpu, orc, mode, level, grid):
    # the sets of a workgroup's lanes lie below, at and above the exact range of counts
    rates = np.array([[level * f, 1.0] for f in (0.3, 0.9, 0.97, 1.03, 1.6)])
    run, _, _ = run_both(gpu, orc, wl.birth_death(level, 1.0), np.array([int(level) - 3], np.int32), 5 * 4000, 0.05,
                         [0.02, 0.05], mode, seed=12, set_rate=rates, traj_per_set=4000, block_size=512,
                         grid_size=grid)
    pipelined(run)


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_RTN", "UNI_BF16_SR"])
@pytest.mark.parametrize("grid", [1, 128])
def test_suspended_chains_keep_their_place(gpu, orc, mode, grid):
    n = 300 if grid == 1 else 20_000
    run, _, _ = run_both(gpu, orc, wl.telegraph(), np.array([1, 0, 0], np.int32), n, 12.0, wl.snapshot_grid(12.0, 13),
                         mode, seed=2, block_size=512, grid_size=grid, n_chunks=4, first_window=2)
    pipelined(run)


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_RTN"])
def test_records_beside_refills(gpu, orc, mode):
    # a record of 5 entries overflows in some trajectories and stays empty in others
    run_records(gpu, orc, wl.telegraph(0.05, 0.05, 20.0, 1.0), np.array([1, 0, 0], np.int32), 700, 30.0,
                [10.0, 30.0], mode, 0b11, 5, seed=3, block_size=512, grid_size=1)


@pytest.mark.parametrize("mode", ["UNI_BF16_SR", "UNI_F16_SR", "UNI_BF16_SR_NORM", "UNI_BF16_RTN"])
def test_targets_rounded_up_to_the_total(gpu, orc, mode):
    # such a target selects the last reaction that can fire: here the last of all can in
    # some events only (Y is mostly zero), and X is always the last but one
    m = wl._build("tail", ["X", "Y"], [
        {"change": {"X": +1}, "k": 20.0},
        {"reactants": {"X": 1}, "change": {"Y": +1}, "k": 0.02},
        {"reactants": {"X": 1}, "change": {"X": -1}, "k": 1.0},
        {"reactants": {"Y": 1}, "change": {"Y": -1}, "k": 2.0},
    ])
    run, _, _ = run_both(gpu, orc, m, np.array([20, 0], np.int32), 640, 20.0, [10.0, 20.0], mode, seed=7,
                         max_events=5000)
    pipelined(run)
