"""Networks whose counts can fall below zero: a loss of order zero or by a Hill law, a
first-order reaction that removes two. A mass-action reaction has propensity zero at a
count below its order, also a negative one; a Hill law takes the negative count. Every
launch shape gives the same trajectories: those of one wave for 64 trajectories, whose
guards test the counts themselves. (The oracle stops every mass-action reaction there,
also those of order zero, so it is no reference here.)
"""
import re

import numpy as np
import pytest

from paper_2605_00479_amd import ssa, workloads as wl
from test_gpu_parity import gpu   # noqa: F401 (gpu is a fixture)

MODES = ["FP64", "FP32", "MIX_F16_SR", "MIX_F16_RTN", "MIX_BF16_SR", "UNI_F16_SR", "UNI_F16_SRA",
         "UNI_BF16_SR_NORM"]


def zero_order_loss():
    """X is taken at a constant rate; its first- and second-order reactions stop below 1 and 2."""
    return wl._build("zero_order_loss", ["X", "Y"], [
        {"change": {"X": +1}, "k": 6.0},
        {"change": {"X": -1}, "k": 5.0},
        {"reactants": {"X": 1}, "change": {"X": -1, "Y": +1}, "k": 0.4},
        {"reactants": {"X": 2}, "change": {"X": -2}, "k": 0.2},
        {"reactants": {"Y": 1}, "change": {"Y": -1}, "k": 1.0},
    ])


def takes_two():
    """A first-order reaction that removes two of four species (more than the kernel stores states of)."""
    return wl._build("takes_two", ["X", "Y", "Z", "W"], [
        {"change": {"X": +1}, "k": 4.0},
        {"reactants": {"X": 1}, "change": {"X": -2, "Y": +1}, "k": 1.0},
        {"reactants": {"Y": 1, "X": 1}, "change": {"Y": -1, "Z": +1}, "k": 0.5},
        {"reactants": {"Z": 1}, "change": {"Z": -1, "W": +1}, "k": 1.0},
        {"reactants": {"W": 1, "Y": 1}, "change": {"W": -1}, "k": 0.7},
        {"reactants": {"Y": 1}, "change": {"Y": -1}, "k": 0.3},
    ])


def hill_loss():
    """A Hill law removes its own regulator: counts below zero, odd powers of them, falling sums."""
    return wl._build("hill_loss", ["X"], [
        {"change": {"X": +1}, "k": 3.0},
        {"change": {"X": -2}, "hill": ("repress", "X", 0.1, 6.0, 9.0, 3)},
        {"change": {"X": +1}, "hill": ("activate", "X", 0.4, 2.0, 7.0, 1)},
        {"reactants": {"X": 1}, "change": {"X": -1}, "k": 0.5},
    ])


# guards outside the careful path, and every batch careful
FLAGS = [(zero_order_loss, "true", "false"), (takes_two, "true", "false"), (hill_loss, "true", "true"),
         (wl.birth_death, "false", "false"), (wl.schlogl, "false", "false"), (wl.dimer_open, "false", "false"),
         (wl.telegraph, "false", "false"), (wl.repressilator, "false", "false")]


@pytest.mark.parametrize("make,guard,careful", FLAGS)
def test_generated_flags(tmp_path, make, guard, careful):
    spec = make()
    path = tmp_path / "k.hip"
    item = {"model": ssa.Model(spec), "x0": np.zeros(spec.n_species, np.int32), "n_traj": 1}
    ssa.ssa_dump_source([item], 1.0, [1.0], "FP64", path)
    src = path.read_text()
    assert re.search(r"needs_guard\(\) \{ return ([\w:]+);", src).group(1) == guard
    assert re.search(r"bool CAREFUL = (\w+);", src).group(1) == careful


@pytest.mark.gpu
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("make", [zero_order_loss, takes_two, hill_loss])
def test_launch_shapes_agree_below_zero(gpu, make, mode):
    spec = make()
    n, t_end, x0 = 700, 20.0, np.full(spec.n_species, 2, np.int32)
    ts = wl.snapshot_grid(t_end, 9)
    item = {"model": gpu.Model(spec), "x0": x0, "n_traj": n}
    first = None
    for launch in (dict(block_size=256), dict(block_size=64, grid_size=2), dict(block_size=512),
                   dict(block_size=512, grid_size=1), {}):
        print(f"[negative] {spec.name} mode={mode} launch={launch}", flush=True)
        run = gpu.ssa_ensemble_run([item], t_end, ts, 17, mode, max_events=20_000, **launch)
        assert run.info()["block_size"] == launch.get("block_size", 512)
        snap, st = run.snapshots(0), run.stats(0)
        if first is None:
            first = snap, st
            assert snap.min() < 0
            continue
        np.testing.assert_array_equal(snap, first[0])
        for k in st:
            np.testing.assert_array_equal(st[k], first[1][k])


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR", "UNI_BF16_SR_NORM"])
def test_two_workgroups_to_a_cu_below_zero(gpu, mode):
    spec = zero_order_loss()
    item = {"model": gpu.Model(spec), "x0": np.array([2, 0], np.int32), "n_traj": 64 * 600}
    out = []
    for launch in (dict(block_size=512, grid_size=150), dict(block_size=256)):
        print(f"[negative] two to a CU {mode} {launch}", flush=True)
        run = gpu.ssa_ensemble_run([item], 3.0, [1.0, 3.0], 5, mode, max_events=20_000, **launch)
        out.append((run.snapshots(0), run.stats(0)))
    np.testing.assert_array_equal(out[0][0], out[1][0])
    for k in out[0][1]:
        np.testing.assert_array_equal(out[0][1][k], out[1][1][k])
