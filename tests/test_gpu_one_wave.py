"""The one-wave kernel (block sizes of 64 to 256: a wave runs 64 trajectories, forming its
own draws) against the oracle: what the default launch, which is the pipelined kernel up to
some size, does not run. Every case asserts which kernel it ran."""
import numpy as np
import pytest

from paper_2605_00479_amd import workloads as wl
from test_gpu_parity import (ORACLE_THREADS, assert_parity, gpu, largest_network, low_count_network,   # noqa: F401
                             run_both, run_records)

pytestmark = pytest.mark.gpu

WAVE, WORKGROUP = dict(block_size=64), dict(block_size=256)
EACH = pytest.mark.parametrize("launch", [WAVE, WORKGROUP], ids=["64", "256"])


def one_wave(run, launch):
    assert run.info()["block_size"] == launch["block_size"] <= 256


@EACH
@pytest.mark.parametrize("mode", ["FP64", "FP32", "MIX_F16_SR", "MIX_F16_RTN", "UNI_F16_SR", "UNI_BF16_SR_NORM"])
def test_zero_guards(gpu, orc, mode, launch):
    run, _, _ = run_both(gpu, orc, low_count_network(), np.array([0, 0], np.int32), 64 * 40, 20.0,
                         wl.snapshot_grid(20.0, 21), mode, seed=5, **launch)
    one_wave(run, launch)


@EACH
@pytest.mark.parametrize("mode,levels", [("MIX_F16_SR", (1500.0, 2100.0, 2600.0)),
                                         ("UNI_F16_SR", (1500.0, 2100.0, 2600.0)),
                                         ("MIX_BF16_SR", (180.0, 250.0, 330.0))])
def test_count_conversions_of_parameter_sets(gpu, orc, mode, levels, launch):
    # sets below, at and above the exact range of counts, in one wave
    rates = np.array([[kb, 1.0] for kb in levels], np.float64)
    run, _, _ = run_both(gpu, orc, wl.birth_death(levels[1], 1.0), np.array([int(levels[1])], np.int32), 3 * 70, 1.5,
                         wl.snapshot_grid(1.5, 7), mode, seed=11, set_rate=rates, traj_per_set=70,
                         max_events=200_000, **launch)
    one_wave(run, launch)


@EACH
@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR"])
def test_a_table_of_sets(gpu, orc, mode, launch):
    run, _, _ = run_both(gpu, orc, wl.dimer_open(), np.array([0, 0], np.int32), 48 * 40, 10.0, wl.snapshot_grid(10.0, 11),
                         mode, seed=1, set_rate=wl.dimer_sweep_rates(48), traj_per_set=40, max_events=3_000_000, **launch)
    one_wave(run, launch)


@EACH
@pytest.mark.parametrize("mode", ["FP64", "MIX_BF16_SR", "UNI_F16_SR"])
def test_hill_laws(gpu, orc, mode, launch):
    run, _, _ = run_both(gpu, orc, wl.repressilator(), np.array([0, 0, 0, 0, 0, 20], np.int32), 600, 60.0,
                         wl.snapshot_grid(60.0, 61), mode, seed=3, max_events=10_000_000, **launch)
    one_wave(run, launch)


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR", "UNI_F16_SR"])
def test_largest_network(gpu, orc, mode):
    run, _, _ = run_both(gpu, orc, largest_network(), np.full(32, 3, np.int32), 64 * 12, 2.0, wl.snapshot_grid(2.0, 5),
                         mode, seed=9, **WORKGROUP)
    one_wave(run, WORKGROUP)


@pytest.mark.parametrize("mode", ["MIX_F16_SR", "UNI_BF16_SR"])
def test_large_networks_keep_two_waves_a_simd(gpu, orc, mode):
    run, _, _ = run_both(gpu, orc, largest_network(), np.full(32, 3, np.int32), 300, 1.0, [0.5, 1.0], mode, seed=2,
                         **WORKGROUP)
    one_wave(run, WORKGROUP)
    assert run.info()["vgprs"] <= 256


def test_the_default_for_a_large_ensemble_of_a_large_network(gpu, orc):
    # more workgroups of 64 trajectories than CUs, and 64 reactions
    n = 64 * 300
    run, _, _ = run_both(gpu, orc, largest_network(), np.full(32, 3, np.int32), n, 0.5, [0.5], "FP64", seed=4,
                         indices=np.arange(0, n, 37))
    assert run.info()["block_size"] == 256


@EACH
@pytest.mark.parametrize("mode,chunks", [("FP64", 1), ("MIX_F16_SR", 3), ("UNI_BF16_SR_NORM", 2)])
def test_event_records(gpu, orc, mode, chunks, launch):
    # some trajectories have more recorded firings than the record holds
    rec, ref = run_records(gpu, orc, wl.telegraph(0.05, 0.05, 20.0, 1.0), np.array([1, 0, 0], np.int32), 300, 120.0,
                           wl.snapshot_grid(120.0, 9), mode, 0b11, 6, seed=4, n_chunks=chunks, **launch)
    assert (ref["rec_n"] > 6).any() and (ref["rec_n"] < 6).any()


@EACH
@pytest.mark.parametrize("mode,cap", [("FP64", 1), ("MIX_F16_SR", 33), ("UNI_BF16_RTN", 300)])
def test_event_caps(gpu, orc, mode, cap, launch):
    run, _, st = run_both(gpu, orc, wl.birth_death(), np.array([3], np.int32), 300, 1e4, [1e4], mode, seed=cap,
                          max_events=cap, grid_size=1, **launch)
    one_wave(run, launch)
    assert (st["n_events"] == cap).all()


@EACH
@pytest.mark.parametrize("mode,chunks", [("FP64", 1), ("MIX_BF16_SR", 1), ("MIX_F16_SR", 3)])
def test_several_networks(gpu, orc, mode, chunks, launch):
    W = wl.config_heterogeneous(n_traj_total=5 * 150)
    t_end, ts = 15.0, wl.snapshot_grid(15.0, 16)
    print(f"[gpu-parity] one wave, heterogeneous mode={mode} chunks={chunks} {launch}", flush=True)
    run = gpu.ssa_ensemble_run(gpu.items_from_workload(W, {}), t_end, ts, 1, mode, traj_id_base=1000,
                               max_events=W.max_events, n_chunks=chunks, **launch)
    one_wave(run, launch)
    base = 1000
    for i, it in enumerate(W.items):
        ref = orc.simulate(it.model, mode, it.x0, t_end, ts, 1, n_traj=it.n_traj, traj_id_base=base,
                           max_events=W.max_events, threads=ORACLE_THREADS)
        assert_parity(ref, run.snapshots(i), run.stats(i), mode, it.model.name)
        base += it.n_traj


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR"])
@pytest.mark.parametrize("grid,chunks,window,reorder", [(1, 1, 0, 0), (2, 2, 10, 0), (2, 3, 0, -1), (8, 4, 1, 0)])
def test_wave_major_claims(gpu, orc, mode, grid, chunks, window, reorder):
    # the first claims are static: fewer and more lanes than trajectories, with and without
    # the order of a window before
    W = wl.config_schlogl()
    it = W.items[0]
    run, _, _ = run_both(gpu, orc, it.model, it.x0, 1500, 2.0, wl.snapshot_grid(2.0, 21), mode, seed=W.seed,
                         max_events=W.max_events, grid_size=grid, n_chunks=chunks, first_window=window, reorder=reorder,
                         placement=gpu.PLACE_EXPLICIT | gpu.PLACE_WAVE_MAJOR, **WORKGROUP)
    one_wave(run, WORKGROUP)
    assert run.info()["placement"] == gpu.PLACE_EXPLICIT | gpu.PLACE_WAVE_MAJOR


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR"])
def test_captured_windows(gpu, orc, mode):
    W = wl.config_schlogl()
    it = W.items[0]
    for chunks, window, reorder in ((25, 0, 0), (17, 3, -1)):
        run, _, _ = run_both(gpu, orc, it.model, it.x0, 500, 2.0, wl.snapshot_grid(2.0, 51), mode, seed=6,
                             max_events=W.max_events, n_chunks=chunks, first_window=window, reorder=reorder, **WAVE)
        one_wave(run, WAVE)
        assert run.info()["graph"] == 1
