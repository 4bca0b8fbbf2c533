"""The kernel and grid that a run is given, without a GPU (fake_hip.cpp): which of the
event loops, and one or two of its workgroups to a CU (256 CUs here)."""
import re

import numpy as np
import pytest

from paper_2605_00479_amd import ssa, workloads as wl
from host_library import item, launched, load, start

CUS = 256


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    return str(tmp_path_factory.mktemp("host"))


@pytest.fixture
def lib(folder, monkeypatch):
    return load(folder, monkeypatch)


def parts(reactions):
    """A network of so many reactions, births at 4 and losses."""
    n = reactions // 2
    sp = [f"X{i}" for i in range(n)]
    return wl._build("parts", sp, [r for s in sp for r in ({"change": {s: 1}, "k": 4.0},
                                                           {"reactants": {s: 1}, "change": {s: -1}, "k": 0.5})])


def shape(lib, its, mode, t_end=1e4, **launch):
    rc, h, log = start(lib, its, mode, t_end, **launch)
    assert rc == 0
    lib.ssa_run_destroy(h)
    (k,) = launched(log)
    return k


PL, PH, ONE = "ssa_kernel_pl", "ssa_kernel_ph", "ssa_kernel"


@pytest.mark.parametrize("reactions,mode,rounds,kernel", [
    # more than 16 reactions: no two workgroups to a CU
    (18, "FP64", 2, PL), (18, "FP64", 2.1, ONE), (24, "MIX_F16_SR", 1, PL), (24, "MIX_F16_SR", 1.1, ONE),
    (26, "FP64", 1, PL), (26, "FP64", 1.1, ONE), (64, "FP64", 1, PL), (64, "UNI_BF16_SR", 16, ONE),
    # 13 to 16: 16-bit modes and binary32 beyond two rounds; 5 to 12: beyond twelve
    (16, "FP64", 64, PH), (16, "MIX_F16_SR", 2, PH), (16, "MIX_F16_SR", 2.1, ONE), (14, "FP32", 8, ONE),
    (12, "MIX_F16_SR", 12, PH), (12, "MIX_F16_SR", 12.1, ONE), (12, "FP64", 100, PH), (6, "FP32", 13, ONE),
    (4, "MIX_F16_SR", 100, PH),
    (2, "FP64", 2, PL), (2, "FP64", 2.1, PH), (2, "MIX_F16_SR", 1, PL), (2, "MIX_F16_SR", 1.1, PH),
])
def test_default_kernel_by_reactions_and_rounds(lib, reactions, mode, rounds, kernel):
    if reactions > 16:
        lib.fake_set(b"ph_lds", 0)   # (its kernel is empty)
    wgs = int(rounds * CUS)
    name, grid, threads = shape(lib, [item(parts(reactions), 64 * wgs)], mode)
    assert name == kernel
    assert (grid, threads) == {PL: (min(wgs, CUS), 512), PH: (min(wgs, 2 * CUS), 512),
                               ONE: (min(-(-wgs // 4), 2 * CUS), 256)}[kernel]


def test_short_trajectories_that_outnumber_the_lanes_stay_pipelined(lib):
    for rounds, kernel in ((2, PH), (6, ONE), (9, PH)):
        assert shape(lib, [item(parts(16), 64 * rounds * CUS)], "MIX_F16_SR", t_end=2.0)[0] == kernel


def test_a_chosen_kernel_is_kept(lib):
    lib.fake_set(b"ph_lds", 0)
    its = [item(parts(32), 64 * 16 * CUS)]
    assert shape(lib, its, "FP64", block_size=512) == (PL, CUS, 512)
    assert shape(lib, its, "FP64", block_size=256) == (ONE, 2 * CUS, 256)
    assert shape(lib, its, "FP64", grid_size=64) == (PL, CUS, 512)      # 16,384 lanes asked for
    assert shape(lib, its, "FP64", grid_size=65) == (ONE, 65, 256)


def sweep(reactions, factors):
    spec = parts(reactions)
    return np.asarray(spec.rate)[None, :] * np.asarray(factors)[:, None]


@pytest.mark.parametrize("mode,factors,alone", [
    ("FP64", np.geomspace(0.01, 1.0, 64), 8),     # spread 4.4
    ("MIX_F16_SR", np.geomspace(0.01, 1.0, 64), 8),
    ("FP64", np.linspace(0.7, 1.3, 64), 4), ("MIX_F16_SR", np.linspace(0.7, 1.3, 64), 2),
    ("FP64", np.ones(9), 4), ("UNI_F16_SR", np.ones(9), 2),
])
def test_sweeps_have_cus_to_themselves_by_their_spread(lib, mode, factors, alone):
    for rounds, kernel in ((alone, PL), (alone + 0.1, PH)):
        n = 64 * int(rounds * CUS)
        assert shape(lib, [item(parts(4), n, sweep(4, factors))], mode)[0] == kernel


def test_sweeps_of_many_reactions(lib):
    lib.fake_set(b"ph_lds", 0)
    wide_range = np.geomspace(0.05, 1.0, 32)
    for reactions, mode, kernel in ((32, "FP64", PL), (34, "FP64", ONE), (64, "FP64", ONE), (32, "MIX_F16_SR", PL)):
        n = 64 * (CUS if reactions > 32 else 2 * CUS)
        assert shape(lib, [item(parts(reactions), n, sweep(reactions, wide_range))], mode)[0] == kernel
    # two registers a constant: also where the pipelined kernel is asked for
    assert shape(lib, [item(parts(64), 640, sweep(64, wide_range))], "FP64", block_size=512)[0] == ONE


def test_several_networks(lib):
    its = [item(parts(12), 64 * 4 * CUS), item(parts(2), 64 * 4 * CUS)]
    assert shape(lib, its, "MIX_BF16_SR")[0] == PL
    its = [item(parts(12), 64 * 40 * CUS), item(parts(2), 64 * CUS)]
    assert shape(lib, its, "MIX_BF16_SR")[0] == PH


@pytest.mark.parametrize("mode", ["FP64", "FP32", "UNI_BF16_SR"])
def test_kernels_are_launched_with_the_lds_they_are_built_for(lib, tmp_path, mode):
    # a ring of more batches than the launch has LDS for would be accessed out of range
    sizes = {}
    for wgs in (1, 4 * CUS):
        its = [item(wl.birth_death(), 64 * wgs)]
        rc, h, log = start(lib, its, mode)
        lib.ssa_run_destroy(h)
        sizes.update({line.split()[1]: int(line.split()[4]) for line in log if "ssa_kernel" in line})
    ssa.ssa_dump_source(its, 1.0, [1.0], mode, tmp_path / "k.hip", max_events=1)
    built = re.findall(r"pipe_lds\(bool half\) \{ return half \? (\d+) : (\d+);", (tmp_path / "k.hip").read_text())
    assert [(sizes[PH], sizes[PL])] == [tuple(map(int, b)) for b in built]
