"""The tables of a run on their way to the device: their block goes back to the cache only
once the stream has passed the copy, also where the run is refused after it, and a call
whose tables are large returns while earlier work on its stream still runs."""
import numpy as np
import pytest

from paper_2605_00479_amd import ssa, workloads as wl
from host_library import item, load, start


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    return str(tmp_path_factory.mktemp("host"))


def test_a_refused_run_waits_for_its_copy(folder, monkeypatch):
    lib = load(folder, monkeypatch)
    lib.fake_set(b"waves_per_cu", 0)   # no workgroup of the kernel fits a CU
    rc, _, log = start(lib, [item(wl.birth_death(), 100)], "FP64", block_size=256)
    assert rc == ssa.SSA_E_UNSUPPORTED
    calls = [line.split()[0] for line in log]
    assert "memcpy_async" in calls and "launch" not in calls
    assert "stream_synchronize" in calls[calls.index("memcpy_async"):]


def big_sweep():
    """6.4 MB of rates (200,000 sets of four)."""
    spec = wl.schlogl()
    return [item(spec, 200_000, np.asarray(spec.rate) * np.full((200_000, 1), 1e-6))]


def test_large_tables_do_not_queue_behind_the_stream(folder, monkeypatch):
    # an asynchronous copy of that size from pageable memory returns only once the stream's
    # earlier work has ended
    lib = load(folder, monkeypatch)
    spec = wl.schlogl()
    for its, call in (([item(spec, 75_000, np.asarray(spec.rate) * np.ones((20_000, 1)))], "memcpy_async"),
                      (big_sweep(), "memcpy")):
        rc, h, log = start(lib, its, "FP64")
        assert rc == 0
        lib.ssa_run_destroy(h)
        assert [line.split()[0] for line in log if line.startswith("memcpy")] == [call]


@pytest.mark.gpu
def test_a_call_returns_while_earlier_work_runs():
    import torch
    assert torch.cuda.is_available()
    W = wl.config_schlogl()
    it = W.items[0]
    model = ssa.Model(it.model)
    busy = [{"model": model, "x0": it.x0, "n_traj": 5000}]
    sweep = big_sweep()
    with torch.cuda.stream(torch.cuda.Stream()):
        for items, t in ((busy, 0.1), (sweep, 0.01)):   # kernels loaded, blocks in the cache
            ssa.ssa_ensemble_run(items, t, [t], 1, "FP64", max_events=10**8).wait()
        first = ssa.ssa_ensemble_run(busy, 400.0, [400.0], 1, "FP64", max_events=10**8)   # 0.3 s
        done = torch.cuda.Event()
        done.record()
        second = ssa.ssa_ensemble_run(sweep, 0.01, [0.01], 1, "FP64", max_events=10**8)
        early = not done.query()
        first.wait()
        second.wait()
        assert early
