"""ssa_ensemble_run_noalloc while its stream captures a graph: the rates, initial counts and
snapshot times of the call go into the graph, not the address of host memory that is
freed when the call returns. On the CPU the tables that reach the device are compared
with an ordinary call's (fake_hip.cpp); on the GPU the graph is replayed after the
inputs are gone, and every replay is compared with an ordinary run."""
import ctypes
import gc

import numpy as np
import pytest

from paper_2605_00479_amd import ssa, workloads as wl
from host_library import item, load, start


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    return str(tmp_path_factory.mktemp("host"))


class Outputs:
    """Stands in for a device tensor of the caller."""

    def __init__(self, n):
        self.a = np.zeros(n, np.uint8)

    def data_ptr(self):
        return self.a.ctypes.data

    def numel(self):
        return self.a.size


@pytest.mark.parametrize("sets", [1, 3, 200])
def test_captured_tables_are_the_calls_own(folder, monkeypatch, sets):
    lib = load(folder, monkeypatch)
    rates = np.random.default_rng(1).uniform(0.1, 2.0, (sets, 4))
    its = [item(wl.telegraph(), 600, rates)]
    out = [tuple(Outputs(600 * 16) for _ in range(4))]
    rc, h, _ = start(lib, its, "FP64")
    assert rc == 0
    lib.ssa_run_destroy(h)
    lib.fake_tables()
    seen = []
    for capturing in (0, 1):
        lib.fake_set(b"capturing", capturing)
        rc, _, log = start(lib, its, "FP64", entry="noalloc", outputs=out)
        assert rc == 0
        size = 256 * 4 + 8 * 4 * sets   # times, Hill constants and counts lie in blocks of 256 bytes
        base = lib.fake_tables()
        assert base, "nothing has reached the device"
        seen.append(ctypes.string_at(base, size))
        ctypes.memset(base, 0, size)
        copies = [line for line in log if line.startswith("mem")]
        uploads = [line for line in log if line.startswith("launch ssa_upload")]
        assert (len(copies), len(uploads) > 0) == ((1, False), (0, True))[capturing]
    assert seen[0] == seen[1] and any(seen[0])


def test_the_allocating_entry_refuses_a_capture(folder, monkeypatch):
    lib = load(folder, monkeypatch)
    lib.fake_set(b"capturing", 1)
    rc, _, log = start(lib, [item(wl.telegraph(), 600)], "FP64")
    assert rc == ssa.SSA_E_DEVICE and not [line for line in log if line.startswith(("mem", "launch"))]


@pytest.mark.gpu
@pytest.mark.parametrize("sets,chunks,mode", [(1, 1, "FP64"), (150, 1, "MIX_F16_SR"), (3, 4, "FP64")])
def test_replays_of_a_captured_call(sets, chunks, mode):
    import torch
    assert torch.cuda.is_available()
    spec, n, ts = wl.telegraph(), 1200, wl.snapshot_grid(20.0, 9)
    rng = np.random.default_rng(2)

    def make():
        # inputs of this call alone
        it = {"model": ssa.Model(spec), "x0": np.array([1, 0, 0], np.int32), "n_traj": n}
        if sets > 1:
            it["set_rates"] = np.asarray(spec.rate) * np.random.default_rng(7).uniform(0.5, 1.5, (sets, 4))
            it["traj_per_set"] = -(-n // sets)
        return [it]

    def empty():
        return [(torch.full((9, 3, n), -7, dtype=torch.int32, device="cuda"),
                 torch.zeros(n, dtype=torch.int64, device="cuda"),
                 torch.zeros(n, dtype=torch.float64, device="cuda"),
                 torch.zeros(n, dtype=torch.uint8, device="cuda"))]

    print(f"[noalloc-capture] sets={sets} chunks={chunks} {mode}", flush=True)
    kw = dict(max_events=100_000, n_chunks=chunks)
    ref = ssa.ssa_ensemble_run(make(), 20.0, ts, 5, mode, **kw)
    snap, st = ref.snapshots(0), ref.stats(0)
    ssa.ssa_ensemble_run_noalloc(make(), 20.0, ts, 5, mode, empty(), **kw)   # looks the scratch array up
    torch.cuda.synchronize()
    out, graph = empty(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        ssa.ssa_ensemble_run_noalloc(make(), 20.0, ts, 5, mode, out, **kw)
    gc.collect()
    junk = [np.full(rng.integers(100, 40_000), 3.5) for _ in range(200)]   # over what the call has freed
    for replay in range(4):
        for t in out[0]:
            t.fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out[0][0].cpu().numpy(), snap, err_msg=f"replay {replay}")
        np.testing.assert_array_equal(out[0][1].cpu().numpy().astype(np.uint64), st["n_events"])
        np.testing.assert_array_equal(out[0][2].cpu().numpy(), st["t_last"])
        np.testing.assert_array_equal(out[0][3].cpu().numpy(), st["status"])
        other = ssa.ssa_ensemble_run(make(), 5.0, [5.0], replay, mode, max_events=100_000)   # eager work between
        other.wait()
    assert len(junk) == 200
