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
