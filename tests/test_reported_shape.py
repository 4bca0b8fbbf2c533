"""The launch shape that ssa_run_info reports, given back as a request, launches the same."""
import ctypes

import pytest

from paper_2605_00479_amd import ssa, workloads as wl
from host_library import item, launched, load, start

CUS = 256


@pytest.fixture(scope="module")
def folder(tmp_path_factory):
    return str(tmp_path_factory.mktemp("host"))


@pytest.mark.parametrize("mode", ["FP64", "MIX_F16_SR"])
@pytest.mark.parametrize("launch", [{}, dict(block_size=512), dict(block_size=512, grid_size=3),
                                    dict(block_size=512, grid_size=64), dict(block_size=512, grid_size=300),
                                    dict(block_size=256), dict(block_size=64, grid_size=7)])
@pytest.mark.parametrize("wgs", [1, 5, 255, 256, 257, 313, 511, 512, 600, 5000])
def test_a_reported_shape_repeats_itself(folder, monkeypatch, mode, launch, wgs):
    lib = load(folder, monkeypatch)
    its = [item(wl.birth_death(), 64 * wgs - 7)]

    def shape(**kw):
        rc, h, log = start(lib, its, mode, **kw)
        assert rc == 0
        info = ssa.ssa_run_info()
        assert lib.ssa_run_info_get(h, ctypes.byref(info)) == 0
        lib.ssa_run_destroy(h)
        return launched(log), dict(block_size=info.block_size, grid_size=info.grid_size)

    first, reported = shape(**launch)
    assert shape(**reported) == (first, reported)
