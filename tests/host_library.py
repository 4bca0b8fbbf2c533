"""The library's host code on a HIP runtime of the host (fake_hip.cpp), for tests that
need no GPU: built with g++ into a temporary folder, its kernels compiled by a stand-in
that writes an empty object."""
import ctypes
import os
import subprocess

import numpy as np

from paper_2605_00479_amd import ssa
from paper_2605_00479_amd.csrc import build

HERE = os.path.dirname(os.path.abspath(__file__))


def load(folder, monkeypatch):
    """The library, bound as ssa.lib() for the test; .fake_* are the runtime's own entries."""
    build.embed_device_source()
    rocm = os.environ.get("ROCM_PATH") or "/opt/rocm"
    so = os.path.join(folder, "libssa_host.so")
    if not os.path.exists(so):
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-w", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                        "-D__align__(n)=", "-DHIP_SYMBOL(x)=x", "-I", os.path.join(rocm, "include"),
                        "-I", os.path.join(build.ROOT, "include"), "-I", build.BUILD,
                        os.path.join(build.HERE, "ssa_capi.cpp"), os.path.join(HERE, "fake_hip.cpp"), "-o", so, "-ldl"],
                       check=True)
        cc = os.path.join(folder, "cc")
        with open(cc, "w") as f:
            f.write('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\necho object > "$2"\n')
        os.chmod(cc, 0o755)
    monkeypatch.setenv("SSA_RP_CLANG", os.path.join(folder, "cc"))
    monkeypatch.setenv("SSA_RP_CACHE_DIR", os.path.join(folder, "cache"))
    real = ssa.LIB_PATH
    monkeypatch.setattr(ssa, "_lib", None)
    monkeypatch.setattr(ssa, "LIB_PATH", so)
    lib = ssa.lib()
    assert real != so
    lib.fake_log.restype = ctypes.c_char_p
    lib.fake_tables.restype = ctypes.c_void_p
    lib.fake_set.argtypes = [ctypes.c_char_p, ctypes.c_long]
    lib.fake_reset()
    return lib


def start(lib, items, mode, t_end=1.0, entry="run", outputs=None, **launch):
    """Queue a run; (return code, handle, log lines of the call)."""
    before = len(lib.fake_log())
    d, keep = ssa._desc(items, t_end, [t_end], 1, mode, max_events=10**9, outputs=outputs, **launch)
    h = ctypes.c_void_p()
    if entry == "run":
        rc = lib.ssa_ensemble_run(ctypes.byref(d), ctypes.byref(h))
    else:
        rc = lib.ssa_ensemble_run_noalloc(ctypes.byref(d))
    return rc, h, lib.fake_log()[before:].decode().splitlines()


def launched(log):
    """(kernel, workgroups, threads) of a log's simulation launches."""
    return [(w[1], int(w[2]), int(w[3])) for w in (line.split() for line in log)
            if w[0] == "launch" and w[1].startswith("ssa_kernel")]


def item(spec, n_traj, rates=None):
    it = {"model": ssa.Model(spec), "x0": np.full(spec.n_species, 3, np.int32), "n_traj": n_traj}
    if rates is not None:
        it["set_rates"] = rates
        it["traj_per_set"] = -(-n_traj // len(rates))
    return it
