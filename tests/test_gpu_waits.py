"""The clock wave's short divisions and the fp16 quotient return the IEEE quotient on the
ranges that the kernel uses them on (tests/gpu_wait_checks.hip includes the device template)."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libgpu_wait_checks.so")


@pytest.mark.gpu
def test_waiting_times_and_quotients_are_ieee():
    import torch  # one HIP runtime per process: torch's, loaded first
    assert torch.cuda.is_available()
    if not os.path.exists(LIB):
        pytest.fail("tests/libgpu_wait_checks.so is not built (run __graft_entry__.build())")
    lib = ctypes.CDLL(LIB)
    lib.gpu_check_waits.argtypes = [ctypes.c_uint, ctypes.POINTER(ctypes.c_ulonglong)]
    out = (ctypes.c_ulonglong * 7)()
    print("[gpu-facts] waiting times: 2^20 pairs an exponent; every pair of fp16 values", flush=True)
    assert lib.gpu_check_waits(1 << 20, out) == 0
    assert list(out) == [0] * 7, f"binary64 / bfloat16 / FP32 waits, fp16 quotients: {list(out)}"
