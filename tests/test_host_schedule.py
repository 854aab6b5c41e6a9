"""Launch schedules of the operation lists, on the CPU: small operations share fused launches and chains, and every
operation still runs after everything it depends on (dependencies re-derived from the buffers in C++),
for small systems where everything is fused, large ones where little is, and with operations kept on their own
kernels."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import fsgen

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2004_03682_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("host") / "libschedcheck.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", out,
                    os.path.join(HERE, "host", "schedule_check.cpp"), os.path.join(CSRC, "plan_ccsd.cpp")], check=True)
    lib = ctypes.CDLL(out)
    lib.schedule_check.restype = ctypes.c_int
    return lib


SYSTEMS = [(2, 3, 1, 0), (8, 24, 1, 0), (6, 14, 4, 5), (9, 37, 5, 6), (13, 67, 3, 2), (20, 120, 8, 6)]


@pytest.mark.parametrize("real", [0, 1])
@pytest.mark.parametrize("keep_every", [0, 1, 3])
@pytest.mark.parametrize("spec", SYSTEMS)
def test_schedules_respect_every_dependency(lib, spec, keep_every, real):
    nocc, nvirt, nirrep, nact = spec
    s = fsgen.make_system(nocc, nvirt, nirrep, 0.05, 11, nact=nact)
    irr = np.ascontiguousarray(s.irrep, dtype=np.int32)
    eps = np.ascontiguousarray(s.eps, dtype=np.float64)
    act = np.ascontiguousarray(s.active, dtype=np.int32)
    steps, fused, count = ((ctypes.c_int * 5)() for _ in range(3))
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    bad = lib.schedule_check(nocc, nvirt, nirrep, ptr(irr), ptr(eps), len(act), ptr(act), keep_every, real, steps,
                                 fused, count)
    assert bad == 0
    print(list(count), list(steps), list(fused))
    if keep_every == 1:
        assert list(steps) == list(count) and not any(fused)
    if keep_every == 0 and nvirt <= 37:
        # a small system's residual runs in fused launches only, a fraction of its operations
        assert steps[0] == fused[0] <= count[0] // 3


@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 17, 40])
def test_long_chains_are_cut_at_the_kernels_limit(n, tmp_path):
    """One limit for the planner and the kernel (the build asserts that the kernel has room for it)."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path / "libchaincheck.so")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, "-o", out,
                    os.path.join(HERE, "host", "chain_check.cpp")], check=True)
    limit = ctypes.c_int()
    chains = ctypes.CDLL(out).chain_check(n, ctypes.byref(limit))
    assert limit.value == 8 and chains == (n + limit.value - 1) // limit.value
