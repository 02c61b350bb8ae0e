"""Creating sparse handles where memory runs out or a wait reports an error: on the CPU, with the HIP runtime's calls answered by a library
(hip_on_host.cpp) that a child process loads before the product's, whose kernels then do not run."""
import os
import subprocess
import sys

import pytest

from paper_2008_03433_amd import binding

HERE = os.path.dirname(os.path.abspath(__file__))

CHILD = r'''
import ctypes, sys
import numpy as np
C = ctypes
hip = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
lib = C.CDLL(sys.argv[2])
for f in ("live", "peak", "pinned_live", "pinned_peak"):
    getattr(hip, "host_hip_" + f).restype = C.c_size_t
hip.host_hip_reset.argtypes = [C.c_size_t]
hip.host_hip_answer.argtypes = [C.c_size_t, C.c_void_p]
lib.tron_last_error.restype = C.c_char_p
lib.tron_tuning_set.argtypes = [C.c_char_p, C.c_int64]
lib.tron_dataset_create_csr.argtypes = [C.c_int64, C.c_int64] + [C.c_void_p] * 4 + [C.c_int, C.c_void_p, C.POINTER(C.c_void_p)]
lib.tron_dataset_destroy.argtypes = [C.c_void_p]
lib.tron_dataset_destroy.restype = None
UNLIMITED = C.c_size_t(-1).value

def knob(name, value):
    assert lib.tron_tuning_set(name.encode(), value) == 0, lib.tron_last_error()

def problem(n, d, counts, rng):
    rowptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(counts, out=rowptr[1:])
    col = np.concatenate([np.sort(rng.choice(d, m, replace=False)) for m in counts if m]).astype(np.int32)
    val, y = rng.standard_normal(len(col)), np.where(rng.random(n) < 0.5, 1.0, -1.0)
    starts = np.zeros(d + 1, dtype=np.int64)
    np.cumsum(np.bincount(col, minlength=d), out=starts[1:])
    hip.host_hip_answer(starts.nbytes, starts.ctypes.data)   # what the sort on the device would give
    return rowptr, col, val, y

def create(n, d, arrays):
    """(status, handle)"""
    h = C.c_void_p()
    rc = lib.tron_dataset_create_csr(n, d, *[a.ctypes.data for a in arrays], 0, None, C.byref(h))
    return rc, h

rng = np.random.default_rng(5)
'''


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "libhip_on_host.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "hip_on_host.cpp")], check=True)
    return out


def run(runtime, body):
    r = subprocess.run([sys.executable, "-c", CHILD + body, runtime, binding.lib_path()], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("segmented", [0, 1])
def test_the_layouts_fit_but_not_beside_the_work_space_of_their_building(runtime, segmented):
    """Whichever allocation beyond what the host's way needs is refused, the handle is created, that way."""
    run(runtime, f"segmented = {segmented}" + r'''
n, d = 3000, 4000
arrays = problem(n, d, rng.integers(0, 60, n), rng)
knob("csr_segmented", segmented)
need = {}
for way in (0, 1):
    knob("csr_device_build", way)
    hip.host_hip_reset(UNLIMITED)
    rc, h = create(n, d, arrays)
    assert rc == 0, lib.tron_last_error()
    need[way] = hip.host_hip_peak()
    held = hip.host_hip_live()
    if way == 0: expected = held
    assert held == expected
    lib.tron_dataset_destroy(h)
    assert hip.host_hip_live() == hip.host_hip_pinned_live() == 0
assert need[1] > 1.5 * need[0]
refused = 0
for limit in range(need[0], need[1] + 1, (need[1] - need[0]) // 200):
    hip.host_hip_reset(limit)
    rc, h = create(n, d, arrays)
    assert rc == 0, (limit, lib.tron_last_error())
    assert hip.host_hip_live() == expected
    refused += hip.host_hip_refused()
    lib.tron_dataset_destroy(h)
    assert hip.host_hip_live() == hip.host_hip_pinned_live() == 0
assert refused > 100
hip.host_hip_reset(need[0] - 1)   # and what does not fit either way is an error, with nothing left behind
rc, h = create(n, d, arrays)
assert rc == -2 and not h.value and hip.host_hip_live() == 0, (rc, lib.tron_last_error())
''')


def test_an_error_of_the_last_wait_is_reported(runtime):
    run(runtime, r'''
n, d = 3000, 4000
arrays = problem(n, d, rng.integers(0, 60, n), rng)
knob("csr_device_build", 1)
hip.host_hip_reset(UNLIMITED)
hip.host_hip_fail_waits_from(1 << 30)   # count them
rc, h = create(n, d, arrays)
assert rc == 0
waits = hip.host_hip_syncs()
lib.tron_dataset_destroy(h)
for first in range(waits):
    hip.host_hip_reset(UNLIMITED)
    hip.host_hip_fail_waits_from(first)
    rc, h = create(n, d, arrays)
    assert rc < 0 and not h.value, (first, waits, rc)
    assert hip.host_hip_live() == 0
''')


def test_long_arrays_are_not_copied_through_pinned_memory(runtime):
    """A million rows with few entries: what is copied from a place of 4 MB or more goes the way of ordinary memory."""
    run(runtime, r'''
n, d = 1_000_000, 4000
counts = np.zeros(n, dtype=np.int64)
counts[rng.integers(0, n, 5000)] = 20
arrays = problem(n, d, counts, rng)
held = {}
for way in (0, 1):
    knob("csr_device_build", way)
    hip.host_hip_reset(UNLIMITED)
    rc, h = create(n, d, arrays)
    assert rc == 0, lib.tron_last_error()
    held[way] = hip.host_hip_live()
    lib.tron_dataset_destroy(h)
    assert hip.host_hip_pinned_peak() < 8 * n, (way, hip.host_hip_pinned_peak())
assert held[0] == held[1]
''')
