"""Launch sizes and index algebra of the multi-pass rows (no GPU): the headers' own code, built
for the host with the CPU emulation."""

import ctypes
import os
import shutil
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.join(os.path.dirname(__file__), "emu"))

REAL = [1 << i for i in range(8, 23)]
COMPLEX = [1 << i for i in range(8, 22)]
ROWS = [(N, 1) for N in REAL] + [(N, 2) for N in COMPLEX]      # (elements, floats per element)


@pytest.fixture(scope="module")
def emu():
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not available")
    import build_emu
    L = ctypes.CDLL(build_emu.build())
    L.acdc_emu_mp_col_grid.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    L.acdc_emu_mp_quartets.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p]
    return L


def col_grid(emu, B, N, ew, sums):
    out = (ctypes.c_longlong * 4)()
    emu.acdc_emu_mp_col_grid(B, N, ew, sums, out)
    return tuple(out)


@pytest.mark.parametrize("N,ew", ROWS)
def test_column_launches_fit_any_batch(emu, N, ew):
    # HIP refuses launches of 2^32 threads and more; the forward's column
    # launches must stay below it at every accepted batch (2^40 elements),
    # the backward's (blocks of 16 rows) at every batch of 2^36 floats, the
    # most that fits the device's memory
    for B in (1, 2, 511, 65535, 65536, 65537, 1 << 23, (1 << 23) + 1, (1 << 40) // N):
        if B > (1 << 40) // N:
            continue
        rb, threads, groups, rw = col_grid(emu, B, N, ew, 0)
        sets = max(1, N * ew // 16384)
        assert rb >= 1 and groups == -(-B // (rb * rw)) * sets
        assert groups * threads < 1 << 32
        # rows side by side: what fits a set of 16384 floats, and only while
        # every CU has two workgroups
        assert 1 <= rw <= max(1, 16384 // (N * ew)) and (rw == 1 or B // rw >= 512)
        if -(-B // rw) * sets <= 65536:
            assert rb == 1                          # a workgroup of its own for every rw rows and set
        if B <= (1 << 36) // (N * ew):
            rb, threads, groups, rw = col_grid(emu, B, N, ew, 1)
            assert rw == 1 and 1 <= rb <= 16 and groups == -(-B // rb) * sets
            assert groups * threads < 1 << 32


@pytest.mark.parametrize("N", REAL)
def test_quartet_places(emu, N):
    # every quartet has one place, and the map from quartets to places is
    # the inverse of the one from places to quartets
    n = N // 4
    out, back = np.full(n, -1, np.int64), np.full(n, -1, np.int64)
    emu.acdc_emu_mp_quartets(N, 1, out.ctypes.data, back.ctypes.data)
    assert np.array_equal(np.sort(out), np.arange(n))
    assert np.array_equal(out[back], np.arange(n))
