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
    P = ctypes.c_void_p
    L.acdc_emu_mp_quartets.argtypes = [ctypes.c_int, ctypes.c_int, P, P]
    L.acdc_emu_mp_sets.argtypes = [ctypes.c_int, ctypes.c_int, P, P, P]
    L.acdc_emu_mp_spectrum.argtypes = [ctypes.c_int, ctypes.c_int, P, P, P]
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


@pytest.mark.parametrize("N,ew", ROWS)
def test_column_sets(emu, N, ew):
    # every element lies in one set and has a place of its own in its LDS
    # image; the elements of a set's local positions are the set's, and on
    # the place that the column launches read for that position
    set_, place, elem = (np.full(N, -1, np.int64) for _ in range(3))
    C = emu.acdc_emu_mp_sets(N, ew, set_.ctypes.data, place.ctypes.data, elem.ctypes.data)
    R1 = spectrum(emu, N, ew)[2][0]
    assert np.array_equal(np.sort(elem), np.arange(N))
    assert np.array_equal(set_[elem], np.arange(N) // C)
    whole = 16384 // ew
    assert place.min() >= 0 and place.max() < whole
    assert np.unique(set_ * whole + place).size == N
    # local position: float4 chunk (real) or element js w + col; place js W + col
    unit, js_count = (4, 2 * (R1 // 2)) if ew == 1 else (1, R1)
    w, W = C // unit // js_count, whole // unit // js_count
    local = np.arange(N) % C
    chunk, low = local // unit, local % unit
    assert np.array_equal(place[elem], ((chunk // w) * W + chunk % w) * unit + low)


def spectrum(emu, N, ew):
    M = N * ew // 2
    spec, pairs, geo = np.empty(M, np.int64), np.empty(2 * M, np.int32), np.empty(3, np.int32)
    emu.acdc_emu_mp_spectrum(N, ew, spec.ctypes.data, pairs.ctypes.data, geo.ctypes.data)
    R1, R2, L = (int(v) for v in geo)
    return spec, pairs[: R1 * R2].reshape(-1, 2), (R1, R2, L)


@pytest.mark.parametrize("N,ew", ROWS)
def test_spectrum_order(emu, N, ew):
    # the passes of the column, second-level and segment launches (radix R1
    # over the row, R2 over its parts, L-point FFTs) leave spectrum value
    # spec[q] at place q
    spec, _, (R1, R2, L) = spectrum(emu, N, ew)
    M = N * ew // 2
    assert R1 * R2 * L == M
    rng = np.random.default_rng(N)
    x = rng.standard_normal(M) + 1j * rng.standard_normal(M)

    def dif(v, R):                       # radix-R pass over each row of v
        S = v.shape[1]
        n = np.arange(S // R)
        y = np.fft.fft(v.reshape(-1, R, S // R), axis=1)
        y *= np.exp(-2j * np.pi * np.outer(np.arange(R), n) / S)
        return y.reshape(-1, S // R)

    z = np.fft.fft(dif(dif(x[None], R1), R2), axis=1).reshape(-1)
    want = np.fft.fft(x)[spec]
    assert np.array_equal(np.sort(spec), np.arange(M))
    assert np.abs(z - want).max() < 1e-9 * np.abs(want).max()


@pytest.mark.parametrize("N", REAL)
def test_segment_pairs(emu, N):
    # the pairs take every segment once, and hold Z[k] with Z[M-k]: the
    # partner of segment A's k2 is segment B's L-1-k2; pair 0's segments hold
    # their own, at L-k2 and at L-1-k2.  The quartets of a pair are theirs.
    spec, pairs, (R1, R2, L) = spectrum(emu, N, 1)
    M, n = N // 2, N // 4
    assert np.array_equal(np.sort(pairs.reshape(-1)), np.arange(R1 * R2))
    seg = spec.reshape(R1 * R2, L)
    quartet, back = np.empty(n, np.int64), np.empty(n, np.int64)
    emu.acdc_emu_mp_quartets(N, 1, quartet.ctypes.data, back.ctypes.data)
    quartet = quartet.reshape(-1, L)
    for p, (a, b) in enumerate(pairs):
        if p == 0:
            assert a == 0
            assert np.array_equal(seg[a][1:] + seg[a][:0:-1], np.full(L - 1, M))
            assert np.array_equal(seg[b] + seg[b][::-1], np.full(L, M))
            assert np.array_equal(quartet[0], np.concatenate([seg[a][: L // 2], seg[b][: L // 2]]))
        else:
            assert np.array_equal(seg[a] + seg[b][::-1], np.full(L, M))
            assert np.array_equal(quartet[p], np.minimum(seg[a], M - seg[a]))


@pytest.mark.parametrize("N", REAL)
def test_quartet_places(emu, N):
    # every quartet has one place, and the map from quartets to places is
    # the inverse of the one from places to quartets
    n = N // 4
    out, back = np.full(n, -1, np.int64), np.full(n, -1, np.int64)
    emu.acdc_emu_mp_quartets(N, 1, out.ctypes.data, back.ctypes.data)
    assert np.array_equal(np.sort(out), np.arange(n))
    assert np.array_equal(out[back], np.arange(n))
