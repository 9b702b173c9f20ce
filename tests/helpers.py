"""Shared test helpers: the parity metric and the ReLU-margin row filter."""

from __future__ import annotations

import numpy as np

# Max relative error per output (fp32, K <= 16) and for the complex variant.
TOL_REAL = 1e-4
TOL_COMPLEX = 2e-4
# ReLU decisions closer than DELTA * rms(row) to zero may legitimately differ
# between fp32 and fp64, and one flipped mask bit changes that row's gradient.
RELU_DELTA = 1e-5


# Rows per backward workgroup (one partial of the parameter gradients each) of
# the fused widths: the first while the batch fills at most one such workgroup
# on each of 256 CUs, the second beyond (checked against the headers' own rule
# in test_emulation.py).
BWD_ROWS_REAL = {8: (256, 256), 16: (256, 256), 32: (128, 128), 64: (64, 64), 128: (64, 64), 256: (16, 16),
                 512: (16, 16), 1024: (8, 8), 2048: (4, 4), 4096: (4, 8), 8192: (2, 4), 9216: (1, 2), 16384: (1, 2),
                 32768: (1, 1)}
BWD_ROWS_COMPLEX = {8: (256, 512), 16: (256, 512), 32: (128, 256), 64: (64, 128), 128: (32, 64), 256: (32, 64),
                    512: (16, 32), 1024: (8, 16), 2048: (4, 8), 4096: (2, 4), 8192: (1, 2), 16384: (1, 1)}
# The largest batch whose forward runs one wave on each SIMD of 256 CUs (its
# ALONE form), for the widths whose rows share a workgroup.
FWD_ALONE_MAX = {8: 65536, 16: 65536, 32: 32768, 64: 16384, 128: 16384, 256: 4096, 512: 4096, 1024: 2048,
                 2048: 1024, 4096: 1024}


def bwd_tiles(N: int, B: int, complex_: bool = False) -> int:
    few, full = (BWD_ROWS_COMPLEX if complex_ else BWD_ROWS_REAL)[N]
    rows = few if B <= 256 * few else full
    return -(-B // rows)


def rel_err(got, ref) -> float:
    """max_i |got_i - ref_i| / max(|ref_i|, rms(ref over the group)), groups =
    rows (last axis).  Handles complex arrays through their modulus."""
    got = np.asarray(got)
    ref = np.asarray(ref)
    assert got.shape == ref.shape, (got.shape, ref.shape)
    if ref.size == 0:
        return 0.0
    ref2 = ref.reshape(-1, ref.shape[-1]) if ref.ndim > 1 else ref.reshape(1, -1)
    got2 = got.reshape(ref2.shape)
    rms = np.sqrt(np.mean(np.abs(ref2) ** 2, axis=1, keepdims=True))
    den = np.maximum(np.abs(ref2), rms)
    den = np.where(den == 0, 1.0, den)
    err = np.abs(got2.astype(np.complex128 if np.iscomplexobj(ref2) else np.float64) - ref2) / den
    if not np.all(np.isfinite(err)):
        return float("inf")
    return float(err.max())


def relu_safe_rows(cache_v, K: int, delta: float = RELU_DELTA) -> np.ndarray:
    """Rows whose pre-ReLU values |v_k| stay above delta * rms(v_k row) for
    every layer k < K-1 (oracle forward cache)."""
    ok = None
    for k in range(K - 1):
        v = cache_v[k]
        rms = np.sqrt(np.mean(v * v, axis=1, keepdims=True))
        row_ok = np.all(np.abs(v) >= delta * rms, axis=1)
        ok = row_ok if ok is None else ok & row_ok
    if ok is None:
        ok = np.ones(cache_v[0].shape[0], dtype=bool)
    return ok
