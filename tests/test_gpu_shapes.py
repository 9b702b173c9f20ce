"""GPU parity at the shapes where a launch or sum rule changes its split.

Each case runs through the same comparison with the fp64 oracle as the other
GPU parity tests (every element, same tolerance)."""

import numpy as np
import pytest

from oracle import acdc_oracle as O
from paper_1511_05946_amd.workloads import FLAG_BIAS, FLAG_MULTIPASS, make_bias, make_inputs
from tests.helpers import FWD_ALONE_MAX, TOL_REAL, rel_err
from tests.test_gpu_parity import acdc, host, run_case  # noqa: F401

pytestmark = pytest.mark.gpu

P, R, CX, MP = O.FLAG_PERM, O.FLAG_RELU, O.FLAG_COMPLEX, FLAG_MULTIPASS


# Narrow rows: one tile holds 256 (N = 8, 16) down to 16 rows (N = 512; up to
# 512 complex ones), and the image sums split them into phases.  A whole tile
# and one row of the next, and a single row.
@pytest.mark.parametrize("N,B,flags", [(8, 257, P | R | FLAG_BIAS), (16, 256, P), (32, 129, P | R), (64, 1, P),
                                       (64, 129, P | R | FLAG_BIAS), (128, 65, P), (256, 65, P | R),
                                       (512, 17, P | R | FLAG_BIAS), (8, 513, CX | P), (32, 257, CX | P),
                                       (64, 129, CX | P), (256, 65, CX | P)])
def test_narrow_tile_sums(acdc, N, B, flags):  # noqa: F811
    run_case(acdc, N, 3, B, flags, seed=N + B)


# Backward workgroups of half the rows while those leave every CU at most one
# workgroup (256 of them): the last such batch and the first beyond it.
@pytest.mark.parametrize("N,few,flags", [(4096, 4, P | R | FLAG_BIAS), (8192, 2, P), (9216, 1, P), (16384, 1, P | FLAG_BIAS),
                                         (64, 64, CX | P), (1024, 8, CX | P), (4096, 2, CX)])
def test_backward_rows_rule(acdc, N, few, flags):  # noqa: F811
    for B in (256 * few, 256 * few + 1):
        run_case(acdc, N, 2 if flags & R else 1, B, flags, seed=N + B)


# Forward workgroups: one wave a SIMD with loads ahead (ALONE) up to a batch
# per width, whole workgroups beyond, and a persistent loop over tiles where
# they are more than the device holds.  The last batch of the first form, the
# first of the second, and one of several tiles a workgroup.  Rows are
# independent, so copies of a few rows (checked against the oracle) give those
# rows' results bit for bit in either form; the parameter gradients are the
# oracle's with each row's gradient times its copies.
@pytest.mark.parametrize("N,flags", [(8, P | FLAG_BIAS), (32, P), (64, P | FLAG_BIAS), (64, P | R), (128, P),
                                     (256, P | FLAG_BIAS), (256, R), (512, P), (1024, P | R | FLAG_BIAS),
                                     (2048, P | FLAG_BIAS), (2048, P | R), (4096, P)])
def test_forward_rows_rule(acdc, N, flags):  # noqa: F811
    import torch
    K, few = 3, 11
    many = {8: 600011, 32: 400009, 64: 200003, 128: 200003, 256: 60013, 512: 60013, 1024: 30011, 2048: 20011,
            4096: 5003}[N]
    run_case(acdc, N, K, few, flags, seed=N)
    x, A, D, perm, gy = make_inputs(N, K, few, flags, N)
    bias = make_bias(N, K, N) if flags & FLAG_BIAS else None
    xt, At, Dt, pt, gt = (torch.from_numpy(t).cuda() for t in (x, A, D, perm, gy))
    bt = torch.from_numpy(bias).cuda() if bias is not None else None
    y0, s0 = acdc.forward(xt, At, Dt, pt, flags, save=True, bias=bt)
    u0 = acdc.saved_layer_inputs(s0, xt, K, flags)
    gx0 = acdc.backward(xt, gt, At, Dt, pt, flags, saved=s0, bias=bt)[0]
    for B in (FWD_ALONE_MAX[N], FWD_ALONE_MAX[N] + 1, many):
        print(f"[case] N={N} B={B} flags={flags}", flush=True)
        whole = lambda t: t.repeat(-(-B // few), 1)[:B].contiguous()  # noqa: E731
        xs = whole(xt)
        y, s = acdc.forward(xs, At, Dt, pt, flags, save=True, bias=bt)
        assert torch.equal(y, whole(y0))
        for a, b in zip(acdc.saved_layer_inputs(s, xs, K, flags), u0):
            assert torch.equal(a, whole(b))
        got = acdc.backward(xs, whole(gt), At, Dt, pt, flags, saved=s, bias=bt)
        assert torch.equal(got[0], whole(gx0))
        if not flags & R:
            copies = np.bincount(np.arange(B) % few, minlength=few).astype(np.float64)[:, None]
            ref = O.backward(x, gy * copies, A, D, perm, flags & 7, B=bias)
            for g, r in zip(got[1:], ref[1:]):
                assert rel_err(host(g), r) < TOL_REAL


def test_workspace_of_a_batch_serves_smaller_ones(acdc):  # noqa: F811
    # one workspace for a whole epoch: its last, ragged batch may run more
    # (smaller) backward workgroups than the full ones
    import torch
    N, K = 4096, 2
    full = torch.zeros(1100, N, device="cuda")
    ws = torch.empty(acdc.backward_workspace_bytes(full, K, 0, have_saved=True), dtype=torch.uint8, device="cuda")
    x = torch.randn(1003, N, device="cuda")
    A, D = torch.ones(K, N, device="cuda"), torch.ones(K, N, device="cuda")
    _, saved = acdc.forward(x, A, D, None, 0, save=True)
    gx, gA, _ = acdc.backward(x, x, A, D, None, 0, saved=saved, workspace=ws)
    # identity layers: dL/dx = x, dL/da = sum of x^2 over the rows
    ref = (x.double() ** 2).sum(0)
    assert float((gx - x).abs().max()) < 1e-5
    assert float(((gA.double() - ref) / ref).abs().max()) < 1e-5


# Multi-pass rows: every segment plan, the first DIF radix 2 to 16, a second
# level (N = 2^18; 2^21 complex: radix 32, 256 permutation sets), one
# permutation set a row or several; without permutations the DIT and DIF passes
# join in one launch.
@pytest.mark.parametrize("N,K,B,flags", [(512, 3, 3, P | R | FLAG_BIAS | MP), (1024, 2, 3, R | MP),
                                         (2048, 2, 5, P | FLAG_BIAS | MP), (8192, 3, 3, P | R | FLAG_BIAS | MP),
                                         (16384, 2, 3, R | FLAG_BIAS | MP), (32768, 3, 2, R | MP),
                                         (65536, 3, 3, R | FLAG_BIAS), (131072, 2, 2, P), (131072, 3, 2, FLAG_BIAS),
                                         (1 << 18, 3, 2, 0), (512, 3, 3, CX | MP), (1024, 2, 3, CX | P | MP),
                                         (2048, 2, 3, CX | P | MP), (8192, 3, 2, CX | P | MP), (32768, 3, 2, CX),
                                         (131072, 2, 2, CX | P), (1 << 18, 2, 1, CX), (16384, 2, 3, CX | P | MP),
                                         (1 << 21, 2, 1, CX | P), (1 << 21, 2, 1, CX), (16384, 3, 3, P | MP)])
def test_multipass_plans(acdc, N, K, B, flags):  # noqa: F811
    run_case(acdc, N, K, B, flags, seed=N % 1000 + B + flags)


# Row blocks of the image sums: B rows x units / 512 rows a block, 1 to 16
# (N = 65536: 4 pairs and 4 sets; N = 512: one pair and set; complex 32768: 8
# segments and 4 sets), whole and ragged.
@pytest.mark.parametrize("N,K,B,flags", [(65536, 1, 259, P), (512, 1, 1023, P | MP), (512, 2, 1537, P | MP),
                                         (256, 2, 9001, FLAG_BIAS | MP), (32768, 1, 131, CX | P),
                                         (512, 2, 4099, CX | MP)])
def test_multipass_row_block_edges(acdc, N, K, B, flags):  # noqa: F811
    run_case(acdc, N, K, B, flags, seed=N % 1000 + B)


# Narrow multi-pass rows share a column workgroup from 1024 rows on (B / 512
# rows side by side, at most those of 16384 floats): the last batch of one row
# a workgroup, whole and ragged last workgroups, the most rows there are.
@pytest.mark.parametrize("N,B,flags", [(256, 1023, P | R | MP), (256, 1027, P | R | FLAG_BIAS | MP),
                                       (256, 40000, P | MP), (2048, 4101, P | R | MP), (8192, 1025, P | FLAG_BIAS | MP),
                                       (256, 1025, CX | P | MP), (512, 20001, CX | P | MP), (2048, 3000, CX | MP)])
def test_multipass_narrow_rows_share_workgroups(acdc, N, B, flags):  # noqa: F811
    rows = np.unique(np.concatenate([np.arange(0, B, max(1, B // 120)), np.arange(max(0, B - 70), B)]))
    run_case(acdc, N, 3, B, flags, seed=N + B, rows=rows)


# Column launches whose workgroups take several rows in turn: more rows than
# the grid has workgroups (65536, of up to 64 rows at N = 256).  Rows are
# independent, so copies of a few rows give those rows' results, bit for bit.
@pytest.mark.parametrize("N,B,flags", [(256, 64 * 65536 + 3, P | R | FLAG_BIAS | MP), (256, 32 * 65536 + 3, CX | P | MP),
                                       (65536, 16387, P | R), (32768, 16387, CX)])
def test_multipass_more_rows_than_workgroups(acdc, N, B, flags):  # noqa: F811
    import torch
    K, few, fl = 2, 7, flags & ~CX
    x, A, D, perm, gy = (torch.from_numpy(t).cuda() for t in make_inputs(N, K, few, flags, N + 1))
    bias = torch.from_numpy(make_bias(N, K, N)).cuda() if flags & FLAG_BIAS else None
    y0, s0 = acdc.forward(x, A, D, perm, fl, save=True, bias=bias)
    gx0 = acdc.backward(x, gy, A, D, perm, fl, saved=s0, bias=bias)[0]
    n = -(-B // few)
    whole = lambda t: t.repeat(n, 1)[:B].contiguous()  # noqa: E731
    y, s = acdc.forward(whole(x), A, D, perm, fl, save=True, bias=bias)
    assert torch.equal(y, whole(y0))
    del y
    gx = acdc.backward(whole(x), whole(gy), A, D, perm, fl, saved=s, bias=bias)[0]
    assert torch.equal(gx, whole(gx0))


def test_multipass_tables_rebuilt_per_layer(acdc):  # noqa: F811
    # five layers' permutation tables at the widest row are past 256 MB, so
    # each layer's are built in turn; 256 sets a row
    run_case(acdc, 1 << 22, 5, 1, P, seed=3)


@pytest.mark.parametrize("N,B,flags", [(256, 1100, P | R | FLAG_BIAS | MP), (8192, 37, P | FLAG_BIAS | MP),
                                       (65536, 37, P | R | FLAG_BIAS), (65536, 150, R | FLAG_BIAS), (4096, 37, CX | P | MP),
                                       (1 << 18, 3, CX | P), (131072, 5, CX)])
def test_multipass_workspace_holds_all(acdc, N, B, flags):  # noqa: F811
    # a workspace of exactly the stated size, all NaN patterns, between bytes
    # that no call may change; the results are those of a roomy one
    import torch
    K, fl = 3, flags & ~CX
    x, A, D, perm, gy = (torch.from_numpy(t).cuda() for t in make_inputs(N, K, B, flags, N + B))
    bias = torch.from_numpy(make_bias(N, K, N)).cuda() if flags & FLAG_BIAS else None

    def space(need, roomy):
        buf = torch.full((need * (2 if roomy else 1) + 8192,), 255, dtype=torch.uint8, device="cuda")
        return buf, buf[4096: buf.numel() - 4096]

    def untouched(buf):
        return bool((buf[:4096] == 255).all()) and bool((buf[-4096:] == 255).all())

    outs = []
    for roomy in (False, True):
        buf, ws = space(acdc.forward_workspace_bytes(x, K, fl, bias), roomy)
        y, saved = acdc.forward(x, A, D, perm, fl, save=True, bias=bias, workspace=ws)
        assert untouched(buf)
        got = [y, saved]
        for have in (True, False):
            buf, ws = space(acdc.backward_workspace_bytes(x, K, fl, have, bias), roomy)
            got += acdc.backward(x, gy, A, D, perm, fl, saved=saved if have else None, bias=bias, workspace=ws)
            assert untouched(buf)
        outs.append(got)
    for tight, wide in zip(*outs):
        assert bool(torch.isfinite(torch.view_as_real(tight) if tight.is_complex() else tight).all())
        assert torch.equal(tight, wide)
