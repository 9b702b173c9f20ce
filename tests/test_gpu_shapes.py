"""GPU parity at the shapes where a launch or sum rule changes its split.

Each case runs through the same comparison with the fp64 oracle as the other
GPU parity tests (every element, same tolerance)."""

import pytest

from oracle import acdc_oracle as O
from paper_1511_05946_amd.workloads import FLAG_BIAS
from tests.test_gpu_parity import acdc, run_case  # noqa: F401

pytestmark = pytest.mark.gpu

P, R, CX = O.FLAG_PERM, O.FLAG_RELU, O.FLAG_COMPLEX


# Narrow rows: one tile holds 256 (N = 8, 16) down to 16 rows (N = 512; up to
# 512 complex ones), and the image sums split them into phases.  A whole tile
# and one row of the next, and a single row.
@pytest.mark.parametrize("N,B,flags", [(8, 257, P | R | FLAG_BIAS), (16, 256, P), (32, 129, P | R), (64, 1, P),
                                       (64, 129, P | R | FLAG_BIAS), (128, 65, P), (256, 65, P | R),
                                       (512, 17, P | R | FLAG_BIAS), (8, 513, CX | P), (32, 257, CX | P),
                                       (64, 129, CX | P), (256, 65, CX | P)])
def test_narrow_tile_sums(acdc, N, B, flags):  # noqa: F811
    run_case(acdc, N, 3, B, flags, seed=N + B)
