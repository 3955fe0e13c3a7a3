"""The near field of small leaves by parent box (uniform trees of at least 4096
parents and at most 8 particles a leaf, here depth 5): crowded parents that take
several rounds of targets and tiles of sources, in one leaf, over a parent's 8
leaves and over 8 leaves of 8 parents, against the direct sum (leaves that all
touch have no far field); and the flag of coincident points, with at most 32 and
with more targets in the parent.

FP64 to 1e-12 (rounding of at most 800 terms); mixed to 2e-6 normwise (FP32
terms and sums of at most 800 of them: sqrt(800) 2^-24 = 1.7e-6)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu

DEPTH, H = 5, 1.0 / 32
MIXED, FP64 = B.FMM_PREC_MIXED, B.FMM_PREC_FP64


@pytest.mark.parametrize("corner,leaves", [((4, 6, 8), 1), ((4, 6, 8), 2), ((5, 7, 9), 2), ((0, 0, 0), 2), ((30, 30, 30), 2)])
@pytest.mark.parametrize("n", [3, 31, 32, 33, 64, 65, 255, 257, 300, 800])
def test_crowded_parents_against_the_direct_sum(corner, leaves, n):
    rng = np.random.default_rng(n + 7 * corner[0] + leaves)
    pos = H * (np.array(corner) + leaves * rng.random((n, 3)))
    q = rng.standard_normal(n)
    phi, force = oracle.direct(pos, q)[:2]
    for prec, tol in ((FP64, 1e-12), (MIXED, 2e-6)):
        out = run_gpu(pos, q, DEPTH, 3, prec)
        assert_close(out[0], phi, tol, what="phi")
        assert_close(out[1], force, tol, what="force")


@pytest.mark.parametrize("crowd", [0, 20, 40, 300])
@pytest.mark.parametrize("prec", [FP64, MIXED])
def test_coincident_points_raise_the_flag(crowd, prec):
    pos, q = W.uniform_gauss(1000, 61)
    pos[:crowd] = H * (np.array([9, 4, 17]) + np.random.default_rng(crowd).random((crowd, 3)))  # one leaf
    assert run_gpu(pos, q, DEPTH, 4, prec)[3] == 0
    for a, b in ((0, crowd // 2 + 1), (990, 991), (crowd // 3, 995)):
        bad = pos.copy()
        bad[b] = bad[a]
        assert B.STATUS_NAMES[run_gpu(bad, q, DEPTH, 4, prec, check=False)[3]] == "FMM_E_COINCIDENT"
