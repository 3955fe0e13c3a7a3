"""The near field's layout of a leaf's targets over a wave (sets of 64, then the
rest split over copies that share the sources): every remainder class against
the exact sum.

A leaf at depth 1 sees every particle (no far field), so with n particles in
one octant and m outside the result is the direct sum.  FP64 to 1e-12 (rounding
of at most 700 terms, each 1 / r to about 2 ulp, against the oracle's FP64
sum); mixed to 2e-6 normwise (FP32 terms and sums of at most 700 of them:
sqrt(700) 2^-24 = 1.6e-6)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 3, 5, 8, 15, 16, 21, 24, 31, 32, 33, 47, 63, 64, 65, 70, 127, 129, 191, 193, 256,
                               257, 300, 511, 513])
def test_every_group_layout_against_the_direct_sum(n):
    rng = np.random.default_rng(500 + n)
    pos = np.concatenate([0.5 * rng.random((n, 3)), 0.5 + 0.5 * rng.random((130, 3))])
    q = rng.standard_normal(len(pos))
    phi, force = oracle.direct(pos, q)[:2]
    for prec, tol in ((B.FMM_PREC_FP64, 1e-12), (B.FMM_PREC_MIXED, 2e-6)):
        out = run_gpu(pos, q, 1, 4, prec)
        assert_close(out[0], phi, tol, what="phi")
        assert_close(out[1], force, tol, what="force")


def test_close_pairs_keep_their_accuracy():
    # separations of 1e-3 .. 1e-9 leaf widths, within a leaf and across a face:
    # the FP64 1 / r (estimate and one third-order step) and the mixed offsets
    # (taken in FP64, then rounded) lose nothing with the separation; the
    # coordinates' own rounding (2^-53 of 0.5 leaf widths over 1e-9) bounds FP64
    rng = np.random.default_rng(9)
    a = rng.random((64, 3)) * 0.4 + 0.05
    d = rng.standard_normal((64, 3))
    d *= (10.0 ** -rng.uniform(3, 9, 64) / np.linalg.norm(d, axis=1))[:, None]
    face = a.copy()
    face[:, 0] = 0.5
    pos = np.concatenate([a, a + d, face - np.abs(d) * [1, 0, 0], face + np.abs(d) * [1, 0, 0]])
    q = rng.standard_normal(len(pos))
    phi, force = oracle.direct(pos, q)[:2]
    for prec, tol in ((B.FMM_PREC_FP64, 1e-6), (B.FMM_PREC_MIXED, 2e-6)):
        out = run_gpu(pos, q, 1, 4, prec)
        assert_close(out[0], phi, tol, what="phi")
        assert_close(out[1], force, tol, what="force")
