"""M2P's lane groups: leaves of at most 16, at most 32, at most 64 and more
particles with W lists, at the least, middle and highest orders, against the
oracle of the adaptive tree: FP64 to rounding (1e-12), mixed within its gate
(potential and force 1e-5)."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaf_max,p", [(12, 1), (14, 12), (30, 5), (60, 6), (60, 11), (150, 4)])
def test_each_lane_group_against_the_oracle(leaf_max, p):
    rng = np.random.default_rng(leaf_max + p)
    blobs = [0.3 + 0.02 * rng.standard_normal((900, 3)), [0.71, 0.3, 0.6] + 0.004 * rng.standard_normal((900, 3))]
    pos = np.clip(np.concatenate(blobs + [rng.random((1600, 3))]), 0.0, 1.0)
    q = rng.standard_normal(len(pos))
    phi, force, _, st = oracle.fmm_adaptive(pos, q, leaf_max, 7, p, side=1.0)
    assert st["w"] > 0
    for prec, tol in ((B.FMM_PREC_FP64, 1e-12), (B.FMM_PREC_MIXED, 1e-5)):
        out = run_gpu(pos, q, 7, p, prec, leaf_max=leaf_max)
        assert_close(out[0], phi, tol, what="phi")
        assert_close(out[1], force, tol, what="force")
