"""P2M's groups of lanes per leaf: 1, 2 and 4 (many leaves), 16 (few, or large
ones) and 64 (very few), with empty leaves, leaves below and above a group.

Charges are zero but for some whole leaves and some scattered particles, so the
oracle's FMM over those alone has the same potential and force there: FP64 to
1e-12 (rounding), at any number of particles.  Adaptive
trees take the same rule and meet their own oracle in the tests of that tree."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, energy_rel, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depth,p", [(3000, 5, 5), (200001, 5, 4), (540001, 5, 5), (700, 4, 1), (9001, 4, 7),
                                       (300001, 4, 6), (50, 2, 3), (2000, 3, 12), (70001, 3, 8)])
def test_lanes_against_the_oracle_on_the_charged_particles(n, depth, p):
    pos, q = W.uniform_gauss(n, 300 + n % 97)
    cell = np.floor(pos * 2**depth).astype(np.int64)
    keep = (cell[:, 1:] == 2 ** (depth - 1)).all(1) & (cell[:, 0] % 3 == 0)  # some leaves of a row
    keep[np.flatnonzero(keep)[1200:]] = False
    keep[:400] = True
    q = np.where(keep, q, 0.0)
    out = run_gpu(pos, q, depth, p, B.FMM_PREC_FP64)
    ref = oracle.fmm(pos[keep], q[keep], depth, p)
    assert_close(out[0][keep], ref[0], 1e-12, what="phi")
    assert_close(out[1][keep], ref[1], 1e-12, what="force")
    assert energy_rel(out[2], ref[2]) <= 1e-12
