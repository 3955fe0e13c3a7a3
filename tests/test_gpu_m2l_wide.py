"""The FP64 M2L of large trees to rounding at every order: the block form (uniform
tree of depth 5) and the gather form of many targets (an adaptive tree of the same
boxes), both against the oracle.

One particle sits in each of the 32^3 cells, so the adaptive tree (leaves of at
most 4) divides every box above the cap and has the uniform tree's boxes, lists
and expansions.  Charges are zero but for 200 particles, so the oracle's FMM over
those and some uncharged ones has the same potentials and forces there: 1e-12."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, energy_rel, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [4, 5, 6, 7, 8, 9, 10, 11, 12])
def test_block_and_gather_forms_against_the_oracle(p):
    rng = np.random.default_rng(400 + p)
    cells = np.stack(np.meshgrid(*[np.arange(32)] * 3, indexing="ij"), axis=-1).reshape(-1, 3)
    pos = rng.permutation(cells + 0.05 + 0.9 * rng.random(cells.shape)) / 32.0
    q = np.zeros(len(pos))
    q[:200] = rng.standard_normal(200)
    keep = np.arange(1500)
    phi, force, energy = oracle.fmm(pos[keep], q[keep], 5, p)
    for leaf_max in (0, 4):
        out = run_gpu(pos, q, 5, p, B.FMM_PREC_FP64, leaf_max=leaf_max)
        assert_close(out[0][keep], phi, 1e-12, what="phi")
        assert_close(out[1][keep], force, 1e-12, what="force")
        assert energy_rel(out[2], energy) <= 1e-12
