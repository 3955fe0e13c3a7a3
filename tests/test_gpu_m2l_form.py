"""The plain FP64 / FP32 M2L where it serves above p = 3 (csrc/m2l_form.h): adaptive
trees of many targets at p 4 .. 7 (p = 6: the last row on the vector unit); and a
plan that goes from one form to the other and back by re-planning.

FP64 against the oracle to rounding (1e-12); FP32 within the mixed gate (1e-5)
of the oracle.  A re-planned plan gives the bits of a plan made for those
positions."""
import numpy as np
import pytest

import oracle
from gpu_util import assert_close, B, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu

MIXED, FP64 = B.FMM_PREC_MIXED, B.FMM_PREC_FP64


@pytest.mark.parametrize("p,n", [(4, 9001), (5, 12001), (6, 16001), (7, 16001)])
def test_large_adaptive_trees_against_the_oracle(p, n):
    # some 1900 to 3700 divided parents: leaves of at most 2 particles
    pos, q = W.uniform_gauss(n, 20 + p)
    phi, force, _, st = oracle.fmm_adaptive(pos, q, 2, 5, p, side=1.0)
    assert st["boxes"] > 8 * 1800
    for prec, kind, tol in ((FP64, B.FMM_M2L_AUTO, 1e-12), (MIXED, B.FMM_M2L_F32, 1e-5)):
        out = run_gpu(pos, q, 5, p, prec, leaf_max=2, m2l_kind=kind)
        assert_close(out[0], phi, tol, what="phi")
        assert_close(out[1], force, tol, what="force")


def test_replans_across_the_forms():
    import torch

    n, p, depth, leaf = 9001, 4, 5, 2
    many, q = W.uniform_gauss(n, 31)             # about 1900 divided parents: plain
    few = np.floor(8.0 * many) / 8.0 + 1e-3 * (0.5 + many)  # a corner of each of 512 cells: 1097
    tq = torch.tensor(q, device="cuda")
    for prec, kind in ((FP64, B.FMM_M2L_AUTO), (MIXED, B.FMM_M2L_F32)):
        f = B.FMM(torch.tensor(many, device="cuda"), p=p, depth=depth, precision=prec, side=1.0, leaf_max=leaf,
                  m2l_kind=kind)
        for x in (many, few, few, many, few):
            B.fmm_replan(f.plan, torch.tensor(x, device="cuda"))
            phi, force, e = f.evaluate(tq)
            ref = run_gpu(x, q, depth, p, prec, leaf_max=leaf, m2l_kind=kind)
            assert (phi.cpu().numpy() == ref[0]).all() and (force.cpu().numpy() == ref[1]).all()
            assert e.item() == ref[2]
        f.close()
