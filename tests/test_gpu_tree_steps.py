"""The leaf sort on both sides of its rule for few work-groups (n = 32768), leaves
of more and fewer particles than a quad that start at every residue, and the
energy's sum by one block (n <= 4096) and by many.

Sorted order: a plan's results do not depend on the order of its input, so a
permuted input gives the permuted output to rounding of the sums (order inside
a leaf follows the user index): 1e-12 normwise in FP64; two runs of one input
are the same to the bit; the energy is half the sum of q phi to 1e-13 of the
sum of magnitudes."""
import numpy as np
import pytest

from gpu_util import assert_close, B, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depth,leaf_max", [(1, 3, 0), (5, 3, 0), (1023, 3, 0), (1025, 4, 0), (4096, 3, 0), (4097, 4, 0), (32767, 3, 0),
                                              (32768, 4, 0), (32769, 4, 0), (40001, 3, 0), (20000, 5, 24),
                                              (40001, 5, 24)])
def test_sorted_order_and_energy(n, depth, leaf_max):
    pos, q = W.uniform_gauss(n, 700 + n % 13)
    a = run_gpu(pos, q, depth, 4, B.FMM_PREC_FP64, leaf_max=leaf_max)
    b = run_gpu(pos, q, depth, 4, B.FMM_PREC_FP64, leaf_max=leaf_max)
    assert (a[0] == b[0]).all() and (a[1] == b[1]).all() and a[2] == b[2]
    assert abs(a[2] - 0.5 * (q * a[0]).sum()) <= 1e-13 * np.abs(q * a[0]).sum()
    o = np.random.default_rng(n).permutation(n)
    c = run_gpu(pos[o], q[o], depth, 4, B.FMM_PREC_FP64, leaf_max=leaf_max)
    if n > 1:
        assert_close(c[0], a[0][o], 1e-12, what="phi")
        assert_close(c[1], a[1][o], 1e-12, what="force")


@pytest.mark.parametrize("side", [1.0, 0.0])
def test_replans_keep_the_maps_and_reset_the_sums(side):
    import torch

    n = 5000
    pos, q = W.uniform_gauss(n, 3)
    other, _ = W.uniform_gauss(n, 4)
    tq = torch.tensor(q, device="cuda")
    f = B.FMM(torch.tensor(pos, device="cuda"), p=4, depth=3, lo=(0.0, 0.0, 0.0), side=side)
    for x in (other, pos, other):
        tx = torch.tensor(x, device="cuda")
        B.fmm_replan(f.plan, tx)
        for _ in range(2):
            phi, force, e = f.evaluate(tq)
        ref = run_gpu(x, q, 3, 4, B.FMM_PREC_FP64, side=side)
        assert (phi.cpu().numpy() == ref[0]).all() and (force.cpu().numpy() == ref[1]).all()
        assert e.item() == ref[2]
