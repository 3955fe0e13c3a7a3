"""The reflection-reduced M2L (FP64 plans and FMM_M2L_F32, p >= 4) in each of
its forms: few targets (depth 2 and 3: the waves of a work-group split the
offset orbits), the block form (uniform, depth 5, mostly empty boxes) and the
gather form of large adaptive trees.

FP64 against the oracle's FMM to rounding (1e-12) at every order whose class
sizes, last k chunk or register split differ; where the oracle would take
minutes (depth 5 above p = 5), against the split-BF16 form, which shares no M2L
kernel and no operator table with it, within the mixed gate (energy 1e-6, RMS
force 1e-5, potential 1e-5)."""
import pytest

import oracle
from gpu_util import assert_close, B, energy_rel, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu

MIXED, FP64 = B.FMM_PREC_MIXED, B.FMM_PREC_FP64


def check(out, ref, norm_phi, norm_f, tol_e):
    assert_close(out[0], ref[0], norm_phi, what="phi")
    assert_close(out[1], ref[1], norm_f, what="force")
    assert energy_rel(out[2], ref[2]) <= tol_e


@pytest.mark.parametrize("depth,p", [(2, 4), (2, 9), (3, 4), (3, 5), (3, 7), (3, 8), (3, 10), (3, 11), (3, 12),
                                     (5, 4), (5, 5)])
def test_fp64_against_the_oracle(depth, p):
    pos, q = W.uniform_gauss(1501, 60 + p)
    check(run_gpu(pos, q, depth, p, FP64), oracle.fmm(pos, q, depth, p), 1e-12, 1e-12, 1e-12)


@pytest.mark.parametrize("p", [6, 7, 8, 9, 10, 11, 12])
def test_block_form_against_the_split_form(p):
    pos, q = W.uniform_gauss(30001, 80 + p)
    ref = run_gpu(pos, q, 5, p, FP64)
    split = run_gpu(pos, q, 5, p, MIXED, m2l_kind=B.FMM_M2L_BF16X3)
    check(split, ref, 1e-5, 1e-5, 1e-6)
    check(run_gpu(pos, q, 5, p, MIXED, m2l_kind=B.FMM_M2L_F32), ref, 1e-5, 1e-5, 1e-6)


@pytest.mark.parametrize("p", [4, 10, 12])
def test_gather_form_of_a_large_adaptive_tree(p):
    pos, q, _ = W.molecular_clusters(20000, 90 + p)
    ref = run_gpu(pos, q, 6, p, FP64, side=0.0, leaf_max=12)
    split = run_gpu(pos, q, 6, p, MIXED, side=0.0, leaf_max=12, m2l_kind=B.FMM_M2L_BF16X3)
    check(split, ref, 1e-5, 1e-5, 1e-6)
    check(run_gpu(pos, q, 6, p, MIXED, side=0.0, leaf_max=12, m2l_kind=B.FMM_M2L_F32), ref, 1e-5, 1e-5, 1e-6)


@pytest.mark.parametrize("depth,leaf_max,n,p", [(2, 0, 300, 12), (4, 0, 3001, 7), (4, 0, 3001, 11), (5, 2, 6001, 4),
                                                (4, 2, 2500, 9), (5, 2, 6001, 12)])
def test_small_form_with_one_and_two_work_groups_per_target(depth, leaf_max, n, p):
    # 8 and 296 work-groups (two share 16 targets) and, on adaptive trees, about
    # 250 and 700 (one); two runs are the same to the bit in both
    pos, q = W.uniform_gauss(n, 40 + p)
    a = run_gpu(pos, q, depth, p, FP64, leaf_max=leaf_max)
    b = run_gpu(pos, q, depth, p, FP64, leaf_max=leaf_max)
    for x, y in zip(a[:2], b[:2]):
        assert (x == y).all()
    ref = oracle.fmm_adaptive(pos, q, leaf_max, depth, p, side=1.0) if leaf_max else oracle.fmm(pos, q, depth, p)
    check(a, ref, 1e-12, 1e-12, 1e-12)
