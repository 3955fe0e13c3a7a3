"""The workspace may be any device memory: a plan in fine-grained memory
(hipExtMallocWithFlags), where not every GPU has floating-point atomic adds,
gives the bits of one in ordinary memory.  Sizes whose FP64 M2L is shared by
two work-groups (depth 2 to 4), and one that is not."""
import ctypes
import re

import numpy as np
import pytest

from gpu_util import B, run_gpu
from paper_2209_13121_amd import workloads as W

pytestmark = pytest.mark.gpu

FINE_GRAINED = 1  # hipDeviceMallocFinegrained


def runtime():
    """The HIP runtime that torch mapped."""
    path = next(m.group(0) for m in map(re.compile(r"/\S*libamdhip64\.so\S*").search, open("/proc/self/maps")) if m)
    return ctypes.CDLL(path)


@pytest.mark.parametrize("n,depth,p", [(300, 2, 12), (4096, 3, 4), (3001, 4, 9), (5000, 5, 5)])
def test_fine_grained_workspace_gives_the_same_bits(n, depth, p):
    import torch

    pos, q = W.uniform_gauss(n, 11 + p)
    ref = run_gpu(pos, q, depth, p, B.FMM_PREC_FP64)
    tp, tq = torch.tensor(pos, device="cuda"), torch.tensor(q, device="cuda")
    out = torch.zeros(4 * n + 1, device="cuda", dtype=torch.float64)
    cfg = B.make_config(p=p, depth=depth)
    size = B.fmm_workspace_size(cfg, n)
    hip, lib = runtime(), B.load()
    ws, plan = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipExtMallocWithFlags(ctypes.byref(ws), ctypes.c_size_t(size), ctypes.c_uint(FINE_GRAINED)) == 0
    try:
        ptr = lambda k: ctypes.c_void_p(out.data_ptr() + 8 * k)  # noqa: E731
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert lib.fmm_plan(ctypes.byref(cfg), n, ctypes.c_void_p(tp.data_ptr()), ws, size, stream,
                            ctypes.byref(plan)) == 0
        assert lib.fmm_evaluate(plan, ctypes.c_void_p(tq.data_ptr()), ptr(0), ptr(n), ptr(4 * n), stream) == 0
        assert lib.fmm_check(plan) == 0
        assert lib.fmm_destroy(plan) == 0
    finally:
        torch.cuda.synchronize()
        assert hip.hipFree(ws) == 0
    got = out.cpu().numpy()
    assert (got[:n] == ref[0]).all() and (got[n:4 * n].reshape(n, 3) == ref[1]).all()
    assert got[4 * n] == ref[2]
    assert np.isfinite(got).all()
