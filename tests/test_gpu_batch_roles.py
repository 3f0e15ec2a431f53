"""Row counts and tensor counts at the edges of the batched MFMA kernels'
producer and consumer roles, against the FP64 oracle.

n1 = 32, 33, 64, 65 and 96 are the edges of one, two and three 32-row blocks
(two waves share a tensor from two blocks on) and of the adjoint's 16-row
chunks; 1, 4, 5 and 33 tensors are the edges of the forward's steps of four
and the adjoint's chunks of 32; 1, 32 and 33 right-hand sides those of a
group; ranks 1, 16, 17 and 32 those of a row block.
"""
import pytest

import workloads
from oracle import matvec as om
from tests.plans import assert_close, random_struct, struct_to_abi
from tests.test_gpu_batch import _run

pytestmark = pytest.mark.gpu

CASES = [
    ((32, 9, 3), 1, (1, 5), 16, (32, 1)),
    ((33, 8, 2), 2, (4, 33), 17, (33, 1)),
    ((64, 5, 3), 1, (5, 1), 32, (1, 32)),
    ((65, 8, 2), 3, (33,), 16, (33,)),
    ((96, 3, 2), 1, (4, 5), 1, (32, 33)),
]


# FP32: the bound of the other batched tests.  BF16X3 drops the lo x lo
# products, 2^-16 of a product each, and keeps FP32 sums: 1e-4.
@pytest.mark.parametrize("prec,tol", [("fp32", 1e-5), ("bf16x3", 1e-4)])
@pytest.mark.parametrize("dims,q,ms,rmax,nrhs", CASES)
def test_batch_role_edges(gpu_lib, dims, q, ms, rmax, nrhs, prec, tol):
    import numpy as np
    import torch
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan
    print(f"batch roles dims={dims} q={q} m={ms} rmax={rmax} rhs={nrhs} {prec}", flush=True)
    structs = [random_struct(dims, q, m, rmax, 300 + c) for c, m in enumerate(ms)]
    kw = {"precision": lib.TV_PREC_BF16X3} if prec == "bf16x3" else {}
    plans = [TuckerPlan.from_factors(S.dims, S.q, S.m, *struct_to_abi(S), **kw) for S in structs]
    X = [workloads.complex_normal((S.m, n), 310 + c) for c, (S, n) in enumerate(zip(structs, nrhs))]
    Y = [workloads.complex_normal((S.q * S.nv, n), 320 + c)
         for c, (S, n) in enumerate(zip(structs, nrhs))]
    cx = lambda a: torch.from_numpy(a.astype(np.complex64)).cuda()  # noqa: E731
    fwd = _run(plans, 0, [cx(x) for x in X], nrhs)
    adj = _run(plans, 1, [cx(y) for y in Y], nrhs)
    for c, S in enumerate(structs):
        assert_close(fwd[c], om.alg1(S, X[c]), tol, what=("forward", c))
        assert_close(adj[c], om.alg2(S, Y[c]), tol, what=("adjoint", c))
