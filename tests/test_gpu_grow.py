"""The assembly's own plan (U of Algorithm 3, grown a column at a time) keeps
its column-GEMM adjoint, in lower slabs, where the workspace holds no slab of all
i3.  The plan has no entry point of its own: its functions are called by their
C++ names."""
import ctypes as C

import numpy as np
import pytest

from oracle import matvec as om
from tests.plans import adj_terms, assert_close, random_struct, struct_to_abi

pytestmark = pytest.mark.gpu


class _Grid(C.Structure):
    _fields_ = [("n1", C.c_int32), ("n2", C.c_int32), ("n3", C.c_int32), ("q", C.c_int32),
                ("m", C.c_int64)]


class _Stage(C.Structure):
    _fields_ = [("ptr", C.c_void_p), ("bytes", C.c_size_t)]


@pytest.mark.parametrize("prec,tol", [(0, 1e-5), (1, 1e-4)])
@pytest.mark.parametrize("dims,q,budget", [((33, 20, 40), 3, 1 << 21), ((130, 9, 31), 2, 1 << 21),
                                           ((33, 20, 40), 12, 3 << 21), ((33, 20, 40), 3, 1 << 28)])
def test_grown_plan_adjoint_in_little_workspace(gpu_lib, dims, q, budget, prec, tol):
    import torch
    from paper_2103_06393_amd import lib
    print(f"grown plan {dims} q={q} budget={budget} precision {prec}", flush=True)
    so = C.CDLL(str(lib.LIB_PATH))
    bound = so._ZN2tv16plan_arena_boundERK7tv_gridPKi14tv_precision_e
    bound.restype = C.c_size_t
    create = so._ZN2tv16grow_plan_createERK7tv_gridPKi14tv_precision_ePvmP12ihipStream_tPP9tv_plan_s
    stage = so._ZN2tv19grow_plan_set_stageEP9tv_plan_sRKNS_9HostStageEm
    append = so._ZN2tv16grow_plan_appendEP9tv_plan_sPKiPKdS5_S5_S5_P12ihipStream_t
    S = random_struct(dims, q, 12, 7, 41)
    ranks, cores, u1, u2, u3 = struct_to_abi(S)
    g, rmax = _Grid(*dims, q, S.m), (C.c_int32 * 3)(7, 7, 7)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    nb = bound(C.byref(g), rmax, prec)
    arena = torch.empty(nb, dtype=torch.uint8, device="cuda")
    plan = C.c_void_p()
    assert create(C.byref(g), rmax, prec, C.c_void_p(arena.data_ptr()), C.c_size_t(nb), st,
                  C.byref(plan)) == 0
    try:
        stage(plan, C.byref(_Stage(None, 0)), C.c_size_t(budget))
        ptr = lambda a: a.ctypes.data_as(C.c_void_p)  # noqa: E731
        o = [0, 0, 0, 0]
        for j in range(S.m):
            r = np.ascontiguousarray(ranks[q * j:q * (j + 1)])
            n = [int(np.prod(r.astype(np.int64), axis=1).sum()),
                 *(int(d * r[:, i].sum()) for i, d in enumerate(dims))]
            col = [np.ascontiguousarray(v[a:a + b]) for v, a, b in zip((cores, u1, u2, u3), o, n)]
            assert append(plan, ptr(r), *(ptr(v) for v in col), st) == 0, lib.tv_last_error()
            o = [a + b for a, b in zip(o, n)]
        info = lib.tv_plan_info(plan.value)
        need = lib.tv_workspace_bytes(plan.value, 1, 1)
        assert info.kernel[1] == 2 and need <= budget
        if prec == 0:                   # (two planes of y may fit where three do not)
            assert (info.tile_t2[1] < dims[2]) == (budget < 1 << 28)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        rng = np.random.default_rng(6)
        y = rng.standard_normal(q * S.nv) + 1j * rng.standard_normal(q * S.nv)
        yd = torch.from_numpy(y.astype(np.complex64)).cuda()
        x = torch.empty(S.m, dtype=torch.complex64, device="cuda")
        lib.tv_rmatvec(plan.value, yd.data_ptr(), q * S.nv, 1, x.data_ptr(), S.m, ws.data_ptr(),
                       need, st.value)
        assert_close(x.cpu().numpy(), om.alg2(S, y)[:, 0], tol, terms=adj_terms(S, y), what="U^* y")
    finally:
        lib.tv_plan_destroy(plan.value)
