"""BF16X3 GEMMs over all voxel rows in one workgroup (row_cap 8) at 10, 12, 14
and 16 blocks of 32 rows, both edges of each, against the FP64 oracle; and
entries near the largest float and non-finite ones in the two-plane split."""
import numpy as np
import pytest

from oracle import matvec as om
from tests.plans import adj_terms, assert_close, fwd_terms, random_struct, struct_to_abi

pytestmark = pytest.mark.gpu


def _plan(S, row_cap, slab, splits):
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan
    P = TuckerPlan.from_factors(S.dims, S.q, S.m, *struct_to_abi(S),
                                precision=lib.TV_PREC_BF16X3)
    for op in (0, 1):
        lib.tv_plan_configure(P.handle, op, path=1, row_cap=row_cap, slab_i3=slab, gemm_nbw=2,
                              splits=splits)
    return P


def _vectors(S, seed):
    rng = np.random.default_rng(seed)
    cx = lambda n: (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)  # noqa: E731
    return cx(S.m), cx(S.q * S.nv)


# 1e-4 of the moduli of the terms, as in the other BF16X3 tests (2^-17 a product)
@pytest.mark.parametrize("n1,n2,n3,q,m,slab,splits", [
    (129, 13, 12, 2, 7, 0, 1), (160, 16, 8, 1, 9, 0, 2),     # 10 blocks
    (161, 7, 21, 1, 6, 5, 1), (192, 11, 12, 3, 3, 0, 3),     # 12
    (193, 9, 15, 1, 8, 0, 1), (224, 17, 8, 2, 5, 3, 2),      # 14
    (225, 19, 7, 1, 5, 0, 2), (256, 8, 16, 1, 11, 0, 1),     # 16
])
def test_full_row_tiles(gpu_lib, n1, n2, n3, q, m, slab, splits):
    import torch
    print(f"full-row tile n1={n1} n2={n2} n3={n3} q={q} m={m} slab={slab} splits={splits}",
          flush=True)
    S = random_struct((n1, n2, n3), q, m, 9, 51)
    P = _plan(S, 8, slab, splits)
    x, y = _vectors(S, 3)
    for _ in range(2):
        assert_close(P.matvec(torch.from_numpy(x).cuda()).cpu().numpy(), om.alg1(S, x)[:, 0],
                     1e-4, terms=fwd_terms(S, x), what="Z x")
        assert_close(P.rmatvec(torch.from_numpy(y).cuda()).cpu().numpy(), om.alg2(S, y)[:, 0],
                     1e-4, terms=adj_terms(S, y), what="Z^* y")


@pytest.mark.parametrize("n1,row_cap", [(40, 0), (180, 8)])
def test_two_planes_at_the_ends_of_the_range(gpu_lib, n1, row_cap):
    """y near the largest float (above the largest bf16, so its high plane is
    that one), y and the factors tiny, and non-finite entries, which reach every
    result."""
    import torch
    print(f"two planes n1={n1}", flush=True)
    S = random_struct((n1, 9, 11), 2, 5, 6, 52)
    P = _plan(S, row_cap, 0, 1)
    _, y = _vectors(S, 4)
    top = float(np.finfo(np.float32).max)
    for s in (top / np.abs(np.stack([y.real, y.imag])).max() / 64, 2.0 ** -100):
        ys = (y * np.float32(s)).astype(np.complex64)
        got = P.rmatvec(torch.from_numpy(ys).cuda()).cpu().numpy().astype(np.complex128) / s
        y64 = ys.astype(np.complex128) / s
        assert_close(got, om.alg2(S, y64)[:, 0], 1e-4, terms=adj_terms(S, y64), what="Z^* y")
    e = np.zeros_like(y)
    e[7] = complex(top * 0.999, 0)
    got = P.rmatvec(torch.from_numpy(e).cuda()).cpu().numpy().astype(np.complex128) / top
    e64 = e.astype(np.complex128) / top
    assert_close(got, om.alg2(S, e64)[:, 0], 1e-4, terms=adj_terms(S, e64), what="one entry")
    for bad in (np.inf, np.nan):
        yb = y.copy()
        yb[:: S.nv] = complex(bad, 1.0)
        assert not np.isfinite(P.rmatvec(torch.from_numpy(yb).cuda()).cpu().numpy()).any()
