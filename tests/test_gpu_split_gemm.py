"""The split-bf16 GEMM of the decompress-then-GEMM products at every row tile
(1 to 8 blocks of 32 real rows, one to three tiles) and both column tiles,
against the FP64 oracle, and the exactness of its operand split."""
import numpy as np
import pytest

from oracle import matvec as om
from tests.plans import adj_terms, assert_close, fwd_terms, random_struct, struct_to_abi

pytestmark = pytest.mark.gpu


def _plan(S, prec, nbw, splits=1):
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan
    P = TuckerPlan.from_factors(S.dims, S.q, S.m, *struct_to_abi(S), precision=prec)
    for op in (0, 1):
        lib.tv_plan_configure(P.handle, op, path=1, splits=splits, gemm_nbw=nbw)
    return P


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,q,m,rmax,nbw", [
    ((11, 37, 7), 3, 5, 8, 4),      # 1 block
    ((32, 19, 14), 1, 9, 8, 2),     # 2 blocks, a whole tile
    ((47, 8, 33), 3, 4, 12, 2),     # 3 blocks, columns one past a tile
    ((80, 16, 16), 1, 33, 12, 4),   # 5 blocks, one column tile exactly
    ((95, 30, 9), 2, 7, 12, 2),     # 6 blocks
    ((109, 13, 21), 3, 3, 12, 4),   # 7 blocks
    ((128, 43, 6), 2, 6, 12, 4),    # 8 blocks, columns one short of two tiles
    ((205, 11, 12), 1, 5, 12, 4),   # two tiles of 7 blocks
    ((264, 9, 29), 1, 4, 10, 2),    # three tiles of 6 blocks
])
def test_row_tiles_match_oracle(gpu_lib, dims, q, m, rmax, nbw, prec):
    """FP32: every entry is a sum of rounded terms: modes 3 and 2 (at most
    rmax FP32 sums each), one rounding per chunk of the GEMM (8 stacked rows
    or columns) and the split's dropped products (2^-23), all relative to the
    moduli of the terms.  BF16X3: 2^-17 per product, 1e-4 as elsewhere."""
    import torch
    S = random_struct(dims, q, m, rmax, 7)
    P = _plan(S, prec, nbw)
    chunks = max(rmax * m, dims[1] * dims[2]) / 8
    tol = 1e-4 if prec else (2 * rmax + chunks + 8) * 2.0 ** -24
    rng = np.random.default_rng(3)
    x = rng.standard_normal(m) + 1j * rng.standard_normal(m)
    y = rng.standard_normal(S.q * S.nv) + 1j * rng.standard_normal(S.q * S.nv)
    x, y = x.astype(np.complex64), y.astype(np.complex64)
    got = P.matvec(torch.from_numpy(x).cuda()).cpu().numpy()
    assert_close(got, om.alg1(S, x)[:, 0], tol, terms=fwd_terms(S, x), what="Z x")
    got = P.rmatvec(torch.from_numpy(y).cuda()).cpu().numpy()
    assert_close(got, om.alg2(S, y)[:, 0], tol, terms=adj_terms(S, y), what="Z^* y")


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** 60])
def test_split_is_exact_under_scaling(gpu_lib, scale):
    """The three bf16 parts hold all 24 bits whatever the exponent: scaling the
    operand by a power of two scales the result by it, bit for bit."""
    import torch
    S = random_struct((70, 12, 9), 2, 6, 8, 5)
    P = _plan(S, 0, 4, splits=2)
    g = torch.Generator(device="cuda").manual_seed(2)
    for rows, fn in ((S.m, P.matvec), (S.q * S.nv, P.rmatvec)):
        v = torch.randn(rows, dtype=torch.complex64, device="cuda", generator=g)
        assert torch.equal(fn(v * scale), fn(v) * scale)


def test_noalloc_takes_what_fp32_operands_fitted(gpu_lib):
    """An adjoint whose slab, partials and y fit the static scratch in FP32
    but not with y as three bf16 planes runs in lower slabs there."""
    import torch
    from paper_2103_06393_amd import lib
    S = random_struct((64, 64, 40), 3, 104, 6, 9)
    P = _plan(S, 0, 4)
    assert lib.tv_workspace_bytes(P.handle, 1, 1) > lib.TV_STATIC_SCRATCH_BYTES
    rows = S.q * S.nv
    y = torch.randn(rows, dtype=torch.complex64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(4))
    x = torch.empty(S.m, dtype=torch.complex64, device="cuda")
    lib.tv_rmatvec_noalloc(P.handle, y.data_ptr(), rows, 1, x.data_ptr(), S.m,
                           torch.cuda.current_stream().cuda_stream)
    ref = P.rmatvec(y)
    # FP32 sums of 1/8 of 64 x 40 columns in another order
    assert float((x - ref).norm() / ref.norm()) < 320 * 2.0 ** -24


@pytest.mark.parametrize("dims,q,m,rmax,slab", [
    ((8, 1, 1), 2, 3, 1, 0),        # one column, rank 1
    ((9, 3, 40), 1, 4, 3, 17),      # few i2; slabs of 16 + 1 values of i3
    ((20, 33, 9), 2, 5, 9, 0),      # i2 one past a block, an i3 count past 8
    ((24, 64, 20), 1, 3, 24, 7),    # up to 24 b, a ragged last slab
    ((40, 97, 18), 1, 3, 32, 0),    # 32 b: 8 i3 or fewer a workgroup
    ((48, 64, 48), 1, 3, 40, 0),    # over 32 b
])
def test_decompression_edges_match_oracle(gpu_lib, dims, q, m, rmax, slab):
    """Both directions over the decompression's edges: blocks of 32 i2 and 32
    (i3, a) rows, groups of four b, slabs.  Tolerance as for the row tiles."""
    import torch
    from paper_2103_06393_amd import lib
    S = random_struct(dims, q, m, rmax, 11)
    P = _plan(S, 0, 2)
    for op in (0, 1):
        lib.tv_plan_configure(P.handle, op, path=1, splits=1, slab_i3=slab, gemm_nbw=2)
    tol = (2 * rmax + max(rmax * m, dims[1] * dims[2]) / 8 + 8) * 2.0 ** -24
    rng = np.random.default_rng(6)
    x = (rng.standard_normal(m) + 1j * rng.standard_normal(m)).astype(np.complex64)
    y = rng.standard_normal(S.q * S.nv) + 1j * rng.standard_normal(S.q * S.nv)
    y = y.astype(np.complex64)
    for _ in range(2):              # the second call finds the first one's workspace
        got = P.matvec(torch.from_numpy(x).cuda()).cpu().numpy()
        assert_close(got, om.alg1(S, x)[:, 0], tol, terms=fwd_terms(S, x), what="Z x")
        got = P.rmatvec(torch.from_numpy(y).cuda()).cpu().numpy()
        assert_close(got, om.alg2(S, y)[:, 0], tol, terms=adj_terms(S, y), what="Z^* y")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("dims,q,m,rmax,kernels,aca", [
    ((20, 13, 7), 2, 5, 5, (1, 1), False),        # tiny: fused
    ((24, 4, 90), 3, 12, 4, (0, 0), False),       # a narrow grid: phased fused kernels
    ((33, 35, 37), 3, 40, 8, (1, 1), False),      # small
    ((32, 64, 24), 3, 80, 8, (2, 2), True),       # scratch-sized, over 256 rows
    ((64, 64, 64), 3, 20, 8, (2, 1), False),      # few stacked rows
    ((160, 64, 64), 3, 24, 8, (2, 1), True),      # adjoint slab past the static scratch
])
def test_new_plan_path_agrees_with_fused(gpu_lib, dims, q, m, rmax, kernels, aca, prec):
    """The path a plan starts with by its size, and its products and the ACA
    products' against those of the fused kernels' fewest-columns tile on the
    same plan, three vectors with leading dimensions at once.  Tolerances of
    the two forms' own tests, added."""
    import torch
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import AcaTuckerOperator, TuckerPlan
    S = random_struct(dims, q, m, rmax, 17)
    P = TuckerPlan.from_factors(S.dims, S.q, S.m, *struct_to_abi(S), precision=prec)
    assert tuple(P.info.kernel) == kernels
    g = torch.Generator(device="cuda").manual_seed(8)
    rows = S.q * S.nv
    A = AcaTuckerOperator(P, torch.randn(S.m + 7, S.m, dtype=torch.complex64, device="cuda",
                                         generator=g))
    more = (lib.tv_aca_workspace_bytes(P.handle, 1, 1) -
            lib.tv_workspace_bytes(P.handle, 1, 1)) > 8 * S.m + 255
    assert more == (aca and kernels[1] != 2)
    x = torch.randn(3, S.m + 2, dtype=torch.complex64, device="cuda", generator=g)[:, :S.m].t()
    v = torch.randn(3, A.m, dtype=torch.complex64, device="cuda", generator=g).t()
    y = torch.randn(3, rows + 1, dtype=torch.complex64, device="cuda", generator=g)[:, :rows].t()
    a = P.matvec(x), P.rmatvec(y), A.matvec(v), A.rmatvec(y)
    for op, cap in ((0, 8), (1, 2)):
        lib.tv_plan_configure(P.handle, op, path=0, tile_t2=0, splits=1, row_cap=cap)
    P._ws.clear()
    A._ws.clear()
    b = P.matvec(x), P.rmatvec(y), A.matvec(v), A.rmatvec(y)
    for u, w in zip(a, b):
        assert float((u - w).norm() / w.norm()) < (2e-4 if prec else 2e-5)


@pytest.mark.parametrize("dims,m", [((32, 64, 24), 80), ((64, 64, 64), 80), ((33, 35, 37), 40)])
def test_noalloc_is_rmatvec_on_a_new_plan(gpu_lib, dims, m):
    """Bit for bit, on the GEMM path and on the fused one."""
    import torch
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan
    S = random_struct(dims, 3, m, 8, 73)
    P = TuckerPlan.from_factors(S.dims, S.q, S.m, *struct_to_abi(S))
    y = torch.randn(S.q * S.nv, dtype=torch.complex64, device="cuda",
                    generator=torch.Generator(device="cuda").manual_seed(1))
    x = torch.empty(S.m, dtype=torch.complex64, device="cuda")
    lib.tv_rmatvec_noalloc(P.handle, y.data_ptr(), S.q * S.nv, 1, x.data_ptr(), S.m,
                           torch.cuda.current_stream().cuda_stream)
    assert torch.equal(x, P.rmatvec(y))


def test_adjoint_sums_without_bias_on_smooth_columns(gpu_lib):
    """Smooth positive columns against a random y: rounding errors of either
    sign average out over the 512 chunks and 64 rows, errors of one sign do
    not.  One rounding of the running sum per chunk: 2^-25 sqrt(512) = 6.7e-7
    of a term's partial sum at most, about half that rms, and 2^-23 for the
    factors: 1e-6 of the result."""
    import torch
    from paper_2103_06393_amd import lib
    dims, m = (64, 64, 64), 8
    cores, facs = [], []
    for j in range(m):
        us = []
        for n in dims:
            u = 1.0 + 0.5 * np.cos(np.pi * (np.arange(n) + 0.5) * (j + 1) / (8 * n))
            us.append((u / np.linalg.norm(u)).reshape(n, 1).astype(complex))
        cores.append([np.full((1, 1, 1), 1.0 + 0.25j * j)])
        facs.append([tuple(us)])
    S = om.from_factors(dims, 1, cores, facs)
    P = _plan(S, lib.TV_PREC_FP32, 2)
    rng = np.random.default_rng(3)
    y = (rng.standard_normal(S.nv) + 1j * rng.standard_normal(S.nv)).astype(np.complex64)
    x = P.rmatvec(torch.from_numpy(y).cuda()).cpu().numpy().reshape(-1)
    ref = om.alg2(S, y.astype(np.complex128).reshape(-1, 1)).reshape(-1)
    assert np.linalg.norm(x - ref) <= 1e-6 * np.linalg.norm(ref)
