"""Operands at the ends of FP32's range, infinities and NaN in the split-bf16
GEMM of FP32 plans: tiny operands keep all their bits, products too large for
the scaled planes and non-finite operands give what FP32 products give."""
import warnings

import numpy as np
import pytest

from oracle import matvec as om
from tests.plans import (adj_terms, assert_close, fwd_terms, random_struct, rel_err,
                         struct_to_abi)

pytestmark = pytest.mark.gpu

# (grid, q, columns, largest rank, 64-column units of the tile, splits): 1, 2,
# 5, 8 blocks of rows and two tiles of 7, ragged rows, columns and ranks
SHAPES = [((11, 37, 7), 3, 5, 8, 4, 1), ((32, 19, 14), 1, 9, 8, 2, 2),
          ((80, 16, 17), 2, 13, 9, 4, 1), ((128, 43, 6), 1, 6, 12, 2, 3),
          ((205, 11, 12), 1, 5, 7, 4, 2)]


def _plan(S, abi, nbw, splits, precision=0):
    from paper_2103_06393_amd import lib
    from paper_2103_06393_amd.ops import TuckerPlan
    P = TuckerPlan.from_factors(S.dims, S.q, S.m, *abi, precision=precision)
    for op in (0, 1):
        lib.tv_plan_configure(P.handle, op, path=1, splits=splits, gemm_nbw=nbw)
    return P


def _vectors(S, seed):
    rng = np.random.default_rng(seed)
    cx = lambda n: (rng.standard_normal(n) + 1j * rng.standard_normal(n)).astype(np.complex64)  # noqa: E731
    return cx(S.m), cx(S.q * S.nv)


def _products(P, x, y):
    import torch
    return (P.matvec(torch.from_numpy(x).cuda()).cpu().numpy(),
            P.rmatvec(torch.from_numpy(y).cuda()).cpu().numpy())


@pytest.mark.parametrize("dims,q,m,rmax,nbw,splits", SHAPES)
def test_tiny_vectors_keep_their_bits(gpu_lib, dims, q, m, rmax, nbw, splits):
    """A power of two on x or y changes the result's relative error by no more
    than what FP32 loses below 2^-149: at 2^-116 of vectors near 1 with sums of
    factors above 2^-12 that is 2^-20 of one entry in a thousand."""
    print(f"tiny vectors {dims} q={q} m={m} nbw={nbw} splits={splits}", flush=True)
    S = random_struct(dims, q, m, rmax, 31)
    P = _plan(S, struct_to_abi(S), nbw, splits)
    x, y = _vectors(S, 5)
    ref = om.alg1(S, x)[:, 0], om.alg2(S, y)[:, 0]
    one = [rel_err(a, r) for a, r in zip(_products(P, x, y), ref)]
    s = 2.0 ** -116
    for e, a, r in zip(one, _products(P, (x * s).astype(np.complex64),
                                      (y * s).astype(np.complex64)), ref):
        assert rel_err(a.astype(np.complex128) / s, r) <= 1.05 * e + 1e-9


@pytest.mark.parametrize("dims,q,m,rmax,nbw,splits", SHAPES)
def test_tiny_factors_keep_their_bits(gpu_lib, dims, q, m, rmax, nbw, splits):
    """U1 at 2^-115 (multiples of 2^-135) beside cores at 2^60: every step scales
    exactly."""
    print(f"tiny factors {dims} q={q} m={m} nbw={nbw} splits={splits}", flush=True)
    S = random_struct(dims, q, m, rmax, 32)
    ranks, cores, u1, u2, u3 = struct_to_abi(S)
    u1 = np.round(u1 * 2.0 ** 20) * 2.0 ** -20
    P = _plan(S, (ranks, cores, u1, u2, u3), nbw, splits)
    T = _plan(S, (ranks, cores * 2.0 ** 60, u1 * 2.0 ** -115, u2, u3), nbw, splits)
    x, y = _vectors(S, 6)
    for a, b in zip(_products(P, x, y), _products(T, x, y)):
        assert np.array_equal(b, a * np.float32(2.0 ** -55))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dims,q,m,rmax,nbw,splits", SHAPES)
def test_columns_of_any_size(gpu_lib, dims, q, m, rmax, nbw, splits, precision):
    """Cores from 2^-90 to 2^90, another power of two for each column: the
    adjoint's entries scale with their columns, bit for bit."""
    print(f"columns' sizes {dims} q={q} m={m} nbw={nbw} splits={splits}", flush=True)
    S = random_struct(dims, q, m, rmax, 35)
    e = np.linspace(-90, 90, m).astype(int)
    ranks, cores, u1, u2, u3 = struct_to_abi(S)
    big = np.concatenate([S.t[j][k].G.reshape(-1, order="F") * 2.0 ** float(e[j])
                          for j in range(m) for k in range(q)])
    P = _plan(S, (ranks, cores, u1, u2, u3), nbw, splits, precision)
    T = _plan(S, (ranks, big, u1, u2, u3), nbw, splits, precision)
    x, y = _vectors(S, 9)
    a, b = (_products(Q, x, y)[1] for Q in (P, T))
    assert np.array_equal(b, a * np.float32(2.0) ** e.astype(np.float32))


@pytest.mark.parametrize("scale", [2.0 ** 100, 2.0 ** 118])
@pytest.mark.parametrize("dims,q,m,rmax,nbw,splits", SHAPES)
def test_huge_vectors(gpu_lib, dims, q, m, rmax, nbw, splits, scale):
    """Vectors whose products overflow the scaled planes, all of them or one
    entry: FP32 roundings of modes 3 and 2 (rmax sums each), of 8 products per
    chunk and of the chunks' sum, relative to the moduli of the terms."""
    print(f"huge vectors {dims} q={q} m={m} nbw={nbw} splits={splits}", flush=True)
    S = random_struct(dims, q, m, rmax, 33)
    P = _plan(S, struct_to_abi(S), nbw, splits)
    tol = (2 * rmax + max(rmax * m, dims[1] * dims[2]) / 8 + 16) * 2.0 ** -24
    for some in (False, True):
        x, y = _vectors(S, 7)
        if some:
            x[m // 2] *= scale
            y[len(y) // 3] *= scale
        else:
            x, y = (x * scale).astype(np.complex64), (y * scale).astype(np.complex64)
        f, a = _products(P, x, y)
        x64, y64 = x.astype(np.complex128) / scale, y.astype(np.complex128) / scale
        assert_close(f.astype(np.complex128) / scale, om.alg1(S, x64)[:, 0], tol,
                     terms=fwd_terms(S, x64), what="Z x")
        assert_close(a.astype(np.complex128) / scale, om.alg2(S, y64)[:, 0], tol,
                     terms=adj_terms(S, y64), what="Z^* y")


def _kind(re, im):
    """0 finite, 1 NaN, 2 +inf, 3 -inf."""
    r = np.stack([re, im])
    return np.isnan(r) + 2 * np.isposinf(r) + 3 * np.isneginf(r)


def _mul(ar, ai, br, bi):
    return ar * br - ai * bi, ar * bi + ai * br


def _slab(S, k, j, xr=1.0, xi=0.0):
    """Re and Im of mode 2 and 3 of one tensor, (r1, n2 n3), x_j applied to the
    core after mode 3, in real arithmetic as the kernels do it."""
    t = S.t[j][k]
    H = np.einsum("abc,ic->abi", t.G, t.U[2])
    hr, hi = _mul(xr, xi, H.real, H.imag)
    U = t.U[1]
    pr, pi = _mul(hr[:, :, None, :], hi[:, :, None, :], U.real.T[None, :, :, None],
                  U.imag.T[None, :, :, None])
    r1 = H.shape[0]
    return (pr.sum(1).transpose(0, 2, 1).reshape(r1, -1),
            pi.sum(1).transpose(0, 2, 1).reshape(r1, -1), t.U[0])


@pytest.mark.parametrize("val", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("dims,q,m,rmax,nbw,splits", SHAPES)
def test_non_finite_entries(gpu_lib, dims, q, m, rmax, nbw, splits, val):
    """One non-finite entry of x or y makes the results it reaches infinite or
    NaN as real arithmetic does, and no others."""
    print(f"non-finite {dims} q={q} m={m} nbw={nbw} splits={splits} {val}", flush=True)
    n1, n2, n3 = dims
    S = random_struct(dims, q, m, 1, 34)
    P = _plan(S, struct_to_abi(S), nbw, splits)
    x, y = _vectors(S, 8)
    with warnings.catch_warnings(), np.errstate(all="ignore"):
        warnings.simplefilter("ignore")
        xs, ys = x.copy(), y.copy()
        xs[1] = complex(val, 0.5)
        at = (q - 1) * S.nv + (n1 - 1) + n1 * (n2 * n3 // 2)
        ys[at] = complex(val, -0.5)
        f, a = _products(P, xs, ys)
        wf = np.zeros((2, q, n2 * n3, n1))
        wa = np.zeros((2, m))
        for k in range(q):
            yk = ys.reshape(q, n2 * n3, n1)[k].astype(np.complex128)
            for j in range(m):
                xj = complex(xs[j])
                br, bi, U = _slab(S, k, j, xj.real, xj.imag)
                pr, pi = _mul(br[:, :, None], bi[:, :, None], U.real.T[:, None, :],
                              U.imag.T[:, None, :])
                wf[0, k] += pr.sum(0)
                wf[1, k] += pi.sum(0)
                br, bi, U = _slab(S, k, j)
                # Z = y conj(b), x' = conj(U) Z
                zr = sum(yk.real[n][:, None] * br[:, n] + yk.imag[n][:, None] * bi[:, n]
                         for n in range(n2 * n3))
                zi = sum(yk.imag[n][:, None] * br[:, n] - yk.real[n][:, None] * bi[:, n]
                         for n in range(n2 * n3))
                wa[0, j] += (U.real * zr + U.imag * zi).sum()
                wa[1, j] += (U.real * zi - U.imag * zr).sum()
    assert not np.isfinite(wf).all() and not np.isfinite(wa).all()
    assert np.array_equal(_kind(f.real, f.imag), _kind(*wf.reshape(2, -1)))
    assert np.array_equal(_kind(a.real, a.imag), _kind(*wa))
