"""Performance cases of libtuckvsie: what programs that use the library call.

Each case is one kind of call through the public entry points
(``paper_2103_06393_amd.ops`` and, for batches, ``lib.tv_batch_run``):

* ``matvec`` / ``rmatvec``: Y = Z X (Algorithm 1) or X = Z^* Y (Algorithm 2)
  of one Tucker plan with p right-hand sides, ``grad`` both of them through
  ``TuckerMatvec`` and its backward;
* ``aca_matvec`` / ``aca_rmatvec``: the ACA + Tucker operator U V^* of the
  body-coil grids;
* ``batch``: several coils on one grid with many right-hand sides, both
  directions, through batch objects a program builds once;
* ``compress``: point-current columns to a Tucker plan (columns, truncated
  HOSVD, packing) and its first product;
* ``assemble``: Algorithm 3 (Tucker-based ACA) to an operator and its first
  product.

``tune`` says how the plan's launch configuration was chosen: ``none`` (as
created), ``auto`` (the autotuner ran at set-up) or ``gemm`` (the
decompress-then-GEMM path set with ``tv_plan_configure``, as a program does
that has kept an earlier tuning).  Factors have the form the compression
gives: orthonormal U1..U3 and cores that decay along every mode.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2103_06393_amd import lib
from paper_2103_06393_amd.ops import (AcaTuckerOperator, TuckerMatvec, TuckerPlan,
                                      aca_assemble, batch_create)

C0 = 299_792_458.0


def _case(kind, n, q, m, r1, r2, r3, p=1, prec="fp32", tune="none", coil=0, name=None):
    """r1..r3: (lowest, highest) multilinear rank; coil: coil elements of an
    ACA operator (its V is coil x m), 0 otherwise."""
    c = {"kind": kind, "n1": n[0], "n2": n[1], "n3": n[2], "q": q, "m": m, "p": p,
         "r1lo": r1[0], "r1hi": r1[1], "r2lo": r2[0], "r2hi": r2[1], "r3lo": r3[0],
         "r3hi": r3[1], "prec": prec, "tune": tune, "coil": coil}
    if name:
        c["name"] = name
    return c


def _fields(kind, n, h, freq, operator, m, cap, tol, terms=0, name=None):
    """compress / assemble: m point currents around a box of voxel edge h."""
    c = {"kind": kind, "n1": n[0], "n2": n[1], "n3": n[2], "q": 3, "h": h, "freq": freq,
         "operator": operator, "m": m, "cap": cap, "tol": tol, "terms": terms}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a small head box (32^3, 64 point currents): one product inside an
        # iterative solver, where latency and launches count
        _case("matvec", (32, 32, 32), 3, 64, (6, 12), (6, 12), (6, 12), name="head32_forward"),
        # the smallest work: an odd-sized box and coil, a few vectors at once
        _case("rmatvec", (21, 33, 27), 3, 37, (4, 12), (4, 12), (4, 12), p=4,
              name="odd_box_adjoint_x4"),
        # 64^3 with two rings of 128 elements, tuned at set-up, each direction
        _case("matvec", (64, 64, 64), 3, 256, (7, 10), (7, 10), (8, 13), tune="auto",
              name="rings64_forward"),
        _case("rmatvec", (64, 64, 64), 3, 256, (7, 10), (7, 10), (8, 13), tune="auto",
              name="rings64_adjoint"),
        # a gradient step at 128^3 with piecewise-linear voxels (12 tensors a
        # column): the product and its backward
        _case("grad", (128, 128, 128), 12, 128, (7, 10), (7, 10), (8, 13), tune="gemm",
              name="pwl128_gradient"),
        # the 2 mm body box with its 9450 coil elements in ACA + Tucker form
        _case("aca_matvec", (205, 109, 270), 3, 287, (15, 18), (15, 18), (15, 18), tune="gemm",
              coil=9450, name="body2mm_aca_forward"),
        # the 5 mm body box, piecewise-linear, adjoint, plan as created
        _case("aca_rmatvec", (81, 44, 108), 12, 250, (15, 18), (15, 18), (15, 18), coil=9450,
              name="body5mm_pwl_aca_adjoint"),
        # the largest grid and coil (256^3, 1 mm voxels, 2048 elements), adjoint in FP32
        _case("rmatvec", (256, 256, 256), 3, 2048, (7, 10), (7, 10), (8, 13), tune="gemm",
              name="rings256_adjoint"),
        # the same grid in the BF16 split form, product and backward
        _case("grad", (256, 256, 256), 3, 256, (7, 10), (7, 10), (8, 13), prec="bf16x3",
              tune="gemm", name="rings256_bf16x3_gradient"),
        # several coils on one head grid, 32 excitations each, both directions
        _case("batch", (96, 128, 112), 3, 300, (8, 24), (8, 24), (8, 24), p=32,
              name="coils_batch_x32"),
        # set-up of a plan: 32 point currents on 128^3 compressed at 1e-4
        _fields("compress", (128, 128, 128), 0.002, 298e6, "N", 32, 32, 1e-4,
                name="compress128"),
        # Algorithm 3 on the 5 mm body box: its first terms
        _fields("assemble", (81, 44, 108), 0.005, 123e6, "K", 2000, 0, 1e-3, terms=24,
                name="assemble_body5mm"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["matvec", "matvec", "rmatvec", "rmatvec", "grad", "aca_matvec",
                       "aca_rmatvec", "batch", "compress", "assemble"])
    if kind == "batch":
        n = [rng.randint(20, 128) for _ in range(3)]
        n[0], n[1] = rng.randint(20, 96), n[1] // 8 * 8
        lo = rng.randint(4, 10)
        r = (lo, rng.randint(lo + 2, 16))
        m = max(9, min(rng.randint(24, 300), int(300 * 96 * 128 * 112 / (n[0] * n[1] * n[2]))))
        return _case(kind, n, 3, m, r, r, r, p=rng.randint(9, 32),
                     prec=rng.choice(["fp32", "fp32", "bf16x3"]))
    if kind in ("compress", "assemble"):
        n = [_log_int(rng, 24, 160) for _ in range(3)]
        while n[0] * n[1] * n[2] > 1 << 21:
            n[n.index(max(n))] -= 9
        if kind == "compress":
            return _fields(kind, n, rng.choice([0.001, 0.002, 0.004]), 298e6,
                           rng.choice(["N", "K"]), rng.randint(3, 32), 32, 1e-4)
        while n[0] * n[1] * n[2] > 81 * 44 * 108:
            n[n.index(max(n))] -= 5
        return _fields(kind, n, 0.4 / max(n), 123e6, "K", rng.randint(400, 2000), 0, 1e-3,
                       terms=rng.randint(8, 20))
    # one plan: grids from 16 to 256 voxels a side, odd ones among them
    n = [_log_int(rng, 16, 256) for _ in range(3)]
    nv = n[0] * n[1] * n[2]
    q = rng.choice([3, 3, 12])
    lo = [rng.randint(4, 10) for _ in range(3)]
    if nv > 1 << 20 and rng.random() < 0.5:             # Tucker ranks of an ACA factor U
        lo, n[1] = [15, 15, 15], n[1] // 8 * 8          # odd n2 take at most rank 13
        nv = n[0] * n[1] * n[2]
    r = [(v, v + rng.randint(0, 3)) for v in lo]
    top = int(2e12 / (8.0 * q * nv * r[0][1]))         # well within the largest listed one's work
    m = max(8, min(_log_int(rng, 16, 512), top))
    p = rng.choice([1, 1, 1, 2, 3]) if q * nv * m * r[0][1] < 1 << 35 else 1
    prec = rng.choice(["fp32", "fp32", "fp32", "bf16x3"])
    # a program tunes at set-up or sets the GEMM path on larger grids
    tune = "gemm" if nv > 1 << 19 else rng.choice(["none", "auto"]) if nv < 1 << 17 else "none"
    coil = rng.randint(m, 9450) if kind.startswith("aca") else 0
    return _case(kind, n, q, m, *r, p=1 if kind == "grad" else p, prec=prec, tune=tune, coil=coil)


# ---- inputs -----------------------------------------------------------------

def _normal(shape, gen):
    """CN(0, 1), complex128 on the GPU."""
    z = torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=gen)
    return torch.view_as_complex(z) * math.sqrt(0.5)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _ranks(case, m):
    """(m, q, 3) multilinear ranks: a property of the case, not of the seed."""
    rng = np.random.default_rng([case["n1"], case["n2"], case["n3"], case["q"], m])
    return np.stack([rng.integers(case[f"r{d}lo"], case[f"r{d}hi"] + 1, size=(m, case["q"]))
                     for d in (1, 2, 3)], axis=-1).astype(np.int32)


def _orthonormal(T, n, r, gen):
    """T sets of r orthonormal vectors of length n, (T, r, n): block
    Gram-Schmidt with one repetition."""
    A = _normal((T, r, n), gen)
    for a in range(r):
        v = A[:, a]
        for _ in range(2 if a else 0):
            c = torch.matmul(A[:, :a].conj(), v[:, :, None])
            v = v - torch.matmul(A[:, :a].transpose(1, 2).contiguous(), c)[:, :, 0]
        A[:, a] = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
    return A


def _factors(case, m, gen):
    """Padded factors on the GPU in tensor order t = k + q j: cores
    (T, R3, R2, R1), U_n (T, R_n, n_n); entries past a tensor's ranks are 0."""
    T = m * case["q"]
    rk = torch.from_numpy(_ranks(case, m).reshape(T, 3)).cuda()
    R = [int(v) for v in rk.amax(0)]
    ax = [torch.arange(v, device="cuda") for v in R]
    ok = [ax[d][None, :] < rk[:, d:d + 1] for d in range(3)]
    live = ok[2][:, :, None, None] & ok[1][:, None, :, None] & ok[0][:, None, None, :]
    e = ax[2][:, None, None] + ax[1][None, :, None] + ax[0][None, None, :]
    G = _normal((T, R[2], R[1], R[0]), gen) * (10.0 ** (-0.25 * e))
    G = torch.where(live, G, torch.zeros_like(G))
    U = []
    for d in range(3):
        u = _orthonormal(T, case[f"n{d + 1}"], R[d], gen)
        U.append(torch.where(ok[d][:, :, None], u, torch.zeros_like(u)))
    return rk, live, ok, G, U


def _plan(case, m, gen):
    """The plan a program builds from its factors, and its launch configuration."""
    rk, live, ok, G, U = _factors(case, m, gen)
    dims = (case["n1"], case["n2"], case["n3"])
    host = [G[live].cpu().numpy()] + [u[k].reshape(-1).cpu().numpy() for u, k in zip(U, ok)]
    prec = lib.TV_PREC_BF16X3 if case["prec"] == "bf16x3" else lib.TV_PREC_FP32
    plan = TuckerPlan.from_factors(dims, case["q"], m, rk.cpu().numpy(), *host, precision=prec)
    if case["tune"] == "auto":
        plan.autotune()
    elif case["tune"] == "gemm":
        lib.tv_plan_configure(plan.handle, 0, path=1, splits=1, gemm_nbw=4)
        lib.tv_plan_configure(plan.handle, 1, path=1, splits=16, gemm_nbw=4)
    return plan


def _batch_sizes(case):
    """Columns of the batch's three coils, 0.4 to 1 times m."""
    return [case["m"], max(1, case["m"] * 7 // 10), max(1, case["m"] * 2 // 5)]


def _vec(rows, p, gen):
    """A complex64 operand as programs hold it: (rows,) or column-major (rows, p)."""
    v = _normal((p, rows), gen).to(torch.complex64)
    return v[0] if p == 1 else v.t()


def _sources(case, seed):
    """Point currents on a cylinder around the box, tangential, seeded."""
    rng = np.random.default_rng([seed, case["m"]])
    half = [case[f"n{d}"] * case["h"] / 2 for d in (1, 2, 3)]
    rad = 1.3 * math.hypot(half[0], half[1])
    phi = rng.uniform(0, 2 * math.pi, case["m"])
    z = rng.uniform(-1.5 * half[2], 1.5 * half[2], case["m"])
    a = rng.uniform(0, 2 * math.pi, case["m"])
    pos = np.stack([rad * np.cos(phi), rad * np.sin(phi), z], 1)
    ori = np.stack([-np.cos(a) * np.sin(phi), np.cos(a) * np.cos(phi), np.sin(a)], 1)
    return pos, ori


def prepare(case, seed):
    gen = _gen(seed)
    kind = case["kind"]
    nv = case["n1"] * case["n2"] * case["n3"]
    s = {"case": case, "kind": kind}
    if kind in ("compress", "assemble"):
        s["pos"], s["ori"] = _sources(case, seed)
        s["x"] = _vec(case["m"], 1, gen)
        return s
    if kind == "batch":
        ms, p = _batch_sizes(case), case["p"]
        s["plans"] = [_plan(case, m, gen) for m in ms]
        s["x"] = [_vec(m, p, gen) for m in ms]
        s["y"] = [_vec(case["q"] * nv, p, gen) for m in ms]
        handles = [P.handle for P in s["plans"]]
        s["batch"] = [batch_create(handles, op, [p] * len(ms)) for op in (0, 1)]
        s["ws"] = [torch.empty(lib.tv_batch_workspace_bytes(b), dtype=torch.uint8, device="cuda")
                   for b, _ in s["batch"]]
        return s
    s["plan"] = _plan(case, case["m"], gen)
    rows_x = case["coil"] or case["m"]
    if case["coil"]:
        V = _normal((case["coil"], case["m"]), gen).to(torch.complex64)
        s["op"] = AcaTuckerOperator(s["plan"], V)
    if kind in ("matvec", "aca_matvec", "grad"):
        s["x"] = _vec(rows_x, case["p"], gen)
    if kind in ("rmatvec", "aca_rmatvec", "grad"):
        s["y"] = _vec(case["q"] * nv, case["p"], gen)
    if kind == "grad":
        s["x"].requires_grad_(True)
    return s


# ---- one pass ---------------------------------------------------------------

def _batch_run(state, op, inputs, rows):
    p = state["case"]["p"]
    out = [torch.empty((p, r), dtype=torch.complex64, device="cuda").t() for r in rows]
    ws = state["ws"][op]
    lib.tv_batch_run(state["batch"][op][0], [v.data_ptr() for v in inputs],
                     [v.stride(1) for v in inputs], [v.data_ptr() for v in out],
                     [v.stride(1) for v in out], ws.data_ptr(), ws.numel(),
                     torch.cuda.current_stream().cuda_stream)
    return out


def run(state):
    kind, c = state["kind"], state["case"]
    if kind == "matvec":
        return state["plan"].matvec(state["x"])
    if kind == "rmatvec":
        return state["plan"].rmatvec(state["y"])
    if kind == "grad":
        y = TuckerMatvec.apply(state["x"], state["plan"])
        g, = torch.autograd.grad(y, state["x"], state["y"])
        return {"y": y.detach(), "grad": g}
    if kind == "aca_matvec":
        return state["op"].matvec(state["x"])
    if kind == "aca_rmatvec":
        return state["op"].rmatvec(state["y"])
    if kind == "batch":
        return {"y": _batch_run(state, 0, state["x"], [P.rows for P in state["plans"]]),
                "x": _batch_run(state, 1, state["y"], [P.m for P in state["plans"]])}
    dims = (c["n1"], c["n2"], c["n3"])
    k0 = 2 * math.pi * c["freq"] / C0
    basis = lib.field_code("pwc", c["operator"])
    if kind == "compress":
        plan = TuckerPlan.compress_dipoles(dims, c["h"], k0, basis, state["pos"], state["ori"],
                                           c["tol"], 1, c["cap"])
        out = {"ranks": plan.export_factors()[0], "y": plan.matvec(state["x"])}
        plan.close()
        return out
    op, info = aca_assemble(dims, c["h"], k0, basis, state["pos"], state["ori"], c["tol"],
                            max_terms=c["terms"])
    return {"rc": info["rc"], "pivots": info["pivots"], "v": op.Vc, "y": op.matvec(state["x"])}


# ---- the floor of one pass --------------------------------------------------

def _plan_work(case, m):
    """(factor bytes, flops of one product) of a plan: complex64 factors, and
    modes 2, 3 and 1 of every tensor in real multiply-adds."""
    r = _ranks(case, m).reshape(-1, 3).astype(np.float64)
    n1, n2, n3 = case["n1"], case["n2"], case["n3"]
    fb = 8.0 * np.sum(r[:, 0] * r[:, 1] * r[:, 2] + n1 * r[:, 0] + n2 * r[:, 1] + n3 * r[:, 2])
    dec = r[:, 0] * r[:, 1] * r[:, 2] * n3 + r[:, 0] * r[:, 1] * n2 * n3
    return float(fb), 8.0 * float(np.sum(dec)), 8.0 * float(np.sum(r[:, 0])) * n1 * n2 * n3


def work(case):
    nv = case["n1"] * case["n2"] * case["n3"]
    rows = case["q"] * nv
    if case["kind"] in ("compress", "assemble"):
        # Gram matrices of the three unfoldings (Hermitian: half of them) of
        # every compressed column; the columns need not exist in memory
        cols = case["terms"] or case["m"]
        n = case["n1"] + case["n2"] + case["n3"]
        fl = 4.0 * rows * n * cols
        if case["terms"]:       # and the two products with U per term
            fl += 2 * 8.0 * 8.0 * rows * cols * cols / 2
        return {"bytes": 8.0 * (rows + case["m"] * (1 + case["terms"])), "flops": fl}
    p = case["p"]
    if case["kind"] == "batch":
        w = {"bytes": 0.0, "flops": 0.0}
        for m in _batch_sizes(case):
            fb, dec, mode1 = _plan_work(case, m)
            # both directions: decompress once, apply to the p vectors
            w["bytes"] += 2 * (fb + 8.0 * p * (rows + m))
            w["flops"] += 2 * (dec + mode1 + 8.0 * rows * m * p)
        return w
    fb, dec, mode1 = _plan_work(case, case["m"])
    b = fb + 8.0 * p * (rows + case["m"])
    fl = dec + p * mode1
    if case["coil"]:
        b += 8.0 * case["coil"] * (case["m"] + p)
        fl += 8.0 * case["coil"] * case["m"] * p
    k = 2 if case["kind"] == "grad" else 1
    return {"bytes": k * b, "flops": k * fl}


# ---- the results in 64 bits -------------------------------------------------

def _dense_columns(case, m, gen):
    """Yields (j0, Z block (cols, q, nv)) of the dense matrix, complex128."""
    _, _, _, G, U = _factors(case, m, gen)
    q, n1, n2, n3 = case["q"], case["n1"], case["n2"], case["n3"]
    step = max(1, int((8 << 30) // (16 * q * n1 * n2 * n3)))
    R3, R2, R1 = G.shape[1:]
    for j0 in range(0, m, step):
        j1 = min(m, j0 + step)
        t = slice(q * j0, q * j1)
        g = G[t]
        T = g.shape[0]
        # modes 3, 2, 1: (T, n3, n2, n1) = U3^T (U2^T (U1^T G))
        h = torch.matmul(U[2][t].transpose(1, 2).contiguous(), g.reshape(T, R3, R2 * R1))
        h = torch.matmul(U[1][t].transpose(1, 2).contiguous()[:, None],
                         h.reshape(T, n3, R2, R1))
        h = torch.matmul(h.reshape(T, n3 * n2, R1), U[0][t])
        yield j0, h.reshape(j1 - j0, q, n1 * n2 * n3)


def _exact_products(case, m, gen, x, y):
    """Z x (rows, p) and Z^* y (m, p) for the operands that are not None."""
    rows = case["q"] * case["n1"] * case["n2"] * case["n3"]
    Y = torch.zeros(rows, x.shape[1], dtype=torch.complex128, device="cuda") if x is not None else None
    X = torch.zeros(m, y.shape[1], dtype=torch.complex128, device="cuda") if y is not None else None
    for j0, Z in _dense_columns(case, m, gen):
        Z = Z.reshape(Z.shape[0], rows)
        j1 = j0 + Z.shape[0]
        if x is not None and x.shape[1] > 4:
            Y += torch.matmul(Z.t().contiguous(), x[j0:j1])
        elif x is not None:
            for c in range(x.shape[1]):
                Y[:, c] += (Z * x[j0:j1, c:c + 1]).sum(0)
        if y is not None and y.shape[1] > 4:
            X[j0:j1] = torch.matmul(Z.conj_physical(), y)
        elif y is not None:
            for c in range(y.shape[1]):
                X[j0:j1, c] = (Z.conj_physical() * y[:, c]).sum(1)
    return Y, X


def _wide(v):
    v = v.to(torch.complex128)
    return v[:, None] if v.dim() == 1 else v


def _fields_product(case, seed, x):
    """Z x of the point currents' dense columns, field operator N (eq. 2) or
    K (eq. 5) at the voxel centres."""
    pos, ori = _sources(case, seed)
    k0 = 2 * math.pi * case["freq"] / C0
    n = [case["n1"], case["n2"], case["n3"]]
    ax = [(torch.arange(v, dtype=torch.float64, device="cuda") - (v - 1) / 2) * case["h"] for v in n]
    z, y, x1 = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    pts = torch.stack([x1.reshape(-1), y.reshape(-1), z.reshape(-1)])
    out = torch.zeros(3, pts.shape[1], dtype=torch.complex128, device="cuda")
    for j in range(case["m"]):
        d = pts - torch.from_numpy(pos[j]).cuda()[:, None]
        pj = torch.from_numpy(ori[j]).cuda()[:, None]
        R = torch.sqrt((d * d).sum(0))
        u = d / R
        kr = k0 * R
        g = torch.polar(1 / (4 * math.pi * R), -kr)
        if case["operator"] == "K":
            dg = g * torch.complex(-1 / R, -k0 * torch.ones_like(R))
            col = dg * torch.linalg.cross(u, pj.expand_as(u), dim=0)
        else:
            a = torch.complex(1 - 1 / kr ** 2, -1 / kr)
            b = torch.complex(-1 + 3 / kr ** 2, 3 / kr)
            col = k0 * k0 * g * (a * pj + b * (u * pj).sum(0) * u)
        out += x[j] * col
    return out.reshape(-1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "assemble":
        return None
    gen = _gen(seed)
    if kind == "compress":
        return {"ranks": None,
                "y": _fields_product(case, seed, _vec(case["m"], 1, gen).to(torch.complex128))}
    nv = case["n1"] * case["n2"] * case["n3"]
    rows = case["q"] * nv
    if kind == "batch":
        # the seed's values come in the order of prepare(): every plan's
        # factors, then the operands; the factors are made again from there
        ms, p = _batch_sizes(case), case["p"]
        states = []
        for m in ms:
            states.append(gen.get_state())
            _factors(case, m, gen)
        xs = [_wide(_vec(m, p, gen)) for m in ms]
        ys = [_wide(_vec(rows, p, gen)) for m in ms]
        out = {"y": [], "x": []}
        for m, st, x, y in zip(ms, states, xs, ys):
            gen.set_state(st)
            Y, X = _exact_products(case, m, gen, x, y)
            out["y"].append(Y)
            out["x"].append(X)
        return out
    m, p = case["m"], case["p"]
    start = gen.get_state()
    _factors(case, m, gen)
    V = _normal((case["coil"], m), gen).to(torch.complex64).to(torch.complex128) if case["coil"] else None
    x = y = None
    if kind in ("matvec", "aca_matvec", "grad"):
        x = _wide(_vec(case["coil"] or m, p, gen))
        if V is not None:
            x = torch.matmul(V.conj().t().contiguous(), x)
    if kind in ("rmatvec", "aca_rmatvec", "grad"):
        y = _wide(_vec(rows, p, gen))
    gen.set_state(start)
    Y, X = _exact_products(case, m, gen, x, y)
    if V is not None and X is not None:
        X = torch.matmul(V, X)
    Y, X = (v if v is None or p > 1 else v[:, 0] for v in (Y, X))
    if kind == "grad":
        return {"y": Y, "grad": X}
    return Y if kind in ("matvec", "aca_matvec") else X
