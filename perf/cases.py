"""Workloads of the preconditioner's users, for timing and for comparing results.

``listed()`` names the fixed ones, ``draw(rng)`` gives others of the same
ranges; ``prepare`` builds what a user's program holds before the call
(matrix, handle, right-hand sides; seeded), ``run`` is one pass through the
public entry points, ``work`` its unavoidable bytes and operations, and
``exact`` the values it should return, in FP64 by plain tensor operations.

A case is one of five calls:

* ``apply``     z = M^{-1} r with a kept handle (a caller with its own Krylov
                method);
* ``solve``     one preconditioned CG / GMRES solve on a kept handle;
* ``refactor``  numeric re-setup with new matrix values, then one solve (a
                time step or a Newton step);
* ``batch``     CG on several independent problems packed in one handle;
* ``serve``     the serving loop on a full queue of right-hand sides.

Cases that only apply use FP64 factors: with reduced factors an apply is
defined to the factors' rounding only, while the solves converge to the same
solution, so the reduced precisions are covered by those.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2304_04876_amd import binding as B
from paper_2304_04876_amd import problems as P
from paper_2304_04876_amd import serve as S

PREC = {"fp64": B.FP64, "fp32": B.FP32, "bf16": B.BF16, "fp16": B.FP16}
SIZE = {"fp64": 8, "fp32": 4, "bf16": 2, "fp16": 2}
COARSE = {"gdsw": B.COARSE_GDSW, "rgdsw": B.COARSE_RGDSW}
KRYLOV = {"cg": B.KRYLOV_CG, "gmres": B.KRYLOV_GMRES, "gmres_sr": B.KRYLOV_GMRES_SR}
LOCAL = {"ilu": (B.LOCAL_ILU0, B.ORDER_NATURAL), "band": (B.LOCAL_EXACT, B.ORDER_NATURAL),
         "nd": (B.LOCAL_EXACT, B.ORDER_ND), "auto": (B.LOCAL_EXACT, B.ORDER_AUTO)}


def listed():
    return [
        # the smallest call: the 20^3 workload with the default options, no tuning
        _case("apply", "poisson", 20, 2, "band", name="apply_poisson20_exact"),
        # the preconditioner alone inside a caller's own Krylov method, full-size workload
        _case("apply", "poisson", 128, 8, "ilu", tuned=True, name="apply_poisson128_ilu0"),
        # the same with exact local solves (supernodal factors)
        _case("apply", "poisson", 128, 8, "nd", tuned=True, name="apply_poisson128_nd"),
        # the full-size solve: GDSW-PCG, ILU(0) by 5 + 5 Jacobi sweeps
        _case("solve", "poisson", 128, 8, "ilu", tuned=True, name="solve_poisson128_ilu0"),
        # a ragged grid (boxes of 17 and 18 nodes) with fill: ILU(2) by FastILU
        _case("solve", "poisson", 87, 5, "ilu", level=2, fast=3, tuned=True, name="solve_poisson87_ilu2"),
        # elasticity as in the paper: FP32 exact local solves, reduced coarse space,
        # single-reduce GMRES(30)
        _case("solve", "elasticity", 48, 6, "band", prec="fp32", coarse="rgdsw", krylov="gmres_sr", tuned=True,
              name="solve_elasticity48_fp32"),
        # many small independent problems in one handle, FP32 supernodal factors
        _case("batch", "diffusion", 48, 4, "nd", prec="fp32", count=16, tuned=True, name="batch16_diffusion_nd_fp32"),
        # serving: four resident operators, FP16 ILU(0), four slots each, a full queue
        _case("serve", "poisson", 59, 4, "ilu", prec="fp16", count=32, tuned=True, name="serve_poisson32to59_fp16"),
        # a time step of a reaction-diffusion problem: new values, ILU(0), one solve
        _case("refactor", "poisson", 128, 8, "ilu", name="refactor_poisson128_ilu0"),
        # the same with exact FP64 supernodal factors
        _case("refactor", "poisson", 96, 6, "nd", name="refactor_poisson96_nd"),
        # the same with FP32 band factors on odd boxes (12 to 13 nodes)
        _case("refactor", "poisson", 75, 6, "band", prec="fp32", name="refactor_poisson75_band_fp32"),
        # an implicit step of elastodynamics: FP32 band factors, GDSW space with rotations
        _case("refactor", "elasticity", 24, 3, "band", prec="fp32", krylov="gmres_sr",
              name="refactor_elasticity24_fp32"),
    ]


def _case(kind, problem, N, boxes, local, prec="fp64", coarse="gdsw", krylov="cg", level=0, fast=0, count=1,
          tuned=False, name=None):
    c = dict(kind=kind, problem=problem, N=N, boxes=boxes, local=local, prec=prec, coarse=coarse, krylov=krylov,
             level=level, fast=fast, count=count, tuned=tuned)
    if name:
        c["name"] = name
    return c


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["apply", "apply", "solve", "solve", "refactor", "refactor", "batch", "serve"])
    tuned = rng.random() < 0.5
    prec = rng.choice(["fp64", "fp64", "fp32", "fp16", "bf16"])
    if kind == "apply":
        N = _log_int(rng, 12, 100)
        return _case(kind, "poisson", N, max(2, round(N / rng.uniform(10, 18))), rng.choice(["ilu", "band", "nd"]),
                     tuned=tuned)
    low = "fp16" if prec == "bf16" else prec   # (BF16 with exact factors, which stay symmetric)
    if kind == "batch":
        local = rng.choice(["nd", "auto", "ilu"])
        return _case(kind, "diffusion", rng.randint(24, 48), rng.randint(2, 4), local,
                     prec=low if local == "ilu" else prec, count=rng.randint(3, 16), tuned=tuned)
    if kind == "serve":
        return _case(kind, "poisson", rng.randint(36, 64), 4, "ilu", prec=low, count=rng.randint(8, 32), tuned=True)
    if rng.random() < 0.3:
        Ne = rng.randint(8, 24)
        return _case(kind, "elasticity", Ne, max(2, round(Ne / 8)), rng.choice(["band", "nd", "auto"]),
                     prec=rng.choice(["fp64", "fp32"]), coarse=rng.choice(["gdsw", "rgdsw"]),
                     krylov=rng.choice(["cg", "gmres", "gmres_sr"]), tuned=tuned)
    local = rng.choice(["ilu", "ilu", "nd", "band"])
    level = rng.choice([0, 0, 1, 2]) if local == "ilu" else 0
    prec = low if local == "ilu" else prec
    N = _log_int(rng, 32, 96)
    return _case(kind, "poisson", N, max(2, round(N / rng.uniform(12, 18))), local, prec=prec,
                 coarse=rng.choice(["gdsw", "gdsw", "rgdsw"]), krylov=rng.choice(["cg", "cg", "gmres", "gmres_sr"]),
                 level=level, fast=rng.choice([0, 3]) if level else 0, tuned=tuned)


# ---------------------------------------------------------------------------
# inputs

@functools.lru_cache(maxsize=6)
def _problem(problem, N, boxes):
    """The matrix (the same for every seed), its partition and null space."""
    if problem == "elasticity":
        pr = P.elasticity_q1(N, boxes)
        return pr, P.rigid_body_modes(pr)
    return P.poisson3d(N, boxes), None


def _options(case):
    local, order = LOCAL[case["local"]]
    return dict(local=local, exact_order=order, local_prec=PREC[case["prec"]], coarse=COARSE[case["coarse"]],
                basis_prec=B.FP64 if case["prec"] == "fp64" else B.FP32, ilu_level=case["level"],
                ilu_factor_sweeps=case["fast"])


def _new_values(A, seed):
    """A plus a nonnegative diagonal (a reaction or mass term): CSR values."""
    rng = np.random.default_rng(seed + 7)
    val = A.data.copy()
    rows = np.repeat(np.arange(A.shape[0], dtype=np.int32), np.diff(A.indptr))
    at = np.flatnonzero(A.indices == rows)
    val[at] *= rng.uniform(1.0, 1.1, at.size)
    return val


def _serve_sizes(case):
    """The serving stream's sizes up to the case's (32, 41, 50, 59, ...)."""
    return [n for n in P.SERVE_SIZES if n < case["N"]] + [case["N"]]


def _batch_sizes(case):
    rng = np.random.default_rng(2304 + case["N"])
    return [(int(rng.integers(16, case["N"] + 1)), int(rng.integers(2, case["boxes"] + 1)))
            for _ in range(case["count"])]


def _batch_kappa(case, seed):
    rng = np.random.default_rng([seed, 11])
    return [(N, p, np.exp(rng.standard_normal((N + 1) ** 3)), rng.uniform(-1.0, 1.0, N ** 3))
            for N, p in _batch_sizes(case)]


def _serve_rhs(case, seed):
    sizes = _serve_sizes(case)
    return [(k % len(sizes), P.rhs_uniform(sizes[k % len(sizes)] ** 3, 1000 * seed + k)) for k in range(case["count"])]


class _Handle:
    """A library handle, destroyed with the object."""

    def __init__(self, h):
        self.h = h

    def __del__(self):
        B.gdsw_destroy(self.h)


class _Server(S.Server):
    def __del__(self):
        self.close()


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "serve":
        o = _options(case)
        ops = [_problem("poisson", n, max(2, round(n / 16)))[0] for n in _serve_sizes(case)]
        st["server"] = _Server(ops, slots_per_op=4, local_prec=o["local_prec"], basis_prec=o["basis_prec"])
        st["rhs"] = _serve_rhs(case, seed)
        return st
    if kind == "batch":
        specs = _batch_kappa(case, seed)
        prs = [P.diffusion3d(N, kappa, p) for N, p, kappa, _ in specs]
        st["handle"] = _Handle(B.gdsw_analyze_batch([(q.A, q.part, q.n_parts) for q in prs],
                                                    options=B.gdsw_default_options(**_options(case))))
        B.gdsw_factor(st["handle"].h)
        b = np.concatenate([s[3] for s in specs])
    else:
        pr, Z = _problem(case["problem"], case["N"], case["boxes"])
        st["handle"] = B.Gdsw(pr.A, pr.part, pr.n_parts, pr.dpn, Z, **_options(case))
        b = P.rhs_uniform(pr.n, seed)
        if kind == "refactor":
            st["values"] = _new_values(pr.A, seed)
    if case["tuned"]:
        B.gdsw_autotune(st["handle"].h, reps=3)
    st["b"] = torch.from_numpy(b).cuda()
    st["x"] = torch.zeros_like(st["b"])
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "serve":
        reqs = [S.Request(rid=k, op=op, arrival=0.0, b=b) for k, (op, b) in enumerate(state["rhs"])]
        _, sol = state["server"].run(reqs, keep_solutions=True)
        return [sol[k] for k in range(len(reqs))]
    h, b, x = state["handle"].h, state["b"], state["x"]
    if kind == "apply":
        B.gdsw_apply(h, b, x)
    elif kind == "batch":
        B.gdsw_solve_batch(h, b, x)
    else:
        if kind == "refactor":
            B.gdsw_refactor(h, state["values"])
        B.gdsw_solve(h, b, x, krylov=KRYLOV[case["krylov"]])
    return x


# ---------------------------------------------------------------------------
# bytes and operations no form of the path can do without: matrix values and
# vectors, the stored factor values and the coarse basis read once per apply
# (exact factors: the entries of a fill-reducing order), per Krylov iteration
# one product, one apply and the vector updates; for a re-setup the values
# read once, the factors written once and the operations of the factorization

def work(case):
    s = SIZE[case["prec"]]
    kind = case["kind"]
    if kind == "serve":
        sizes = _serve_sizes(case)
        one = [_apply_work(case, n ** 3, n, max(2, round(n / 16)), 1, 7, s) for n in sizes]
        return {"bytes": sum(70 * one[k % len(sizes)][0] for k in range(case["count"])),
                "flops": sum(70 * one[k % len(sizes)][1] for k in range(case["count"]))}
    if kind == "batch":
        one = [_apply_work(case, N ** 3, N, p, 1, 7, s) for N, p in _batch_sizes(case)]
        return {"bytes": 33 * sum(o[0] for o in one), "flops": 33 * sum(o[1] for o in one)}
    elastic = case["problem"] == "elasticity"
    N = case["N"]
    dpn, stencil = (3, 78) if elastic else (1, 7)
    n = 3 * N * (N + 1) ** 2 if elastic else N ** 3
    nb, nf = _apply_work(case, n, N, case["boxes"], dpn, stencil, s, kind != "apply")
    if kind == "apply":
        return {"bytes": nb, "flops": nf}
    iters = 55 if elastic else 70 if case["local"] == "ilu" else 44
    nb, nf = iters * nb, iters * nf
    if kind == "refactor":
        rows, entries, ops = _factor_size(case, N, case["boxes"], dpn)
        nb += 8 * n * stencil + entries * s
        nf += ops
    return {"bytes": int(nb), "flops": int(nf)}


def _factor_size(case, N, boxes, dpn):
    """(local rows, stored factor entries, operations of the factorization)."""
    m = N / boxes
    rows = dpn * ((m + 2) ** 3 if dpn == 3 else m ** 3 + 6 * m * m)
    if case["local"] == "ilu":
        per = (6, 12, 22, 42)[min(case["level"], 3)]
        entries, ops = rows * (per + 1), rows * per * per
    else:
        entries = min(6.1 * dpn * rows ** (4 / 3), rows * (dpn * (m + 2) ** 2))
        ops = entries * entries / rows
    k = boxes ** 3
    return k * rows, k * entries, k * ops


def _apply_work(case, n, N, boxes, dpn, stencil, s, krylov=True):
    rows, entries, _ = _factor_size(case, N, boxes, dpn)
    basis = 6 * (15 if dpn == 3 else 1) * n
    nb = entries * s + 16 * n + 4 * rows + basis * min(s, 8 if s == 8 else 4)
    nf = 4 * entries + 4 * basis
    if krylov:
        nb += 10 * n * stencil + 72 * n
        nf += 2 * n * stencil + 12 * n
    return int(nb), int(nf)


# ---------------------------------------------------------------------------
# the values in FP64, without the library

def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "serve":
        sizes = _serve_sizes(case)
        return [_poisson_solve(torch.from_numpy(b).to(dev), sizes[op]) for op, b in _serve_rhs(case, seed)]
    if kind == "batch":
        out = []
        for N, p, kappa, b in _batch_kappa(case, seed):
            out.append(_cg_solve(P.diffusion3d(N, kappa, p).A, None, b, dev))
        return torch.cat(out)
    pr, _ = _problem(case["problem"], case["N"], case["boxes"])
    b = P.rhs_uniform(pr.n, seed)
    if kind == "apply":
        return _grid_apply(case["N"], case["boxes"], case["local"] == "ilu", torch.from_numpy(b).to(dev))
    if kind == "refactor":
        return _cg_solve(pr.A, _new_values(pr.A, seed), b, dev)
    if case["problem"] == "poisson":
        return _poisson_solve(torch.from_numpy(b).to(dev), case["N"])
    return _cg_solve(pr.A, None, b, dev)


def _poisson_solve(b, N):
    """The 7-point system by sine transforms."""
    k = torch.arange(1, N + 1, dtype=torch.float64, device=b.device)
    Q = torch.sin(math.pi * k[:, None] * k[None, :] / (N + 1)) * math.sqrt(2.0 / (N + 1))
    lam = 2.0 - 2.0 * torch.cos(math.pi * k / (N + 1))

    def transform(v):
        for _ in range(3):   # each axis in turn
            v = (v.reshape(N * N, N) @ Q).reshape(N, N, N).permute(2, 0, 1).contiguous()
        return v

    v = transform(b.reshape(N, N, N)) / (lam[:, None, None] + lam[None, :, None] + lam[None, None, :])
    return transform(v).reshape(-1)


def _pcg(op, b, dinv, tol=1e-14, maxit=3000):
    """Jacobi-preconditioned CG on the tensor operator `op`."""
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rz, bb = z.clone(), (r * z).sum(), float((b * b).sum())
    for k in range(maxit):
        q = op(p)
        a = rz / (p * q).sum()
        x += a * p
        r -= a * q
        if k % 10 == 9 and float((r * r).sum()) <= tol * tol * bb:
            break
        z = dinv * r
        new = (r * z).sum()
        p = z + (new / rz) * p
        rz = new
    return x


def _cg_solve(A, val, b, dev):
    n = A.shape[0]
    cnt = np.diff(A.indptr)
    w = int(cnt.max())
    at = np.arange(A.nnz) - np.repeat(A.indptr[:-1], cnt) + w * np.repeat(np.arange(n, dtype=np.int64), cnt)
    col, v = np.zeros(n * w, dtype=np.int64), np.zeros(n * w)
    col[at], v[at] = A.indices, A.data if val is None else val
    dinv = np.ones(n)
    rows = np.repeat(np.arange(n), cnt)
    on = A.indices == rows
    dinv[rows[on]] = 1.0 / (A.data if val is None else val)[on]
    col = torch.from_numpy(col.reshape(n, w).T.copy()).to(dev)
    v = torch.from_numpy(v.reshape(n, w).T.copy()).to(dev)

    def op(x):
        y = torch.zeros_like(x)
        for k in range(w):
            y += v[k] * x[col[k]]
        return y

    return _pcg(op, torch.from_numpy(b).to(dev), torch.from_numpy(dinv).to(dev))


def _grid_apply(N, boxes, ilu, r):
    """Eq. (1) for the 7-point Laplacian (6, -1) on boxes of the N^3 grid,
    overlap one, GDSW space with the constants, written on the grid itself."""
    dev = r.device
    g = torch.arange(N, device=dev)
    box = torch.clamp((g + 1) * boxes // (N + 1), max=boxes - 1)
    start = torch.searchsorted(box, torch.arange(boxes, device=dev))
    end = torch.searchsorted(box, torch.arange(boxes, device=dev), right=True)
    r3 = r.reshape(N, N, N)

    def laplace(v, m):
        """6 v - neighbours on tensors [..., z, y, x], neighbours masked by m."""
        u = v * m
        y = 6.0 * v
        for d in (-3, -2, -1):
            k = u.shape[d]
            y.narrow(d, 1, k - 1).sub_(u.narrow(d, 0, k - 1))
            y.narrow(d, 0, k - 1).sub_(u.narrow(d, 1, k - 1))
        return y * m

    # ---- one level: every box with one layer, padded to the largest
    size = int((end - start).max()) + 2
    off = torch.arange(size, device=dev) - 1
    pos = start[:, None] + off[None, :]                        # [boxes, size] grid index per axis
    inside = pos < end[:, None]
    inside &= off[None, :] >= 0
    layer = ((pos == start[:, None] - 1) | (pos == end[:, None])) & (pos >= 0) & (pos < N)
    pos = pos.clamp(0, N - 1)

    def axes(t):
        return t[:, None, None, :, None, None], t[None, :, None, None, :, None], t[None, None, :, None, None, :]

    iz, iy, ix = axes(inside)
    lz, ly, lx = axes(layer)
    mask = (iz & iy & ix) | (lz & iy & ix) | (iz & ly & ix) | (iz & iy & lx)
    pz, py, px = axes(pos)
    idx = (pz * (N * N) + py * N + px).reshape(-1, size, size, size)
    m = mask.reshape(-1, size, size, size).to(torch.float64)
    loc = r[idx] * m
    if ilu:
        # ILU(0) of the 7-point stencil changes the pivots alone
        d = torch.full_like(loc, 6.0)
        s = off[:, None, None] + off[None, :, None] + off[None, None, :] + 3
        for lev in range(3 * size - 2):
            low = torch.zeros_like(d)
            inv = m / d
            for dim in (-3, -2, -1):
                low.narrow(dim, 1, size - 1).add_(inv.narrow(dim, 0, size - 1))
            d = torch.where((s == lev).expand_as(d), 6.0 - low, d)
        y = torch.zeros_like(loc)
        for _ in range(5):
            u, t = m * y / d, loc.clone()
            for dim in (-3, -2, -1):
                t.narrow(dim, 1, size - 1).add_(u.narrow(dim, 0, size - 1))
            y = t * m
        z = torch.zeros_like(loc)
        for _ in range(5):
            u, t = m * z, y.clone()
            for dim in (-3, -2, -1):
                t.narrow(dim, 0, size - 1).add_(u.narrow(dim, 1, size - 1))
            z = t * m / d
        loc = z
    else:
        loc = _pcg(lambda v: laplace(v, m), loc, 1.0 / 6.0)
    out = torch.zeros_like(r)
    out.index_add_(0, idx.reshape(-1), (loc * m).reshape(-1))

    # ---- coarse: faces, edges and vertices on the lower planes of the boxes
    low = (g == start[box]) & (box > 0)
    code = low[:, None, None] * 4 + low[None, :, None] * 2 + low[None, None, :] * 1
    b3 = box[:, None, None] * boxes ** 2 + box[None, :, None] * boxes + box[None, None, :]
    comp = torch.where(code > 0, b3 * 8 + code, torch.zeros_like(b3))
    ncol = boxes ** 3 * 8
    count = torch.bincount(comp.reshape(-1), minlength=ncol).to(torch.float64)
    gamma = (code > 0).to(torch.float64)
    inner = 1.0 - gamma
    on_gamma = gamma / count[comp].sqrt()                      # Phi_Gamma's values
    ones = torch.ones_like(inner)
    parts = [(comp, on_gamma)]
    for dim, bit, stride in ((0, 4, boxes ** 2), (1, 2, boxes), (2, 1, 1)):
        for up in (False, True):
            # interior nodes next to the box's own lower face, or to the next box's
            f = (code == bit).to(torch.float64) * on_gamma
            rhs = torch.zeros_like(f)
            k = N - 1
            if up:
                rhs.narrow(dim, 0, k).add_(f.narrow(dim, 1, k))
            else:
                rhs.narrow(dim, 1, k).add_(f.narrow(dim, 0, k))
            rhs *= inner
            if float(rhs.abs().sum()) == 0.0:
                continue
            X = _pcg(lambda v: laplace(v, inner), rhs, 1.0 / 6.0)
            col = (b3 + (stride if up else 0)) * 8 + bit
            has = inner * (X != 0)
            parts.append((torch.where(has > 0, col, torch.zeros_like(col)), X * has))

    def phi(c):
        v = torch.zeros_like(inner)
        for col, X in parts:
            v += X * c[col]
        return v

    def phi_t(v):
        c = torch.zeros(ncol, dtype=torch.float64, device=dev)
        for col, X in parts:
            c.index_add_(0, col.reshape(-1), (X * v).reshape(-1))
        return c

    c = phi_t(r3)
    if float(c.abs().sum()) > 0.0:
        c = _pcg(lambda v: phi_t(laplace(phi(v), ones)), c, 1.0)
        out = out + phi(c).reshape(-1)
    return out
