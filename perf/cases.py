"""Performance cases: what a program does with this package, over the range of
sizes, precisions and right-hand-side counts in which it is used.

The matrices are compressed wavelet matrices on a 2^grid x 2^grid Haar basis:
functions of levels 0..grid-1 on their cells, an entry kept when the distance of
the two supports is at most a 2^-min(level), values that decay with the level
difference and the distance and carry random signs, and a diagonal that makes
the matrix strictly diagonally dominant.  `height` < 1 keeps the functions whose
support centre lies in [0, 1] x [0, height]: a domain whose number of unknowns is
no power of two.  The pattern (and with it the ordering, the plan and the
workspace, which a program keeps for all matrices of one pattern) depends on the
case alone; values and right-hand sides come from the seed.

Operations
  step    numeric factorization of new values, then the solve of nrhs right-hand
          sides: with an FP64 factor directly, with an FP32 factor refined to 1e-10
  solve   the solve alone with a factor that is kept
  half    L^T solve alone with a kept FP64 factor (a random field sample in precision form)
  grad    forward and backward of the differentiable solve with a kept FP32 factor,
          both refined, with the gradient on the stored pattern
  theta   time steps of the theta scheme over one kept FP64 factor
  lu      LU factorization of a nonsymmetric matrix and the solve of nrhs right-hand sides
  batch   many uneven instances factored together in FP32 and refined
  field   random field samples from kept FP64 factors of a covariance and a mass matrix
"""
import math
import random

import numpy as np
import torch

import paper_2007_01541_amd as wcs

DEV = torch.device("cuda" if torch.cuda.is_available() else "cpu")
F64 = torch.float64
PREC = {"fp64": wcs.FP64, "fp32": wcs.FP32}


def _case(name, op, grid, height=1.0, a=1.5, s=0.5, kind="exp", prec="fp64", nrhs=1, steps=0, count=0, pick=0):
    c = {"op": op, "grid": grid, "height": height, "a": a, "s": s, "kind": kind, "prec": prec, "nrhs": nrhs,
         "steps": steps, "count": count, "pick": pick}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest factorization and solve: an inner system of an outer iteration, where launches count
        _case("step_n1024_fp64", "step", 5),
        # one right-hand side after another against a small kept factor
        _case("solve_n4096_fp64", "solve", 6),
        # a small system in FP32 with refinement, few right-hand sides
        _case("step_n4096_fp32_4rhs", "step", 6, prec="fp32", nrhs=4),
        # a ragged domain and an odd number of right-hand sides
        _case("step_n11k_ragged_fp64_7rhs", "step", 7, height=0.7, a=1.7, nrhs=7),
        # the mid-size FP64 system
        _case("step_n65536_fp64", "step", 8),
        # the headline system, 64 right-hand sides, FP32 factor with refinement
        _case("step_n262144_fp32_64rhs", "step", 9, a=2.0, s=0.75, kind="alg", prec="fp32", nrhs=64),
        # ... and with the FP64 factor
        _case("step_n262144_fp64_64rhs", "step", 9, a=2.0, s=0.75, kind="alg", nrhs=64),
        # the gradient through the solve for a random field
        _case("grad_n65536_fp32", "grad", 8, a=2.0, s=0.75, kind="alg", prec="fp32"),
        # Crank-Nicolson steps of the parabolic problem
        _case("theta_n65536_fp64_10steps", "theta", 8, a=2.0, s=0.375, kind="alg", steps=10),
        # the nonsymmetric system of the polarizable continuum model
        _case("lu_n65536_8rhs", "lu", 8, nrhs=8),
        # many small uneven instances at once
        _case("batch32_fp32_4rhs", "batch", 0, prec="fp32", nrhs=4, count=32, pick=4000),
        # samples of a random field in covariance form
        _case("field_n65536_fp64_64", "field", 8, a=2.0, nrhs=64),
    ]


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "solve", "solve", "half", "grad", "theta", "lu", "batch", "field"])
    nrhs = max(1, round(math.exp(rng.uniform(0.0, math.log(70.0)))))
    if op == "batch":
        return _case("", op, 0, prec="fp32", nrhs=min(nrhs, 16), count=rng.randint(2, 32), pick=rng.randint(1, 10 ** 6))
    grid = rng.choice([5, 6, 7, 8, 8])
    height = rng.choice([1.0, round(rng.uniform(0.35, 0.95), 3)])
    a = round(rng.uniform(1.2, 2.0), 2)
    s = rng.choice([0.25, 0.375, 0.5, 0.75])
    kind = rng.choice(["exp", "alg"])
    if op == "step" and rng.random() < 0.15:
        grid, height, nrhs = 9, round(rng.uniform(0.35, 0.95), 3), min(nrhs, 64)
    if op in ("half", "grad", "theta"):
        nrhs = 1
    prec = {"step": rng.choice(["fp32", "fp64"]), "grad": "fp32"}.get(op, "fp64")
    return _case("", op, grid, height, a, s, kind, prec, nrhs, steps=rng.randint(2, 20) if op == "theta" else 0)


# ------------------------------------------------------------------ patterns

def _pairs_1d(j, jp, grid, a):
    """Coarse cell, fine cell and distance (in units of 2^-grid) of the 1-D cell pairs of two levels in reach."""
    r, big, small = 1 << (jp - j), 1 << (grid - j), 1 << (grid - jp)
    w = int(math.floor(a * big / small))
    o = torch.arange(-1 - w, r + w + 1, device=DEV)
    gap = torch.where(o >= r, o * small - big, torch.where(o < 0, -(o + 1) * small, torch.zeros_like(o)))
    k = torch.arange(1 << j, device=DEV).repeat_interleave(o.numel())
    m = k * r + o.repeat(1 << j)
    ok = (m >= 0) & (m < (1 << jp))
    return k[ok], m[ok], gap.repeat(1 << j)[ok]


def _functions(j, cell):
    """The functions on each cell of a level, one column each (the scaling function with the first wavelets)."""
    if j == 0:
        return cell[:, None] * 0 + torch.arange(4, device=DEV)[None, :]
    return 4 ** j + 3 * cell[:, None] + torch.arange(3, device=DEV)[None, :]


class Pattern:
    """Lower pattern of one case on the GPU, its decay factors, and the analysis."""

    def __init__(self, grid, height, a):
        n0 = 4 ** grid
        level = torch.zeros(n0, dtype=torch.int64, device=DEV)
        centre = torch.full((n0, 2), 0.5, dtype=F64, device=DEV)
        for j in range(grid):
            cell = torch.arange(4 ** j, device=DEV)
            f = _functions(j, cell)
            level[f] = j
            centre[f] = (torch.stack([cell % (1 << j), cell // (1 << j)], 1).to(F64) + 0.5)[:, None, :] * 2.0 ** -j
        kept = centre[:, 1] < height if height < 1.0 else torch.ones(n0, dtype=torch.bool, device=DEV)
        number = torch.cumsum(kept, 0) - 1
        n = int(kept.sum())
        rows, cols, dist = [], [], []
        for j in range(grid):
            for jp in range(j, grid):
                k, m, g = _pairs_1d(j, jp, grid, a)
                reach = (a * (1 << (grid - j))) ** 2
                big, small = 1 << (grid - j), 1 << (grid - jp)
                step = max(1, (1 << 24) // k.numel())
                for x0 in range(0, k.numel(), step):
                    gx = g[x0:x0 + step]
                    p, q = torch.nonzero((gx * gx)[:, None] + (g * g)[None, :] <= reach, as_tuple=True)
                    p = p + x0
                    dx = (2 * m[p] + 1) * small - (2 * k[p] + 1) * big
                    dy = (2 * m[q] + 1) * small - (2 * k[q] + 1) * big
                    d = torch.sqrt((dx * dx + dy * dy).to(F64)) * (0.5 * 2.0 ** -grid)
                    coarse = _functions(j, k[q] * (1 << j) + k[p])
                    fine = _functions(jp, m[q] * (1 << jp) + m[p])
                    for c in range(coarse.shape[1]):
                        for f in range(fine.shape[1]):
                            lo, hi = coarse[:, c], fine[:, f]
                            ok = (hi > lo) & kept[lo] & kept[hi]
                            rows.append(number[hi[ok]])
                            cols.append(number[lo[ok]])
                            dist.append(d[ok])
        diag = torch.arange(n, device=DEV)
        row = torch.cat(rows + [diag])
        col = torch.cat(cols + [diag])
        del rows, cols
        key, order = torch.sort(col * n + row)
        del row, col
        self.n = n
        self.col = key // n
        self.row = key - self.col * n
        del key
        self.dist = torch.cat(dist + [torch.zeros(n, dtype=F64, device=DEV)])[order]
        del dist, order
        self.level = level[kept]
        self.nnz = self.row.numel()
        counts = torch.bincount(self.col, minlength=n)
        self.colptr = torch.cat([counts.new_zeros(1), torch.cumsum(counts, 0)])
        self.diag = self.colptr[:-1]
        self.sym = wcs.Symbolic(n, self.colptr.cpu().numpy(), self.row.to(torch.int32).cpu().numpy(),
                                coords=centre[kept].cpu().numpy())

    def decay(self, kind, s, ell):
        dj = (self.level[self.row] - self.level[self.col]).abs().to(F64)
        if kind == "exp":
            return torch.exp2(-1.5 * dj) * torch.exp(-self.dist / ell)
        grid = int(self.level.max()) + 1
        return torch.exp2(-(1.0 + s) * dj) * (1.0 + self.dist * 2.0 ** grid) ** -(2.0 + 2.0 * s)


_patterns, _factors, _batches = {}, {}, {}


def _pattern(grid, height, a):
    key = (grid, height, a)
    if key not in _patterns:
        _patterns[key] = Pattern(*key)
    return _patterns[key]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _sums(n, *terms):
    """Sums of |v| by index, in whole numbers so that every run adds them up alike."""
    t = torch.zeros(n, dtype=torch.int64, device=DEV)
    for i, v in terms:
        t.index_add_(0, i, (v.abs() * 2.0 ** 40).to(torch.int64))
    return t.to(F64) * 2.0 ** -40


def _values(P, kind, s, gen, ell=0.3):
    v = P.decay(kind, s, ell) * (2.0 * torch.rand(P.nnz, generator=gen, device=DEV, dtype=F64) - 1.0)
    v[P.diag] = 0.0
    v[P.diag] = 1.1 * _sums(P.n, (P.row, v), (P.col, v)) + torch.exp2(2.0 * s * P.level.to(F64))
    return v


def _values_lu(P, kind, s, gen):
    v = P.decay(kind, s, 0.3) * (2.0 * torch.rand(P.nnz, generator=gen, device=DEV, dtype=F64) - 1.0)
    v[P.diag] = 0.0
    lo, up = (v * (1.0 + torch.rand(P.nnz, generator=gen, device=DEV, dtype=F64) - 0.5) for _ in range(2))
    by_row = _sums(P.n, (P.row, lo), (P.col, up))
    by_col = _sums(P.n, (P.col, lo), (P.row, up))
    d = 1.1 * torch.maximum(by_row, by_col) + torch.exp2(2.0 * s * P.level.to(F64))
    lo[P.diag] = d
    up[P.diag] = d
    return lo, up


def _rhs(n, k, gen):
    b = torch.randn(n, k, generator=gen, device=DEV, dtype=F64)
    return b[:, 0].contiguous() if k == 1 else b


def _plan(key, make):
    """The factor object (plan and workspace) that a program keeps for one pattern."""
    if key not in _factors:
        _factors[key] = make()
    return _factors[key]


class Batch:
    def __init__(self, count, pick):
        r = random.Random(pick)
        self.spec = []
        for _ in range(count):
            grid = r.randint(5, 7)
            self.spec.append((Pattern(grid, 1.0, round(r.uniform(1.2, 2.0), 3)), r.choice([0.25, 0.5, 0.75]),
                              r.uniform(0.1, 0.5)))
        self.sym = wcs.Symbolic.batch([p.sym for p, _, _ in self.spec])
        self.n = self.sym.n


def _batch(case):
    key = (case["count"], case["pick"])
    if key not in _batches:
        _batches[key] = Batch(*key)
    return _batches[key]


def _inputs(case, seed):
    """The numbers of a case, from the seed alone."""
    g = _gen(seed)
    op, k = case["op"], case["nrhs"]
    if op == "batch":
        B = _batch(case)
        return {"values": torch.cat([_values(p, "exp", s, g, ell) for p, s, ell in B.spec]), "b": _rhs(B.n, k, g)}
    P = _pattern(case["grid"], case["height"], case["a"])
    if op == "lu":
        lo, up = _values_lu(P, case["kind"], case["s"], g)
        return {"values": lo, "upper": up, "b": _rhs(P.n, k, g)}
    v = _values(P, case["kind"], case["s"], g)
    if op == "theta":
        return {"values": v, "f": torch.randn(P.n, case["steps"] + 1, generator=g, device=DEV, dtype=F64),
                "u0": _rhs(P.n, 1, g)}
    if op == "grad":
        return {"values": v, "b": _rhs(P.n, 1, g), "gy": _rhs(P.n, 1, g)}
    if op == "field":
        M = _pattern(case["grid"], case["height"], 0.0)
        return {"values": v, "mass": _values(M, "exp", 0.0, g), "b": _rhs(P.n, k, g), "abar": _rhs(P.n, 1, g)}
    return {"values": v, "b": _rhs(P.n, k, g)}


THETA, DT = 0.5, 0.02


def prepare(case, seed):
    st = dict(_inputs(case, seed), op=case["op"], prec=case["prec"])
    op, k = case["op"], case["nrhs"]
    key = tuple(sorted((n, v) for n, v in case.items() if n != "name"))
    if op == "batch":
        B = _batch(case)

        def make():
            f = wcs.Factor(B.sym, wcs.FP32, max_nrhs=k)
            f.autotune(st["values"])
            return f
        st["factor"] = _plan(key, make)
        return st
    P = _pattern(case["grid"], case["height"], case["a"])
    if op == "step":
        def make():
            f = wcs.Factor(P.sym, PREC[case["prec"]], max_nrhs=k)
            if P.n >= 1 << 18:
                f.autotune(st["values"])      # as the benchmark of the large system does
            return f
        st["factor"] = _plan(key, make)
    elif op == "lu":
        st["factor"] = _plan(key, lambda: wcs.Factor(P.sym, wcs.LU64, max_nrhs=k))
    elif op == "field":
        M = _pattern(case["grid"], case["height"], 0.0)
        st["factor"] = wcs.Factor(P.sym, wcs.FP64, max_nrhs=k)
        st["factor"].numeric(st["values"])
        st["massf"] = wcs.Factor(M.sym, wcs.FP64, max_nrhs=k)
        st["massf"].numeric(st["mass"])
    else:
        f = st["factor"] = wcs.Factor(P.sym, PREC[case["prec"]], max_nrhs=k)
        if op == "theta":
            st["A"] = f.theta_matrix(st["values"], THETA, DT)
            f.numeric(st["A"])
        else:
            f.numeric(st["values"])
        if op == "grad":
            st["values"].requires_grad_(True)
            st["b"].requires_grad_(True)
    return st


def run(st):
    op, f = st["op"], st["factor"]
    if op in ("step", "batch"):
        f.numeric(st["values"])
        if st["prec"] == "fp32":
            return f.solve_refined(st["b"], st["values"], tol=1e-10)[0]
        return f.solve(st["b"])
    if op == "solve":
        return f.solve(st["b"])
    if op == "half":
        return f.solve(st["b"], wcs.SOLVE_LT)
    if op == "grad":
        y = wcs.cholesky_solve(st["values"], st["b"], f, refine=True)
        gv, gb = torch.autograd.grad(y, (st["values"], st["b"]), st["gy"])
        return y.detach(), gv, gb
    if op == "theta":
        return f.theta_steps(st["A"], THETA, DT, st["f"], st["u0"])[0]
    if op == "lu":
        f.numeric_lu(st["values"], st["upper"])
        return f.solve(st["b"])
    return wcs.field_sample(f, st["massf"], st["b"], abar=st["abar"])


def work(case):
    """Values read once, the factor written once and read once by each half of a solve, right-hand sides read and
    written once; an FP32 step needs two solves and one product with the matrix to reach its tolerance."""
    op, k = case["op"], case["nrhs"]
    P = _batch(case) if op == "batch" else _pattern(case["grid"], case["height"], case["a"])
    i = P.sym.info
    n, nz, nl, fl = i["n"], i["nnz_lower"], i["nnz_l"], i["flops"]
    e = 4 if case["prec"] == "fp32" else 8
    solve = (2 * e * nl, 4.0 * nl * k)
    product = (8 * nz, 4.0 * nz * k)
    rhs = 16 * n * k
    if op in ("step", "batch"):
        refined = case["prec"] == "fp32"
        s, p = (2, 1) if refined else (1, 0)
        return {"bytes": 8 * nz + e * nl + s * solve[0] + p * product[0] + rhs,
                "flops": fl + s * solve[1] + p * product[1]}
    if op == "solve":
        return {"bytes": solve[0] + rhs, "flops": solve[1]}
    if op == "half":
        return {"bytes": solve[0] / 2 + rhs, "flops": solve[1] / 2}
    if op == "grad":
        return {"bytes": 4 * solve[0] + 2 * product[0] + 8 * nz + 6 * 8 * n, "flops": 4 * solve[1] + 2 * product[1] + 4.0 * nz}
    if op == "theta":
        t = case["steps"]
        return {"bytes": t * (solve[0] + product[0] + rhs), "flops": t * (solve[1] + product[1])}
    if op == "lu":
        return {"bytes": 16 * nz + 2 * 8 * nl + solve[0] + rhs, "flops": 2.0 * fl + solve[1]}
    m = _pattern(case["grid"], case["height"], 0.0).sym.info
    return {"bytes": 8 * nl + 16 * m["nnz_l"] + rhs + 8 * n, "flops": 2.0 * nl * k + 4.0 * m["nnz_l"] * k}


# ------------------------------------------------------------------ 64-bit values

def _full(P, lo, up):
    """The whole matrix as CSR from its two triangles (up holds the entry mirrored from each stored one)."""
    off = P.row != P.col
    r = torch.cat([P.row, P.col[off]])
    key, order = torch.sort(r * P.n + torch.cat([P.col, P.row[off]]))
    v = torch.cat([lo, up[off]])[order]
    r = key // P.n
    ptr = torch.cat([r.new_zeros(1), torch.cumsum(torch.bincount(r, minlength=P.n), 0)])
    return torch.sparse_csr_tensor(ptr.to(torch.int32), (key - r * P.n).to(torch.int32), v, size=(P.n, P.n))


def _cg(A, d, B):
    """Conjugate gradients preconditioned by the diagonal, started again from the true residual until it stops falling."""
    B = B if B.dim() == 2 else B[:, None]
    X = torch.zeros_like(B)
    last = None
    for _ in range(4):
        R = B - A @ X
        size = float((R.norm(dim=0) / B.norm(dim=0)).max())
        if size < 3e-16 or (last is not None and size > 0.5 * last):
            break
        last = size
        D = torch.zeros_like(B)
        Z = R / d
        p, rz = Z.clone(), (R * Z).sum(0)
        first = R.norm(dim=0)
        for _ in range(200):
            q = A @ p
            al = rz / (p * q).sum(0)
            D += al * p
            R = R - al * q
            if float((R.norm(dim=0) / first).max()) < 1e-13:
                break
            Z = R / d
            new = (R * Z).sum(0)
            p = Z + (new / rz) * p
            rz = new
        X = X + D
    return X


def exact(case, seed):
    op = case["op"]
    if op in ("half", "field"):      # white noise is read in the pivot order, which only the analysis knows
        return None
    x = _inputs(case, seed)
    shape = lambda t: t[:, 0] if case["nrhs"] == 1 else t  # noqa: E731
    if op == "batch":
        B, out, i, z = _batch(case), [], 0, 0
        for p, _, _ in B.spec:
            v = x["values"][z:z + p.nnz]
            b = x["b"][i:i + p.n]
            out.append(_cg(_full(p, v, v), v[p.diag][:, None], b))
            i, z = i + p.n, z + p.nnz
        return shape(torch.cat(out))
    P = _pattern(case["grid"], case["height"], case["a"])
    v = x["values"]
    d = v[P.diag][:, None]
    if op == "lu":
        A = _full(P, v, x["upper"])
        b = x["b"] if x["b"].dim() == 2 else x["b"][:, None]
        y = b / d
        for _ in range(400):
            r = b - A @ y
            y = y + r / d
            if float((r.norm(dim=0) / b.norm(dim=0)).max()) < 3e-16:
                break
        return shape(y)
    if op == "theta":
        lhs = v * (THETA * DT)
        lhs[P.diag] += 1.0
        rhs = v * (-(1.0 - THETA) * DT)
        rhs[P.diag] += 1.0
        A, E = _full(P, lhs, lhs), _full(P, rhs, rhs)
        U = [x["u0"][:, None]]
        for i in range(case["steps"]):
            b = E @ U[-1] + DT * ((1.0 - THETA) * x["f"][:, i:i + 1] + THETA * x["f"][:, i + 1:i + 2])
            U.append(_cg(A, lhs[P.diag][:, None], b))
        return torch.cat(U, 1)
    A = _full(P, v, v)
    if op == "grad":
        y, lam = _cg(A, d, torch.stack([x["b"], x["gy"]], 1)).unbind(1)
        g = -(lam[P.row] * y[P.col] + lam[P.col] * y[P.row])
        g[P.diag] = -lam * y
        return y, g, lam
    return shape(_cg(A, d, x["b"]))
