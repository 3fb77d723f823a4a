"""Persistent triangular sweeps (at most 8 right-hand sides) against the oracle.

The cases hold narrow fronts (one pivot block) with more and fewer than 256
update rows, wide ones with ragged pivot blocks and super-blocks, and roots;
the column counts are the edges of the kernel's three widths.  A batch of two
copies gives a forest.  Right-hand sides with NaN (one of them the all-ones
pattern that marks an empty exchange element) come back as NaN.
"""
import numpy as np
import pytest

import oracle
from workloads import normal_rhs
from tests.helpers import EPS32, EPS64, factor_tol
from tests.test_gpu_parity import CASES, dev, prepared

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd.capi import WcsError  # noqa: E402
from paper_2007_01541_amd import FP32, FP64, SOLVE_FULL, SOLVE_L, SOLVE_LT, Factor, Symbolic  # noqa: E402


@pytest.mark.parametrize("kind,leaf,coords", CASES)
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_sweeps_match_oracle(kind, leaf, coords, prec):
    m, sym, orc = prepared(kind, leaf, coords)
    n = m["n"]
    p = np.diff(sym.export()["relaxed_ptr"])
    print(f"case {kind} prec={prec} n={n} fronts {p.size} largest {p.max()}", flush=True)
    f = Factor(sym, prec, max_nrhs=8)
    f.numeric(dev(m["values"]))
    B = normal_rhs(n, 8, 91)
    tol = factor_tol(m, int(orc.colcount.max()), EPS64 if prec == FP64 else EPS32)
    for part in (SOLVE_FULL, SOLVE_L, SOLVE_LT):
        Xo = orc.solve(B, part)
        for k in (1, 2, 4, 5, 8):
            b = dev(B[:, :k])
            X = f.solve(b, part)
            assert np.abs(X.cpu().numpy() - Xo[:, :k]).max() <= tol * np.abs(Xo).max(), (part, k)
            for _ in range(3):
                assert torch.equal(f.solve(b, part), X), (part, k)


def test_sweeps_of_a_forest():
    m, sym, orc = prepared("g6alg", 32, True)
    n = m["n"]
    both = Symbolic.batch([sym, sym])
    f = Factor(both, FP64, max_nrhs=3)
    v = dev(m["values"])
    f.numeric(torch.cat([v, 2.0 * v]))
    B = normal_rhs(2 * n, 3, 92)
    X = f.solve(dev(B)).cpu().numpy()
    tol = factor_tol(m, int(orc.colcount.max()), EPS64)
    for b, scale in ((0, 1.0), (1, 0.5)):
        Xo = scale * orc.solve(B[b * n:(b + 1) * n])
        assert np.abs(X[b * n:(b + 1) * n] - Xo).max() <= tol * np.abs(Xo).max()


@pytest.mark.parametrize("bits", [0x7FF8000000000000, 0xFFFFFFFFFFFFFFFF])
def test_sweeps_pass_nan_on(bits):
    m, sym, _ = prepared("small")
    f = Factor(sym, FP64, max_nrhs=2)
    f.numeric(dev(m["values"]))
    B = normal_rhs(m["n"], 2, 93)
    B[:, 1] = np.full(m["n"], bits, np.uint64).view(np.float64)
    X = f.solve(dev(B)).cpu().numpy()
    assert np.isfinite(X[:, 0]).all() and np.isnan(X[:, 1]).all()


@pytest.mark.parametrize("n", [64, 200, 300])
def test_forward_sweep_rounds_the_diagonal_term_once(n):
    """FP32 L^-1 P B with dense fronts of n pivots (a narrow one, one ragged
    super-block, two) whose off-diagonal entries are about 1e-6 of the diagonal:
    with u = eps / 2, z_r = X_rr w_r (1 + d) with |d| <= u for X_rr, u for the
    product and sum and u for w_r - (rows past the first super-block); the
    n 1e-6 of the other terms adds less than 0.1 u, their roundings at most
    n 1e-6 (n + 10) u < 0.1 u.  B is exact in FP32; the reference uses the exported L."""
    rng = np.random.default_rng(n)
    G = rng.uniform(-1e-6, 1e-6, (n, n))
    G[np.diag_indices(n)] = rng.uniform(1.0, 2.0, n)
    colptr = np.concatenate([[0], np.cumsum(n - np.arange(n))]).astype(np.int64)
    rowind = np.concatenate([np.arange(c, n) for c in range(n)]).astype(np.int32)
    sym = Symbolic(n, colptr, rowind, leaf_size=n, dense_degree_min=4 * n)
    f = Factor(sym, FP32, max_nrhs=8)
    f.numeric(dev(np.concatenate([G[c:, c] for c in range(n)])))
    ex = sym.export()
    assert ex["relaxed_ptr"].size == 2, "one front"
    Lp, Li, Lx = f.export_L()
    L = np.zeros((n, n), np.longdouble)
    for c in range(n):
        L[Li[Lp[c]:Lp[c + 1]], c] = Lx[Lp[c]:Lp[c + 1]]
    B = (rng.uniform(1.0, 2.0, (n, 8)) * rng.choice([-1.0, 1.0], (n, 8))).astype(np.float32).astype(np.float64)
    Z = np.zeros((n, 8), np.longdouble)
    for r in range(n):
        Z[r] = (B[ex["perm"][r]] - L[r, :r] @ Z[:r]) / L[r, r]
    u = EPS32 / 2
    bound = np.where(np.arange(n) < 256, 2.2, 3.2)[:, None] * u * np.abs(Z)
    for k in (1, 4, 8):
        X = f.solve(dev(B[:, :k]), SOLVE_L).cpu().numpy()
        err = np.abs(X - Z[:, :k])
        print(f"n={n} k={k} largest error {float((err / np.abs(Z[:, :k])).max() / u):.2f} u", flush=True)
        assert np.all(err <= bound[:, :k]), k


def test_a_sweep_that_gives_up_is_reported(monkeypatch):
    """With one poll per wait every sweep gives up (and every workgroup still
    ends): the solution holds NaN, the next status read reports it, once, and a
    solve afterwards is the one before."""
    m, sym, _ = prepared("small")
    v = dev(m["values"])
    b = dev(normal_rhs(m["n"], 8, 94))
    for prec in (FP64, FP32):
        f = Factor(sym, prec, max_nrhs=8)
        f.numeric(v)
        for k in (1, 4, 8):
            X = f.solve(b[:, :k])
            assert torch.isfinite(X).all()
            monkeypatch.setenv("WCS_SWEEP_POLLS", "1")
            print(f"prec={prec} k={k}", flush=True)
            assert torch.isnan(f.solve(b[:, :k])).any()
            with pytest.raises(WcsError) as e:
                f.pivot_check()
            assert e.value.code == -3 and "gave up" in str(e.value)
            assert f.pivot_check() == -1
            f.solve(b[:, :k])
            with pytest.raises(WcsError):
                f.numeric(v)
            with pytest.raises(WcsError) as e:
                f.solve_refined(b[:, :k], v)
            assert e.value.code == -3
            monkeypatch.delenv("WCS_SWEEP_POLLS")
            f.numeric(v)
            assert torch.equal(f.solve(b[:, :k]), X)
