"""Which kernels a solve of few right-hand sides takes: the switches that choose
the level-by-level kernels, and those kernels at the column counts that only
such a switch sends there.
"""
import numpy as np
import pytest

from workloads import normal_rhs
from tests.helpers import EPS32, EPS64, factor_tol
from tests.test_gpu_parity import CASES, dev, prepared

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd import FP32, FP64, SOLVE_FULL, SOLVE_L, SOLVE_LT, Factor  # noqa: E402


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_sixteen_column_switch_counts_from_five(prec, monkeypatch):
    """WCS_SOLVE_KT16_MAX=16: 5..16 right-hand sides take the 16-column kernels,
    where a column's result does not depend on its neighbours, so every count
    gives the columns of sixteen bit for bit; 1..4 stay where they are."""
    m, sym, _ = prepared("small")
    b = dev(normal_rhs(m["n"], 16, 95))
    f = Factor(sym, prec, max_nrhs=16)
    f.numeric(dev(m["values"]))
    default = {k: f.solve(b[:, :k]) for k in (1, 4, 5, 8)}
    monkeypatch.setenv("WCS_SOLVE_KT16_MAX", "16")
    X = f.solve(b)
    for k in (5, 8, 9, 13):
        print(f"prec={prec} k={k}", flush=True)
        assert torch.equal(f.solve(b[:, :k]), X[:, :k]), k
    for k in (1, 4):
        assert torch.equal(f.solve(b[:, :k]), default[k]), k
    monkeypatch.setenv("WCS_SOLVE_KT16_MAX", "4")
    for k in (5, 8):
        assert torch.equal(f.solve(b[:, :k]), default[k]), k


@pytest.mark.parametrize("kind,leaf,coords", CASES)
@pytest.mark.parametrize("rows", ["100000", "64"])
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_fused_fronts_of_few_columns(kind, leaf, coords, rows, prec, monkeypatch):
    """WCS_SOLVE_STEP_ROWS takes the whole factor off the persistent sweep: the
    four-column level kernels, all fronts fused or the small ones beside
    super-block fronts, at the column counts below their width."""
    monkeypatch.setenv("WCS_SOLVE_STEP_ROWS", rows)
    m, sym, orc = prepared(kind, leaf, coords)
    B = normal_rhs(m["n"], 4, 99)
    f = Factor(sym, prec, max_nrhs=4)
    f.numeric(dev(m["values"]))
    tol = factor_tol(m, int(orc.colcount.max()), EPS64 if prec == FP64 else EPS32)
    for part in (SOLVE_FULL, SOLVE_L, SOLVE_LT):
        Xo = orc.solve(B, part)
        for k in (2, 3, 4):
            print(f"case {kind} rows={rows} prec={prec} part={part} k={k}", flush=True)
            X = f.solve(dev(B[:, :k]), part).cpu().numpy()
            assert np.abs(X - Xo[:, :k]).max() <= tol * np.abs(Xo).max(), (part, k)


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_super_block_levels_of_few_columns(prec):
    """The level kernels without fused fronts at the counts that the persistent
    sweep takes by default: fronts of up to 316 pivots in the static workspace,
    with so large a max_nrhs that the sweep's tables alone do not fit."""
    m, sym, orc = prepared(*next(c for c in CASES if c[0] == "g5a13"))
    limit = 64 << 20
    lo, hi = 8, 4096
    while lo + 1 < hi:                       # workspace_size(lo) <= limit < workspace_size(hi)
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if sym.workspace_size(prec, mid) > limit else (mid, hi)
    f = Factor(sym, prec, max_nrhs=hi, static_workspace=True)
    f.numeric(dev(m["values"]))
    B = normal_rhs(m["n"], 8, 100)
    tol = factor_tol(m, int(orc.colcount.max()), EPS64 if prec == FP64 else EPS32)
    for part in (SOLVE_FULL, SOLVE_L, SOLVE_LT):
        Xo = orc.solve(B, part)
        for k in (1, 2, 3, 4, 5, 8):
            print(f"max_nrhs={hi} prec={prec} part={part} k={k}", flush=True)
            X = f.solve(dev(B[:, :k]), part).cpu().numpy()
            assert np.abs(X - Xo[:, :k]).max() <= tol * np.abs(Xo).max(), (part, k)


@pytest.mark.parametrize("kind", ["small", "g6alg", "g5a13"])
@pytest.mark.parametrize("prec", [FP64, FP32])
def test_solve_levels_bitwise(kind, prec, monkeypatch):
    """The solves' levels of their own (by default those with the shorter chain)
    against the thresholds 256, 1024 and none for both: the same factor and the
    same solutions bit for bit, level by level and persistent, whole and half."""
    m, sym, _ = prepared(*next(c for c in CASES if c[0] == kind))
    v = dev(m["values"])
    b = dev(normal_rhs(m["n"], 64, 101))
    ref = None
    for late in (None, "256", "1024", "0"):
        if late is not None:
            monkeypatch.setenv("WCS_LATE_MIN_PIVOTS", late)
        f = Factor(sym, prec, max_nrhs=64)
        f.numeric(v)
        print(f"{kind} prec={prec} late={late}", flush=True)
        out = [f.solve(b[:, :k], part) for part in (SOLVE_FULL, SOLVE_L, SOLVE_LT) for k in (1, 8, 12, 64)]
        if ref is None:
            ref = f.export_L()[2], out
        assert np.array_equal(f.export_L()[2], ref[0])
        assert all(torch.equal(x, y) for x, y in zip(out, ref[1]))
