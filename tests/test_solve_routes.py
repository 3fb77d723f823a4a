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
