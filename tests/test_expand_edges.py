"""The expansion of the stored triangle into full rows at the edges of its
chunks (2048 entries, an eighth of the chunks per XCD): tridiagonal matrices of
whole numbers, so every product A x is exact.
"""
import numpy as np
import pytest

from workloads import normal_rhs
from tests.test_gpu_parity import dev, prepared

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd import FP32, FP64, Factor, Symbolic  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 683, 684, 5462, 5463, 6000, 60000])    # 3 n - 2 entries; 5462: eight whole chunks
def test_expanded_values(n):
    colptr = np.concatenate([2 * np.arange(n), [2 * n - 1]]).astype(np.int64)
    rowind = np.stack([np.arange(n), np.arange(n) + 1], 1).ravel()[:-1].astype(np.int32)
    rng = np.random.default_rng(n)
    values = rng.integers(1, 1000, 2 * n - 1).astype(np.float64)
    f = Factor(Symbolic(n, colptr, rowind), FP64, max_nrhs=1)
    x = rng.integers(-1000, 1000, n).astype(np.float64)
    print(f"n={n}", flush=True)
    y = f.spmv(dev(x), dev(values)).cpu().numpy().ravel()
    d, e = values[0::2], values[1::2]
    ref = d * x
    ref[:-1] += e * x[1:]
    ref[1:] += e * x[:-1]
    assert np.array_equal(y, ref)


def test_expansion_grids(monkeypatch):
    """The expansion beside the first solve of a refinement on grids below, at
    and past one workgroup per XCD and with more chunks than workgroups: one
    workgroup with all chunks, a range each for two and seven, whole multiples
    of eight; bitwise the same refined solution and report."""
    m, sym, _ = prepared("small")
    assert (2 * len(m["rowind"]) - m["n"]) > 256 * 2048
    f = Factor(sym, FP32, max_nrhs=8)
    v = dev(m["values"])
    f.numeric(v)
    b = dev(normal_rhs(m["n"], 8, 98))
    ref = None
    for blocks in ("1", "2", "7", "8", "9", "256", "65536"):
        monkeypatch.setenv("WCS_EXPAND_BLOCKS", blocks)
        print(f"expansion blocks {blocks}", flush=True)
        f.spmv(b, 2.0 * v)                     # other values in between
        X, rep = f.solve_refined(b, v, tol=1e-10)
        if ref is None:
            ref = X, rep
        assert torch.equal(X, ref[0]) and rep == ref[1], blocks
