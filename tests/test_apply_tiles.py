"""The product P^T L B through every tile form (N = 16,384: fronts with fewer
than 128, up to 1,024 and more pivot columns; separator rows held by hundreds of
fronts), against the oracle's product with the exported factor, within the
rounding bound of a sum of at most n terms.  Column counts: one, a ragged one
(no vector form), a multiple of four past a 16-column strip, and past 64.
"""
import numpy as np
import pytest

import oracle
from workloads import normal_rhs, tiny
from tests.helpers import EPS32, EPS64
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd import APPLY_L, FP32, FP64, Factor, Symbolic  # noqa: E402


@pytest.mark.parametrize("prec", [FP64, FP32])
def test_product_tiles(prec):
    m = tiny(7, 1.5).matrix()
    n = m["n"]
    sym = Symbolic(n, m["colptr"], m["rowind"], coords=m["coords"])
    ex = sym.export()
    p = np.diff(ex["relaxed_ptr"])
    print(f"n={n} prec={prec} largest front {p.max()} pivots", flush=True)
    assert p.max() > 1024 and ((p > 128) & (p < 1024)).any() and p.min() < 64
    f = Factor(sym, prec, max_nrhs=68)
    f.numeric(dev(m["values"]))
    Lp, Li, Lx = f.export_L()
    eps = EPS64 if prec == FP64 else EPS32
    for k in (1, 7, 20, 68):
        B = normal_rhs(n, k, 23 + k)
        X = f.apply(dev(B), APPLY_L).cpu().numpy()
        ref = oracle.apply(ex["perm"], Lp, Li, Lx, B, APPLY_L)
        bound = (n + 2) * eps * oracle.apply(ex["perm"], Lp, Li, np.abs(Lx), np.abs(B), APPLY_L)
        assert np.all(np.abs(X - ref) <= bound), k


def test_product_of_more_strips_than_one_launch_takes():
    """A dense front of 1,100 pivots and 1,041 right-hand sides: 66 strips of 16
    columns, more than the 64 of a launch (whose grid is bounded in y), the last
    of one column; bitwise the product of the columns taken a few at a time."""
    n, k = 1100, 1041
    rng = np.random.default_rng(7)
    G = rng.uniform(-1.0, 1.0, (n, n))
    G[np.diag_indices(n)] = n
    colptr = np.concatenate([[0], np.cumsum(n - np.arange(n))]).astype(np.int64)
    rowind = np.concatenate([np.arange(c, n) for c in range(n)]).astype(np.int32)
    f = Factor(Symbolic(n, colptr, rowind, leaf_size=n, dense_degree_min=4 * n), FP64, max_nrhs=k)
    f.numeric(dev(np.concatenate([G[c:, c] for c in range(n)])))
    B = dev(normal_rhs(n, k, 97))
    X = f.apply(B, APPLY_L)
    for c in (0, 1008, 1024, 1040):
        print(f"columns from {c}", flush=True)
        assert torch.equal(f.apply(B[:, c:c + 17], APPLY_L), X[:, c:c + 17]), c
