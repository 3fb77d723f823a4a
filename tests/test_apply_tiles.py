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
