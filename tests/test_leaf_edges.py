"""The leaf kernel at the edges of its tiles: dense blocks of p pivots under a
common dense border of s rows (whole and partial 16-column blocks, 64-row
slabs, one row, no rows), against a double-precision factorization on the host
within the backward-error bound of Cholesky.
"""
import numpy as np
import pytest

from tests.helpers import EPS32, EPS64
from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd import FP32, FP64, Factor, Symbolic  # noqa: E402


def bordered(p, s, blocks, seed):
    """Dense SPD matrix, zero between the blocks; the lower triangle by columns."""
    n = p * blocks + s
    rng = np.random.default_rng(seed)
    G = rng.uniform(-1.0, 1.0, (n, n))
    G = (G + G.T) / 2
    for b in range(blocks):
        lo, hi = b * p, (b + 1) * p
        G[lo:hi, :lo] = 0
        G[lo:hi, hi:blocks * p] = 0
    G[np.diag_indices(n)] = n
    keep = np.tril(G != 0)
    colptr = np.concatenate([[0], np.cumsum(keep.sum(0))]).astype(np.int64)
    rowind = np.concatenate([np.flatnonzero(keep[:, c]) for c in range(n)]).astype(np.int32)
    return G, colptr, rowind, np.concatenate([G[keep[:, c], c] for c in range(n)])


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("p,s", [(1, 0), (1, 3), (15, 1), (16, 48), (17, 63), (63, 65), (64, 0), (64, 130)])
def test_leaf_tiles(p, s, prec):
    G, colptr, rowind, values = bordered(p, s, 3 if s else 1, 11 * p + s)
    n = G.shape[0]
    sym = Symbolic(n, colptr, rowind, leaf_size=64, dense_degree_min=p + s if s else 4096)
    ex = sym.export()
    print(f"p={p} s={s} prec={prec} fronts {np.diff(ex['relaxed_ptr'])}", flush=True)
    f = Factor(sym, prec, max_nrhs=1)
    f.numeric(dev(values))
    Lp, Li, Lx = f.export_L()
    L = np.zeros((n, n))
    for c in range(n):
        L[Li[Lp[c]:Lp[c + 1]], c] = Lx[Lp[c]:Lp[c + 1]]
    P = G[np.ix_(ex["perm"], ex["perm"])]
    if prec == FP32:
        P = P.astype(np.float32).astype(np.float64)     # the values as the FP32 factorization reads them
    # |A - L L^T| <= gamma |L| |L^T|; a multiple of n + 1 for the blocks' inverses
    gamma = 4 * (n + 1) * (EPS64 if prec == FP64 else EPS32)
    assert np.all(np.abs(P - L @ L.T) <= gamma * (np.abs(L) @ np.abs(L).T))


def test_leaf_pivots_to_the_last_place():
    """FP64 leaf pivots sqrt(d) over the mantissas of two binades (diagonal
    matrix: every front is a leaf).  The second Newton step r' = r (3/2 - d r^2 / 2)
    rounds d r^2 / 2 (about 1/2) three times and its difference and product once
    each, l = d r' once more: less than 4 units u = eps / 2 in all, against up to
    1.5 2^-48 = 24 eps from one step on an estimate of 24 bits."""
    n = 4096
    d = np.random.default_rng(5).uniform(1.0, 4.0, n)
    f = Factor(Symbolic(n, np.arange(n + 1, dtype=np.int64), np.arange(n, dtype=np.int32)), FP64, max_nrhs=1)
    f.numeric(dev(d))
    Lp, Li, Lx = f.export_L()
    L = np.zeros(n)
    L[f.sym.export()["perm"]] = Lx[Lp[:-1]]
    ref = np.sqrt(d.astype(np.longdouble))
    worst = float((np.abs(L - ref) / ref).max() / EPS64)
    print(f"largest error {worst:.2f} eps", flush=True)
    assert worst <= 2.0


def test_pivots_of_leaves_past_the_leaf_kernel():
    """The same bound for leaves of 64 pivots under 200 rows, which do not fit
    the leaf kernel's LDS and are factored by the panel kernel: diagonal values,
    stored zeros elsewhere."""
    p, s, blocks = 64, 200, 12
    n = p * blocks + s
    keep = np.zeros((n, n), bool)
    for b in range(blocks):
        keep[b * p:(b + 1) * p, b * p:(b + 1) * p] = True
    keep[blocks * p:] = True
    keep = np.tril(keep)
    colptr = np.concatenate([[0], np.cumsum(keep.sum(0))]).astype(np.int64)
    rowind = np.concatenate([np.flatnonzero(keep[:, c]) for c in range(n)]).astype(np.int32)
    d = np.random.default_rng(6).uniform(1.0, 4.0, n)
    values = np.zeros(rowind.size)
    values[colptr[:-1]] = d
    sym = Symbolic(n, colptr, rowind, user_perm=np.arange(n))
    ex = sym.export()
    leaves = blocks - 1                      # the last block joins the border's front
    assert list(np.diff(ex["relaxed_ptr"])) == [p] * leaves + [p + s] and ex["front_order"][0] == p + s
    f = Factor(sym, FP64, max_nrhs=1)
    f.numeric(dev(values))
    Lp, Li, Lx = f.export_L()
    ref = np.sqrt(d[:p * leaves].astype(np.longdouble))
    worst = float((np.abs(Lx[Lp[:-1]][:p * leaves] - ref) / ref).max() / EPS64)
    print(f"largest error {worst:.2f} eps", flush=True)
    assert worst <= 2.0
