"""The expansion of the stored triangle into full rows at the edges of its
chunks (2048 entries, an eighth of the chunks per XCD): tridiagonal matrices of
whole numbers, so every product A x is exact.
"""
import numpy as np
import pytest

from tests.test_gpu_parity import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from paper_2007_01541_amd import FP64, Factor, Symbolic  # noqa: E402


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
