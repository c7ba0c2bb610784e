"""Correlation matrices with many equal eigenvalues (identity, equicorrelated and
collinear columns, fewer rows than columns) and undefined ones (a constant column,
N <= ddof): clusters on both sides of the largest that the whole-GPU solver
orthogonalises, results against LAPACK, and no call that takes seconds (one
workgroup took 2.5 s over the 1023 equal eigenvalues of 1024 columns)."""
import time

import numpy as np
import pytest

from helpers import lib
from test_gpu_eigen import check, finalize_of, matrix, unit

pytestmark = pytest.mark.gpu


def _block(q, m, seed=0):
    """m eigenvalues of 0.5 (m + 1 equicorrelated columns) beside separate ones."""
    G = np.random.default_rng([q, m, seed]).standard_normal((q - m - 1, 3 * q))
    A = np.zeros((q, q))
    A[:m + 1, :m + 1] = 0.5
    A[m + 1:, m + 1:] = unit(G @ G.T)
    np.fill_diagonal(A, 1.0)
    return A


@pytest.mark.parametrize("q,m", [(25, 10), (40, 36), (60, 50), (100, 90), (260, 255), (400, 256), (400, 257), (520, 300)])
def test_clusters(q, m):
    A = _block(q, m)
    check(A, finalize_of(A))


@pytest.mark.parametrize("q", [25, 41, 60, 61, 130, 300])
@pytest.mark.parametrize("rank", [1, 2, 7])
def test_fewer_rows_than_columns(q, rank):
    G = np.random.default_rng([q, rank]).standard_normal((q, rank))
    A = unit(G @ G.T)
    check(A, finalize_of(A))


@pytest.mark.parametrize("q", [24, 25, 60, 61, 130, 200])
def test_undefined(q):
    L = lib()
    A = matrix("random", q)
    A[2] = A[:, 2] = 0.0
    fin = finalize_of(A)
    ok = np.arange(q) != 2
    assert np.all(np.isnan(fin["corr"][2])) and np.array_equal(fin["corr"][np.ix_(ok, ok)], A[np.ix_(ok, ok)])
    assert all(np.all(np.isnan(fin[k])) for k in ("eigval", "eigvec", "var_pct", "cum_pct"))
    with pytest.raises(L.StatsError) as e:
        finalize_of(A, ddof=2)
    assert e.value.code == L.STATS_E_STATE


@pytest.mark.parametrize("kind", ["identity", "equi", "rank1", "constant"])
def test_1024_columns_in_time(kind):
    q = 1024
    A = matrix("identity" if kind == "constant" else kind, q)
    if kind == "constant":
        A[5, 5] = 0.0
    finalize_of(matrix("identity", 61))  # loads the kernels
    t = time.perf_counter()
    fin = finalize_of(A)
    t = time.perf_counter() - t
    print(f"1024 columns, {kind}: {t * 1e3:.0f} ms", flush=True)
    if kind == "constant":
        assert np.all(np.isnan(fin["eigval"]))
    else:
        check(A, fin)
    assert t < 1.0
