"""Chunks of up to 4096 rows cut into shorter blocks give what one block gives:
the sums of blocks with one shift are added before a mean is taken of them, so no
covariance holds the rounding of a block's mean and one infinity is no undefined mean.

Values 10^12 + integers of 0..999: the shifted sums are exact, so a covariance has
five roundings (S / n, S * that, Q - that, / (n - 1), the reference's) of
quantities of at most 4 M2 (columns of 300 rows and more: |shift - mean| < 1.8 standard
deviations): 10 * 2^-53 of the standard deviations' product, bounded with 32.  A
mean has two roundings of its own size and the reference's."""
import numpy as np
import pytest

from helpers import current_stream, lib, to_dev
from test_gpu_small_chunks import _layout

pytestmark = pytest.mark.gpu

U = 2.0**-53
KINDS = [("rows", 3), ("rows", 10), ("rows", 16), ("noalloc", 10), ("planes", 4), ("planes", 13), ("generic", 5),
         ("mixed24", 1), ("mixed24", 2), ("mixed24", 3), ("records", 20)]


def _planes(kind, x):
    """_layout with no column declared whole and FP64 or int64 values that hold these."""
    L = lib()
    n, p = x.shape
    if kind in ("planes", "generic"):  # generic: every second plane int64
        it = [kind == "generic" and c % 2 == 1 for c in range(p)]
        return ([(L.STATS_I64 if it[c] else L.STATS_F64, c, 0, 0) for c in range(p)], [8] * p,
                [to_dev(x[:, c].astype(np.int64 if it[c] else np.float64)) for c in range(p)])
    if kind == "mixed24":
        rec = np.zeros((n, 3))
        rec[:, :p] = x
        cols = [(L.STATS_F64, 0, 8 * c, 0) for c in range(p)]
        if p > 1:
            rec.view(np.int64)[:, p - 1] = x[:, p - 1].astype(np.int64)
            cols[-1] = (L.STATS_I64, 0, 8 * (p - 1), 0)
        return cols, [24], [to_dev(rec)]
    cols, strides, planes = _layout(kind, x)
    return [(t, pl, off, 0) for t, pl, off, _ in cols], strides, planes


def _check_moments(x, mean, cov):
    n, p = x.shape
    d = (x - 1e12).astype(np.int64)
    s, q = d.sum(0), d.T @ d
    ref = np.array([[(n * int(q[i, j]) - int(s[i]) * int(s[j])) / (n * (n - 1)) for j in range(p)] for i in range(p)])
    sd = np.sqrt(np.diag(ref))
    err = np.max(np.abs(cov - ref) / np.outer(sd, sd))
    assert err <= 32 * U, err
    assert np.max(np.abs(mean - (1e12 + s / n))) <= 4 * U * 1e12


def _values(n, p):
    return 1e12 + np.random.default_rng([n, p]).integers(0, 1000, (n, p)).astype(np.float64)


@pytest.mark.parametrize("kind,p", KINDS)
@pytest.mark.parametrize("n", [300, 1025, 4096])
def test_far_from_zero(kind, p, n):
    print(f"short blocks {kind} p={p} n={n}", flush=True)
    import torch
    L = lib()
    x = _values(n, p)
    cols, strides, planes = _planes(kind, x)
    h = L.stats_open(L.make_config(cols, strides, stream=current_stream(), precision=L.STATS_PREC_FP64))
    torch.cuda.synchronize()
    try:
        (L.stats_accumulate_noalloc if kind == "noalloc" else L.stats_accumulate)(h, planes, n)
        got = L.stats_finalize(h, p)
    finally:
        L.stats_close(h)
    _check_moments(x, got["mean"], got["cov"])


@pytest.mark.parametrize("kind,p", KINDS)
def test_one_infinity(kind, p):
    print(f"short blocks, infinity {kind} p={p}", flush=True)
    import torch
    L = lib()
    n = 3000
    x = _values(n, p)
    cols, strides, planes = _planes(kind, x)
    first = planes[0].view(torch.float64).reshape(n, -1)
    first[1500, 0] = -np.inf  # column 0
    h = L.stats_open(L.make_config(cols, strides, stream=current_stream(), precision=L.STATS_PREC_FP64))
    torch.cuda.synchronize()
    try:
        (L.stats_accumulate_noalloc if kind == "noalloc" else L.stats_accumulate)(h, planes, n)
        got = L.stats_finalize(h, p)
    finally:
        L.stats_close(h)
    assert got["mean"][0] == -np.inf
    if p > 1:
        assert np.max(np.abs(got["mean"][1:] - x[:, 1:].mean(0, dtype=np.longdouble))) <= 4 * U * 1e12


def _pairwise(x):
    import torch
    L = lib()
    n, p = x.shape
    h = L.stats_open(L.make_config([(L.STATS_F64, 0, 8 * c, 0) for c in range(p)], [8 * p],
                                   stream=current_stream(), pairwise=True))
    planes = [to_dev(x)]
    torch.cuda.synchronize()
    try:
        L.stats_accumulate(h, planes, n)
        return L.stats_finalize_pairwise(h, p)
    finally:
        L.stats_close(h)


# the three packings of the pairwise kernel
@pytest.mark.parametrize("p", [1, 4, 7, 13])
@pytest.mark.parametrize("n", [300, 1025, 4096])
def test_pairwise_far_from_zero(p, n):
    print(f"short blocks, pairwise p={p} n={n}", flush=True)
    x = _values(n, p)
    got = _pairwise(x)
    assert np.all(got["n"] == n)
    _check_moments(x, got["mean"], got["cov"])


@pytest.mark.parametrize("p", [4, 7, 13])
@pytest.mark.parametrize("n,rows", [(3000, 700), (200_000, 1500)])
def test_pairwise_missing_and_infinity(p, n, rows):
    """Column 1 is missing beyond its first rows, so whole blocks hold none of it: its
    moments and the pair's are those of the first rows alone.  Column 2's infinity
    gives an infinite mean."""
    print(f"short blocks, pairwise with missing values p={p} n={n}", flush=True)
    x = _values(n, p)
    x[rows:, 1] = np.nan
    x[rows + 100, 2] = np.inf
    got = _pairwise(x)
    assert got["n"][0, 1] == rows and got["n"][0, 0] == n
    if n <= 4096:
        assert got["mean"][2] == np.inf
    y = x[:rows, :2]  # column 0's own mean and variance are over all rows: y's instead
    _check_moments(y, np.array([(y[:, 0] - 1e12).mean() + 1e12, got["mean"][1]]),
                   np.array([[np.var(y[:, 0] - 1e12, ddof=1), got["cov"][0, 1]], got["cov"][1, :2]]))
