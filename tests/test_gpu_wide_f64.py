"""FP64 matrix-core kernel of wide tables against the CPU oracle: column counts
at the edges of its 16-column strips and 128-column groups, row counts at the
edges of its 32-row stages, every element type, groups, and planes."""
import numpy as np
import pytest

import oracle
from helpers import check_raw_against_oracle, corr_scaled_err, current_stream, lib, to_dev

pytestmark = pytest.mark.gpu


def _columns(seed, n, p, dtypes):
    """Values per column: integers or Gaussians, every fifth FP column flagged integer."""
    L = lib()
    rng = np.random.default_rng([seed, n, p])
    arrs, is_int, flags = [], [], []
    for c in range(p):
        dt = np.dtype(dtypes[c % len(dtypes)])
        flag = dt.kind == "f" and c % 5 == 4
        x = rng.integers(-3000, 3000, n) if dt.kind == "i" or flag else rng.normal(3.0 * c, 1.0 + c % 7, n)
        arrs.append(x.astype(dt))
        is_int.append(dt.kind == "i" or flag)
        flags.append(L.STATS_COL_INTEGER if flag else 0)
    return arrs, is_int, flags


def _check(raw, fin_cov, arrs, is_int):
    st = oracle.sufficient_stats(arrs, is_int)
    check_raw_against_oracle(raw, st, is_int)
    if st.n > 1:
        # co-moments against the centred products in FP64 (two passes)
        x = np.stack([a.astype(np.float64) for a in arrs], axis=1)
        d = x - x.mean(0)
        assert corr_scaled_err(fin_cov, d.T @ d / (st.n - 1)) <= 1e-12


@pytest.mark.parametrize("p,n", [(33, 1), (48, 31), (64, 32), (65, 33), (101, 1057), (127, 63), (128, 64), (129, 65),
                                 (144, 1024), (257, 1025), (300, 40)])
def test_fp64_rows(p, n):
    print(f"wide f64 p={p} n={n}", flush=True)
    L = lib()
    arrs, is_int, flags = _columns(1, n, p, [np.float64])
    cols = [(L.STATS_F64, 0, 8 * c, flags[c]) for c in range(p)]
    h = L.stats_open(L.make_config(cols, [8 * p], stream=current_stream(), block_rows=1024))
    try:
        L.stats_accumulate(h, [to_dev(np.stack(arrs, axis=1))], n)
        raw = L.stats_raw(h, p)
        cov = L.stats_finalize(h, p)["cov"] if n > 1 else None
    finally:
        L.stats_close(h)
    _check(raw, cov, arrs, is_int)


@pytest.mark.parametrize("dtypes", [[np.int32], [np.int64, np.float32, np.float64, np.int32], [np.float32]])
def test_types_in_planes(dtypes):
    # four planes of interleaved columns of one type each, FP64 mode
    L = lib()
    n, p = 2081, 70
    arrs, is_int, flags = _columns(2, n, p, dtypes)
    kinds = sorted({np.dtype(d).str for d in dtypes})
    cols, planes, strides = [None] * p, [], []
    for k, ks in enumerate(kinds):
        mine = [c for c in range(p) if arrs[c].dtype.str == ks]
        es = np.dtype(ks).itemsize
        planes.append(to_dev(np.stack([arrs[c] for c in mine], axis=1)))
        strides.append(es * len(mine))
        for i, c in enumerate(mine):
            cols[c] = (L.DTYPE_CODE[np.dtype(ks)], k, es * i, flags[c])
    h = L.stats_open(L.make_config(cols, strides, stream=current_stream(), precision=L.STATS_PREC_FP64))
    try:
        L.stats_accumulate(h, planes, n)
        raw = L.stats_raw(h, p)
        cov = L.stats_finalize(h, p)["cov"]
    finally:
        L.stats_close(h)
    _check(raw, cov, arrs, is_int)


@pytest.mark.parametrize("p", [40, 130])
def test_groups(p):
    L = lib()
    sizes = [33, 0, 1, 5000, 64]
    off = np.concatenate([[0], np.cumsum(sizes)])
    arrs, is_int, flags = _columns(3, int(off[-1]), p, [np.float64])
    cols = [(L.STATS_F64, 0, 8 * c, flags[c]) for c in range(p)]
    h = L.stats_open_groups(L.make_config(cols, [8 * p], stream=current_stream(), block_rows=2048), len(sizes))
    try:
        L.stats_accumulate_segmented(h, [to_dev(np.stack(arrs, axis=1))], off)
        raws = [L.stats_group_raw(h, g, p) for g in range(len(sizes))]
        fin = L.stats_finalize_groups(h, len(sizes), p)
    finally:
        L.stats_close(h)
    for g, n in enumerate(sizes):
        if n:
            _check(raws[g], fin["cov"][g], [a[off[g]:off[g + 1]] for a in arrs], is_int)
