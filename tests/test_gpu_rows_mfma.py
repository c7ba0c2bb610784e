"""Interleaved columns of any type, plain (p <= 32) and in groups (p <= 32), on
the matrix-core kernel with a column per lane, against the CPU oracle: every
row-group width (4, 8, 16 and 32 columns), element type, and row counts at the
edges of its stages."""
import numpy as np
import pytest

import oracle
from helpers import check_final_against_oracle, check_raw_against_oracle, corr_scaled_err, current_stream, lib, to_dev

pytestmark = pytest.mark.gpu

KINDS = {"f64": [np.float64], "f32": [np.float32], "i32": [np.int32],
         "mixed": [np.int64, np.float32, np.int32, np.float64]}


def _table(seed, n, p, kind, pad=8):
    """Row bytes (n, stride), columns, values and integer flags."""
    L = lib()
    rng = np.random.default_rng([seed, n, p])
    dts = [np.dtype(KINDS[kind][c % len(KINDS[kind])]) for c in range(p)]
    offs, at = [], 0
    for dt in dts:
        at = -(-at // dt.itemsize) * dt.itemsize
        offs.append(at)
        at += dt.itemsize
    align = max(dt.itemsize for dt in dts)
    stride = -(-(at + pad) // align) * align
    rec = np.zeros(n, dtype=np.dtype({"names": [f"c{c}" for c in range(p)], "formats": dts, "offsets": offs,
                                      "itemsize": stride}))
    arrs, is_int, cols = [], [], []
    for c, dt in enumerate(dts):
        # FP columns: every third one holds integers and is flagged so
        flag = dt.kind == "f" and c % 3 == 2
        x = rng.integers(-9000, 9000, n) if dt.kind == "i" or flag else rng.normal(50.0 * (c + 1), 2.0 + c, n)
        if dt == np.int64:
            x = x + (1 << 39)
        rec[f"c{c}"] = x.astype(dt)
        arrs.append(np.ascontiguousarray(rec[f"c{c}"]))
        is_int.append(dt.kind == "i" or flag)
        cols.append((L.DTYPE_CODE[dt], 0, offs[c], L.STATS_COL_INTEGER if flag else 0))
    return rec.view(np.uint8).reshape(n, stride), cols, stride, arrs, is_int


def _tol(ref):
    """1e-12, and what the merge of block records allows beside it: block means
    are FP64 (half an ulp each), so the deltas between blocks, in units of a
    column's spread, carry up to 2^-52 |mean| / sd per column of a pair."""
    sd = np.sqrt(np.maximum(np.diag(ref["cov"]), 1e-300))
    return 1e-12 + 2.0 ** -51 * float(np.max(np.abs(ref["mean"]) / sd))


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("p,n", [(1, 1), (3, 513), (4, 511), (5, 4097), (8, 255), (9, 129), (12, 20_001), (15, 1),
                                 (16, 127), (17, 128), (24, 4099), (31, 1025), (32, 130)])
def test_plain(kind, p, n):
    print(f"rows {kind} p={p} n={n}", flush=True)
    L = lib()
    data, cols, stride, arrs, is_int = _table(1, n, p, kind)
    h = L.stats_open(L.make_config(cols, [stride], stream=current_stream(), precision=L.STATS_PREC_FP64))
    try:
        L.stats_accumulate(h, [to_dev(data)], n)
        raw = L.stats_raw(h, p)
        fin = L.stats_finalize(h, p) if n > 1 else None
    finally:
        L.stats_close(h)
    st = oracle.sufficient_stats(arrs, is_int)
    check_raw_against_oracle(raw, st, is_int)
    if n > p:
        ref = oracle.finalize(st)
        check_final_against_oracle(fin, ref, is_int, tol=_tol(ref))


@pytest.mark.parametrize("kind,p", [("f64", 3), ("f64", 10), ("f32", 7), ("i32", 16), ("mixed", 13), ("f64", 24),
                                    ("mixed", 32)])
def test_groups(kind, p):
    print(f"groups {kind} p={p}", flush=True)
    L = lib()
    sizes = [1, 0, 130, 2, 5000, 127, 128, 9001]
    off = np.concatenate([[0], np.cumsum(sizes)])
    data, cols, stride, arrs, is_int = _table(2, int(off[-1]), p, kind, pad=0)
    h = L.stats_open_groups(L.make_config(cols, [stride], stream=current_stream(), block_rows=4096), len(sizes))
    try:
        L.stats_accumulate_segmented(h, [to_dev(data)], off)
        raws = [L.stats_group_raw(h, g, p) for g in range(len(sizes))]
        fin = L.stats_finalize_groups(h, len(sizes), p)
    finally:
        L.stats_close(h)
    for g, n in enumerate(sizes):
        assert fin["n"][g] == raws[g]["n"] == n
        if n == 0:
            continue
        st = oracle.sufficient_stats([a[off[g]:off[g + 1]] for a in arrs], is_int)
        check_raw_against_oracle(raws[g], st, is_int)
        if n > p:
            ref = oracle.finalize(st)
            assert corr_scaled_err(fin["cov"][g], ref["cov"]) <= _tol(ref)


def test_fraction_in_integer_column_and_missing_value():
    # one fraction in the last row of a checked FP32 column is refused; a NaN
    # spreads to its own column's pairs only
    L = lib()
    n, p = 777, 6
    x = np.arange(n * p, dtype=np.float32).reshape(n, p) % 97
    for bad in (True, False):
        y = x.copy()
        y[n - 1, 5 if bad else 1] = 0.5 if bad else np.nan
        cols = [(L.STATS_F32, 0, 4 * c, L.STATS_COL_INTEGER if c == 5 else 0) for c in range(p)]
        h = L.stats_open(L.make_config(cols, [4 * p], stream=current_stream()))
        try:
            L.stats_accumulate(h, [to_dev(y)], n)
            if bad:
                with pytest.raises(L.StatsError) as e:
                    L.stats_raw(h, p)
                assert e.value.code == L.STATS_E_INEXACT
            else:
                C = L.stats_raw(h, p)["C_f64"]
                assert np.array_equal(np.isnan(C), (np.arange(p) == 1)[:, None] | (np.arange(p) == 1)[None, :])
        finally:
            L.stats_close(h)
