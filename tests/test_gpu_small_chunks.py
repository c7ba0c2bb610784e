"""Small chunks are cut into blocks of 256 to 1024 rows, whose shift is the first
row of the 4096 they lie in: an outlier in a short block's first row counts once
against the 2^53 guard, as in blocks of 4096 rows, not once for every row of it.
Every kernel that takes such blocks, exact against the oracle."""
import numpy as np
import pytest

import oracle
from helpers import check_raw_against_oracle, current_stream, lib, to_dev

pytestmark = pytest.mark.gpu

OUT = 20_000_000  # fifteen of them in 4096 rows: 6.0e15 < 2^53; one per row of 256: 1.0e17


def _rows(n, p):
    rng = np.random.default_rng([n, p])
    x = rng.integers(0, 100, (n, p)).astype(np.float64)
    r = np.arange(n)
    x[(r % 256 == 0) & (r % 4096 != 0)] = OUT
    return x


def _layout(kind, x):
    """(columns, strides, planes) of the kernel named."""
    L = lib()
    n, p = x.shape
    if kind in ("rows", "noalloc"):  # interleaved FP64
        return [(L.STATS_F64, 0, 8 * c, L.STATS_COL_INTEGER) for c in range(p)], [8 * p], [to_dev(x)]
    if kind == "planes":  # int32 planes
        return [(L.STATS_I32, c, 0, 0) for c in range(p)], [4] * p, [to_dev(x[:, c].astype(np.int32)) for c in range(p)]
    if kind == "generic":  # planes of several types
        dt = [(L.STATS_I64, np.int64, 8), (L.STATS_I32, np.int32, 4), (L.STATS_F32, np.float32, 4)]
        return ([(dt[c % 3][0], c, 0, L.STATS_COL_INTEGER if c % 3 == 2 else 0) for c in range(p)],
                [dt[c % 3][2] for c in range(p)], [to_dev(x[:, c].astype(dt[c % 3][1])) for c in range(p)])
    if kind.startswith("mixed"):  # records of several types, "mixed" and their bytes
        dt = [np.dtype(t) for t in (np.int32, np.float32, np.float64, np.int64)[:p]]
        offs = np.cumsum([0] + [d.itemsize for d in dt[:-1]]).tolist()
        rec = np.zeros(n, dtype=np.dtype({"names": [str(c) for c in range(p)], "formats": dt, "offsets": offs,
                                          "itemsize": int(kind[5:])}))
        for c in range(p):
            rec[str(c)] = x[:, c]
        cols = [(L.DTYPE_CODE[d], 0, offs[c], L.STATS_COL_INTEGER if d.kind == "f" else 0) for c, d in enumerate(dt)]
        return cols, [int(kind[5:])], [to_dev(rec.view(np.uint8))]
    y = np.zeros((n, 32))  # 256-byte records
    y[:, :p] = x
    return [(L.STATS_F64, 0, 8 * c, L.STATS_COL_INTEGER) for c in range(p)], [256], [to_dev(y)]


def _check(kind, p, n):
    import torch
    print(f"small chunk {kind} p={p} n={n}", flush=True)
    L = lib()
    x = _rows(n, p)
    cols, strides, planes = _layout(kind, x)
    h = L.stats_open(L.make_config(cols, strides, stream=current_stream(), precision=L.STATS_PREC_FP64))
    torch.cuda.synchronize()
    try:
        (L.stats_accumulate_noalloc if kind == "noalloc" else L.stats_accumulate)(h, planes, n)
        raw = L.stats_raw(h, p)
    finally:
        L.stats_close(h)
    st = oracle.sufficient_stats(oracle.columns_of(x), [True] * p)
    check_raw_against_oracle(raw, st, [True] * p)


@pytest.mark.parametrize("kind,p", [("rows", 3), ("rows", 10), ("rows", 16), ("noalloc", 10), ("planes", 4),
                                    ("generic", 1), ("generic", 5), ("records", 20)])
@pytest.mark.parametrize("n", [700, 65_537, 131_072, 131_073, 200_001, 262_144])
def test_outliers_in_first_rows(kind, p, n):
    _check(kind, p, n)


# one column (a row per lane), two of mixed types in rows up to 16 bytes (the same)
# and beyond or more (a column per lane, blocks of 1024 and 2048 rows to 1,572,864)
@pytest.mark.parametrize("kind,p", [("mixed8", 1), ("mixed8", 2), ("mixed16", 2), ("mixed24", 2), ("mixed24", 3),
                                    ("mixed24", 4)])
@pytest.mark.parametrize("n", [1, 262_145, 786_432, 786_433, 1_572_865])
def test_few_columns(kind, p, n):
    _check(kind, p, n)
