"""Missing values at the edges of the pairwise kernel: column counts of each
operand packing (4, 8, 16), row counts around its stages, storage types alone
and mixed, columns that start missing or hold nothing."""
import numpy as np
import pytest

import oracle
from helpers import current_stream, lib, to_dev
from test_gpu_pairwise import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["f64", "f32", "mixed"])
@pytest.mark.parametrize("p,n", [(1, 255), (4, 257), (4, 4099), (5, 127), (8, 128), (8, 3001), (9, 129), (13, 1),
                                 (16, 5000)])
def test_packings(p, n, kind):
    print(f"pairwise {kind} p={p} n={n}", flush=True)
    L = lib()
    rng = np.random.default_rng([p, n])
    dts = [np.dtype({"f64": np.float64, "f32": np.float32, "mixed": (np.float32, np.float64)[c % 2]}[kind])
           for c in range(p)]
    x = rng.normal(np.linspace(-300, 300, p), np.linspace(0.5, 20, p), (n, p))
    x[rng.random((n, p)) < 0.15] = np.nan
    if p > 2:
        x[: min(n, 40), 1] = np.nan  # shift found late
        x[:, 2] = np.nan             # a column without a value
    offs = [8 * c for c in range(p)]
    rec = np.zeros(n, dtype=np.dtype({"names": [f"c{c}" for c in range(p)], "formats": dts, "offsets": offs,
                                      "itemsize": 8 * p}))
    for c in range(p):
        rec[f"c{c}"] = x[:, c]
    cols = [(L.DTYPE_CODE[dts[c]], 0, offs[c], 0) for c in range(p)]
    h = L.stats_open(L.make_config(cols, [8 * p], stream=current_stream(), pairwise=True))
    try:
        L.stats_accumulate(h, [to_dev(rec.view(np.uint8).reshape(n, 8 * p))], n)
        got = L.stats_finalize_pairwise(h, p)
    finally:
        L.stats_close(h)
    with np.errstate(all="ignore"):
        ref = oracle.pairwise_stats([np.ascontiguousarray(rec[f"c{c}"]) for c in range(p)])
    _check(got, ref)
