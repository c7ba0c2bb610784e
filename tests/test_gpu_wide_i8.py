"""Int8 matrix-core kernel of wide FP32 tables against the CPU oracle: row counts
at the edges of its 32-row sub-steps and of its three-slot ring of raw rows,
column counts at the edges of its 32-column tiles and 128-column groups.  The
values are integers below 2^18 (on every block's grid), so each product sum is
exact before one FP64 rounding: 1e-12 leaves room for the merge of the blocks.
The state holds means, so a column's sum carries one rounding at the size of its
values times the row count, which matters where the sum nearly cancels."""
import numpy as np
import pytest

import oracle
from helpers import corr_scaled_err, current_stream, lib, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F,extra", [(36, 0), (96, 1), (128, 0), (132, 1), (164, 2), (228, 0), (256, 1), (260, 0)])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 97, 128, 129, 161, 1024 + 127])
def test_i8_sub_steps_and_tiles(F, extra, n):
    print(f"wide i8 F={F} extra={extra} n={n}", flush=True)
    L = lib()
    rng = np.random.default_rng([F, extra, n])
    x = rng.integers(-(1 << 17), 1 << 17, (n, F)).astype(np.float32)
    ex = [np.arange(1, n + 1, dtype=np.int32), rng.normal(0.0, 3.0, n)][:extra]
    p = F + extra
    cols = [(L.STATS_F32, 0, 4 * c, 0) for c in range(F)] + [(L.STATS_I32, 1, 0, 0), (L.STATS_F64, 2, 0, 0)][:extra]
    h = L.stats_open(L.make_config(cols, [4 * F, 4, 8][:1 + extra], stream=current_stream(), block_rows=1024,
                                   precision=L.STATS_PREC_SPLIT))
    try:
        L.stats_accumulate(h, [to_dev(x)] + [to_dev(e) for e in ex], n)
        raw = L.stats_raw(h, p)
        cov = L.stats_finalize(h, p)["cov"] if n > 1 else None
    finally:
        L.stats_close(h)
    is_int = [False] * F + [True, False][:extra]
    arrs = [x[:, c] for c in range(F)] + ex
    st = oracle.sufficient_stats(arrs, is_int)
    assert raw["n"] == n
    for c, a in enumerate(arrs):
        ref = st.s_int[c] if is_int[c] else float(st.s_exact[c])
        tol = 0 if is_int[c] else 1e-12 * abs(ref) + n * 2.0 ** -52 * np.abs(a).max()
        assert abs((raw["s_int"] if is_int[c] else raw["s_f64"])[c] - ref) <= tol, c
    if n > 1:
        d = np.stack([a.astype(np.float64) for a in arrs], axis=1)
        d -= d.mean(0)
        assert corr_scaled_err(cov, d.T @ d / (n - 1)) <= 1e-12
