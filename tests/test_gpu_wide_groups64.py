"""FP64 wide tables in groups of 64 columns (up to 64 columns, an odd number of such
groups above 128, few blocks) and of 128 (65 to 128 columns, an even number of 64s
with many blocks), around the sizes where the choice changes: integer columns and
pairs exact, the others to 1e-12, plain and in groups."""
import numpy as np
import pytest

from helpers import corr_scaled_err, current_stream, lib

pytestmark = pytest.mark.gpu


def _table(n, p):
    """FP64 rows on the GPU: every other column integers up to 2000 (sums of products stay below 2^53)."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(1000 * n + p)
    x = torch.randint(-2000, 2001, (n, p), generator=g, device="cuda:0").double()
    x[:, 1::2] += torch.rand((n, p // 2), generator=g, device="cuda:0", dtype=torch.float64)
    torch.cuda.synchronize()
    return x


def _columns(L, p):
    return [(L.STATS_F64, 0, 8 * c, L.STATS_COL_INTEGER if c % 2 == 0 else 0) for c in range(p)]


def _check(x, raw, cov):
    y = x[:, ::2]
    C = np.array([[int(v) for v in row[::2]] for row in raw["C_int"][::2]], dtype=np.float64)
    assert raw["n"] == len(x)
    assert [raw["s_int"][c] for c in range(0, x.shape[1], 2)] == [int(v) for v in y.sum(0).tolist()]
    assert np.array_equal(C, (y.T @ y).cpu().numpy())
    d = x - x.mean(0)
    assert corr_scaled_err(cov, (d.T @ d / (len(x) - 1)).cpu().numpy()) <= 1e-12


# 342 blocks of three pairs of 128 are more than 1024 workgroups, 341 are not
@pytest.mark.parametrize("p,n", [(63, 1057), (64, 1500), (128, 1024), (192, 1057), (193, 2049), (193, 341 * 1024),
                                 (193, 341 * 1024 + 1), (320, 1100)])
def test_rows(p, n):
    L = lib()
    x = _table(n, p)
    h = L.stats_open(L.make_config(_columns(L, p), [8 * p], stream=current_stream(), block_rows=1024,
                                   precision=L.STATS_PREC_FP64))
    try:
        L.stats_accumulate(h, [x], n)
        raw = L.stats_raw(h, p)
        cov = L.stats_finalize(h, p)["cov"]
    finally:
        L.stats_close(h)
    _check(x, raw, cov)


@pytest.mark.parametrize("p", [63, 65, 128, 129, 200])
def test_groups(p):
    L = lib()
    off = np.array([0, 700, 700, 731, 6000], dtype=np.int64)
    x = _table(int(off[-1]), p)
    h = L.stats_open_groups(L.make_config(_columns(L, p), [8 * p], stream=current_stream()), len(off) - 1)
    try:
        L.stats_accumulate_segmented(h, [x], off)
        fin = L.stats_finalize_groups(h, len(off) - 1, p)
        for g in range(len(off) - 1):
            if off[g + 1] > off[g]:
                _check(x[off[g]:off[g + 1]], L.stats_group_raw(h, g, p), fin["cov"][g])
    finally:
        L.stats_close(h)
