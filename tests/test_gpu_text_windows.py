"""Segments of text with more lines than the workgroup's line table holds: the
table is sized from the chunk's mean line length, or, for a last chunk, from an
earlier one's, so uneven or changing line lengths fill it several times.  The
block shift stays the segment's first row (large identifiers stay inside the
2^53 guard, decimals keep their digits), and converted values equal Python's."""
import numpy as np
import pytest

import oracle
from helpers import aos_config, check_raw_against_oracle, corr_scaled_err, current_stream, lib

pytestmark = pytest.mark.gpu

ISINT = [True, False]
BASE = 1_000_000_000  # identifiers: their squares alone leave the guard


def _lines(n, length, k0):
    """n lines of `length` bytes: an identifier, and a decimal near 1e8 with zeros in front."""
    out = []
    for k in range(k0, k0 + n):
        f = "%d,%.6f" % (BASE + k, 1e8 + (k * 7919 % 1000) * 1e-3)
        i = f.index(",") + 1
        out.append(f[:i] + "0" * (length - 1 - len(f)) + f[i:])
    return ("\n".join(out) + "\n").encode()


def _rows(txt):
    return np.array([[float(x) for x in ln.split(",")] for ln in txt.decode().split()])


def _dev(b):
    import torch
    return torch.frombuffer(bytearray(b) + b"\0" * 16, dtype=torch.uint8).to("cuda:0")


def _check(h, rows, L):
    raw, fin = L.stats_raw(h, 2), L.stats_finalize(h, 2, mask=[0, 1])
    st = oracle.sufficient_stats(oracle.columns_of(rows), ISINT)
    ref = oracle.finalize(st, mask=[0, 1])
    check_raw_against_oracle(raw, st, ISINT)
    assert fin["cov"][0, 0] == ref["cov"][0, 0]
    # block means are held in FP64: an error of u |mean| in each, against the column's
    # spread, through a merge tree of some eight levels (unshifted sums of squares
    # would lose u mean^2 / sd^2, more than all digits here)
    assert corr_scaled_err(fin["cov"], ref["cov"]) <= 16 * 2.0 ** -53 * 1e8 / ref["cov"][1, 1] ** 0.5


# (long lines, their length, short lines, their length): short lines without one
# starting in the segment's first slice, a little over the table, many windows
@pytest.mark.parametrize("nl,ll,ns,ls", [(750, 4000, 1200, 400), (750, 4000, 4000, 180), (600, 3000, 20_000, 40)])
def test_uneven_lines(nl, ll, ns, ls):
    import torch
    L = lib()
    txt = _lines(nl, ll, 0) + _lines(ns, ls, nl)
    rows = _rows(txt)
    buf = _dev(txt)
    h = L.stats_open(aos_config(p=2, int_cols=ISINT, stream=current_stream()))
    try:
        assert L.stats_accumulate_text(h, buf, len(txt), is_last=True) == len(txt)
        _check(h, rows, L)
        out = torch.zeros((len(rows), 2), dtype=torch.float64, device="cuda:0")
        torch.cuda.synchronize()
        assert L.stats_text_to_binary(h, buf, len(txt), [out], len(rows), is_last=True) == (len(rows), len(txt))
        assert np.array_equal(out.cpu().numpy().view(np.uint64), rows.view(np.uint64))
    finally:
        L.stats_close(h)


def test_shorter_lines_in_the_last_chunk():
    L = lib()
    a, b = _lines(400, 3000, 0), _lines(9000, 350, 400) + _lines(9000, 30, 9400)
    h = L.stats_open(aos_config(p=2, int_cols=ISINT, stream=current_stream()))
    try:
        assert L.stats_accumulate_text(h, _dev(a), len(a)) == len(a)
        assert L.stats_accumulate_text(h, _dev(b), len(b), is_last=True) == len(b)
        _check(h, _rows(a + b), L)
    finally:
        L.stats_close(h)
