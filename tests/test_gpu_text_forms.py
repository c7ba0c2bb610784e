"""Text kernels at the edges of their paths (section "Data Representation and
Sufficient Statistics"): field forms on both sides of the eight-digit steps, the
64-bit significand, the power-of-ten table and exact rounding ties; texts whose
lengths surround the 4 KiB units, the 64 KiB groups of the line count and the
segments; every column count.  Converted values are compared bit for bit with
Python's correctly rounded float() (int() for integer columns)."""
import numpy as np
import pytest

from helpers import current_stream, lib

pytestmark = pytest.mark.gpu


def _dev(b: bytes, shift: int):
    """The text at an address that is shift modulo 16, 0xFF-free garbage around it."""
    import torch
    t = torch.full((len(b) + 64,), ord("7"), dtype=torch.uint8)
    t[16 + shift:16 + shift + len(b)] = torch.frombuffer(bytearray(b), dtype=torch.uint8)
    return t.to("cuda:0")[16 + shift:16 + shift + len(b)]


def _convert(txt, p, ints, n, shift=0):
    import torch
    L = lib()
    cols = [(L.STATS_F64, 0, 8 * k, 0) if not ints >> k & 1 else (L.STATS_I64, 0, 8 * k, L.STATS_COL_INTEGER) for k in range(p)]
    h = L.stats_open(L.make_config(cols, [8 * p], stream=current_stream()))
    try:
        buf = _dev(txt, shift)
        out = torch.zeros((max(n, 1), p), dtype=torch.int64, device="cuda:0")
        rows, used = L.stats_text_to_binary(h, buf, len(txt), [out], n, is_last=True)
    finally:
        L.stats_close(h)
    assert rows == n and used == len(txt)
    return out[:n].cpu().numpy()


def _decimals():
    rng = np.random.default_rng(11)
    f = ["0", "-0", "+0.0", "0.000000000000000000000000001", "1e27", "1E-27", "1e+28", "9e-57", "18446744073709551615",
         "9999999999999999999", "-9007199254740993", "9007199254740993.0", "4503599627370497.5", "0.30000000000000004",
         "12345678", "1234567.", ".5", "-.25e1", "123456789", "1.7976931348623157e20", "5e0", "5e-0", "1e005",
         "1152921504606846977", "36893488147419103233", "0.00000000000000000001"]
    for d in range(1, 21):  # digits before and after the point around the eight-digit steps
        s = "".join(str(x) for x in rng.integers(1, 10, 20))
        for pt in (0, 1, 7, 8, 9, 15, 16, 17):
            if pt <= d:
                f.append((s[:pt] or "0") + ("." + s[pt:d] if pt < d else ""))
    for q in range(-27, 28):  # exact ties and their neighbours, and random significands, at every power
        m = int(rng.integers(1 << 53, 1 << 54)) | 1
        tie = m * 5 ** min(max(-q, 0), 4)
        for w in (tie - 1, tie, tie + 1, int(rng.integers(1, 1 << 62)), int(rng.integers(1, 1 << 20))):
            f.append(f"{w}e{q}" if w % 3 else f"-{w}E{q:+d}")
    return f


@pytest.mark.parametrize("p", [1, 2, 13, 16])
def test_decimal_forms_bit_exact(p):
    f = _decimals()
    f += f[:-len(f) % p] if len(f) % p else []
    rows = [f[k:k + p] for k in range(0, len(f), p)]
    txt = "\n".join(",".join(r) for r in rows).encode()
    got = _convert(txt, p, 0, len(rows))
    want = np.array([[float(x) for x in r] for r in rows])
    assert np.array_equal(got, want.view(np.int64))


@pytest.mark.parametrize("p", [1, 3, 8])
def test_integer_forms_exact(p):
    f = [s + "9" * d for d in range(1, 19) for s in ("", "-", "+")] + ["0", "-0", "00000000000000001", "1" + "0" * 17,
                                                                      "-" + "0" * 20 + "7"]
    f += f[:-len(f) % p] if len(f) % p else []
    rows = [f[k:k + p] for k in range(0, len(f), p)]
    got = _convert(("\n".join(",".join(r) for r in rows) + "\n").encode(), p, (1 << p) - 1, len(rows))
    assert got.tolist() == [[int(x) for x in r] for r in rows]


@pytest.mark.parametrize("size", [4096, 8192, 24576, 65536, 131072])
@pytest.mark.parametrize("width", [1, 40])
def test_units_and_groups(size, width):
    """Texts whose last byte (a digit or the newline) lies around a boundary, at odd addresses."""
    rng = np.random.default_rng(size + width)
    for d, shift, end in ((-1, 0, "\n"), (0, 5, "\n"), (1, 15, ""), (0, 3, "")):
        lines, left = [], size + d - len(end)
        while True:
            frac = "".join(str(x) for x in rng.integers(0, 10, int(rng.integers(1, width + 1))))
            s = "%d,0.%s" % (len(lines) % 1000, frac)
            if left < 2 * len(s) + 60:  # the last line takes the rest, as leading zeros
                lines.append("0" * (left - len(s)) + s)
                break
            lines.append(s)
            left -= len(s) + 1
        txt = ("\n".join(lines) + end).encode()
        assert len(txt) == size + d
        want = [x.split(",") for x in lines]
        got = _convert(txt, 2, 1, len(want), shift)
        assert got[:, 0].tolist() == [int(x[0]) for x in want]
        assert np.array_equal(got[:, 1], np.array([float(x[1]) for x in want]).view(np.int64))
