"""Workloads of the statistics library: one pass from rows (or text) in GPU
memory to the finished statistics on the host.

Every case is a dict of plain values.  "kind" names the path:

  rows      row-major FP64 records of integer-valued columns (Table 1 of the
            paper: identifier, small integers, one real column)
  planes    one dense plane per column: nine int32 planes and an FP64 plane
  f32rows   row-major FP32 records, real-valued, 2 to 16 columns
  wide32    row-major FP32 table, 17 and more columns, and an int32 identifier
  wide64    row-major FP64 table, 17 and more columns
  groups    row-major FP64 records cut into many groups of uneven size
  text      CSV lines parsed and reduced in one pass
  convert   CSV lines converted to binary rows
  pairwise  FP64 records with missing entries (NaN)
"""
import math

import numpy as np
import torch

import paper_2604_23826_amd as L

DEV = "cuda:0"
INT, IDENT = L.STATS_COL_INTEGER, L.STATS_COL_IDENTIFIER


def listed():
    return [
        # an interactive query or a small partition: four chunks of a thousand rows, latency only
        dict(name="rows_tiny", kind="rows", n=4000, p=10, chunks=4),
        # a million Table-1 records (80 MB), the usual single-file table
        dict(name="rows_1e6", kind="rows", n=1_000_000, p=10, chunks=1),
        # 128-byte records, all sixteen columns of the narrow path, odd row count
        dict(name="rows_p16", kind="rows", n=10_000_007, p=16, chunks=1),
        # a GPU's share of the ten-column table in column planes, more than one launch's rows
        dict(name="planes_share", kind="planes", n=300_000_001, p=10, chunks=1),
        # single-precision measurements as most programs hold them
        dict(name="f32rows_p12", kind="f32rows", n=4_000_001, p=12, chunks=1),
        # a wide single-precision table (PCA of 256 features) with its identifier
        dict(name="wide32_256", kind="wide32", n=20_000_003, p=257, chunks=1),
        # a wide double-precision table of odd width
        dict(name="wide64_101", kind="wide64", n=4_000_003, p=101, chunks=1),
        # many 32-column tables of uneven size in one launch
        dict(name="groups_p32", kind="groups", p=32, ngroups=512, lo=1_000, hi=300_000),
        # thousands of small ten-column groups (per-customer statistics)
        dict(name="groups_p10", kind="groups", p=10, ngroups=4096, lo=100, hi=10_000),
        # the paper's first pipeline: CSV text straight into the statistics
        dict(name="text_8e6", kind="text", n=8_000_003, p=10, style="table1"),
        # the one-time CSV to binary conversion, general decimals
        dict(name="convert_2e6", kind="convert", n=2_000_001, p=8, style="decimal"),
        # incomplete data, pairwise-complete statistics
        dict(name="pairwise_p12", kind="pairwise", n=2_000_003, p=12, chunks=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rows", "planes", "f32rows", "wide32", "wide64", "groups", "text", "convert", "pairwise"])
    if kind == "rows":
        return dict(kind=kind, n=_logint(rng, 500, 20_000_000), p=rng.randint(2, 16), chunks=rng.randint(1, 4))
    if kind == "planes":
        return dict(kind=kind, n=_logint(rng, 5_000, 250_000_000), p=rng.randint(4, 10), chunks=rng.randint(1, 3))
    if kind == "f32rows":
        return dict(kind=kind, n=_logint(rng, 1_000, 20_000_000), p=rng.randint(2, 16), chunks=rng.randint(1, 3))
    if kind == "wide32":
        return dict(kind=kind, n=_logint(rng, 5_000, 20_000_000), p=rng.randint(18, 257), chunks=rng.randint(1, 2))
    if kind == "wide64":
        return dict(kind=kind, n=_logint(rng, 2_000, 4_000_000), p=rng.randint(17, 128), chunks=rng.randint(1, 2))
    if kind == "groups":
        lo = _logint(rng, 20, 2_000)
        hi = lo * _logint(rng, 2, 100)
        return dict(kind=kind, p=rng.choice([4, 10, 16, 24, 32]), ngroups=max(8, min(_logint(rng, 16, 4096), 20_000_000 // hi)),
                    lo=lo, hi=hi)
    if kind == "text":
        return dict(kind=kind, n=_logint(rng, 1_000, 8_000_000), p=rng.randint(2, 16),
                    style=rng.choice(["table1", "decimal"]))
    if kind == "convert":
        return dict(kind=kind, n=_logint(rng, 1_000, 2_000_000), p=rng.randint(2, 16),
                    style=rng.choice(["table1", "decimal"]))
    return dict(kind=kind, n=_logint(rng, 1_000, 4_000_000), p=rng.randint(2, 16), chunks=rng.randint(1, 2))


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * seed + 17)
    return g


def _luts():
    """Columns E..K of Table 1 as functions of B (3..8), C (1..10), D (1..100)."""
    E = [float(int(math.log(c) / math.log(b) * 100.0 + 1e-9)) for b in range(3, 9) for c in range(1, 11)]
    F = [float(round(math.log(d) / math.log(b) * 1e4)) for b in range(3, 9) for d in range(1, 101)]
    G = [float(int(abs(math.cos(c)) * 100.0)) for c in range(1, 11)]
    H = [float(int(abs(math.sin(d)) * 100.0)) for d in range(1, 101)]
    cot = [1.0 / math.tan(c) for c in range(1, 11)]
    Ic = [float(round(abs(t) * 1000.0)) for t in cot]
    K = [float(d // c) for c in range(1, 11) for d in range(1, 101)]
    return E, F, G, H, cot, Ic, K


# Table-1 columns in order: A B C D E F G H cotC I K, then uniform integers 0..100.
REAL_COL = 8


def _table1_cols(gen, row0, n, p):
    """Columns 0..p-1 of rows row0 .. row0 + n - 1, one tensor each (FP64)."""
    E, F, G, H, cot, Ic, K = [torch.tensor(t, dtype=torch.float64, device=DEV) for t in _luts()]
    b = torch.randint(0, 6, (n,), generator=gen, device=DEV, dtype=torch.int32)
    c = torch.randint(0, 10, (n,), generator=gen, device=DEV, dtype=torch.int32)
    d = torch.randint(0, 100, (n,), generator=gen, device=DEV, dtype=torch.int32)
    make = [lambda: torch.arange(row0 + 1, row0 + n + 1, device=DEV, dtype=torch.float64),
            lambda: (b + 3).double(), lambda: (c + 1).double(), lambda: (d + 1).double(),
            lambda: E[b * 10 + c], lambda: F[b * 100 + d], lambda: G[c], lambda: H[d],
            lambda: cot[c], lambda: Ic[c], lambda: K[c * 100 + d]]
    for k in range(p):
        if k < len(make):
            yield make[k]()
        else:
            yield torch.randint(0, 101, (n,), generator=gen, device=DEV, dtype=torch.int32).double()


def _table1_rows(gen, n, p, row0=0, step=1 << 23):
    x = torch.empty((n, p), dtype=torch.float64, device=DEV)
    for r in range(0, n, step):
        m = min(step, n - r)
        for k, col in enumerate(_table1_cols(gen, row0 + r, m, p)):
            x[r:r + m, k] = col
    return x


def _gauss(gen, n, p, dtype):
    """Correlated Gaussian rows: means 1e3..1e5, spreads 0.1..10 (a seeded
    mixing of p independent columns with uneven weights)."""
    mu = 10.0 ** (3.0 + 2.0 * torch.rand(p, generator=gen, device=DEV, dtype=torch.float64))
    sig = 10.0 ** (-1.0 + 2.0 * torch.rand(p, generator=gen, device=DEV, dtype=torch.float64))
    W = torch.randn((p, 2 * p), generator=gen, device=DEV, dtype=torch.float64)
    W = W @ W.T
    dd = W.diagonal().rsqrt()
    chol = torch.linalg.cholesky((W * dd[:, None] * dd[None, :]).cpu()).to(DEV)
    x = torch.empty((n, p), dtype=dtype, device=DEV)
    step = 1 << 20
    for r in range(0, n, step):
        m = min(step, n - r)
        z = torch.randn((m, p), generator=gen, device=DEV, dtype=torch.float64)
        x[r:r + m] = (mu + sig * (z @ chol.T)).to(dtype)
    return x


def _text_table(case, seed):
    """4096 distinct line tails (all fields after the identifier), as padded
    bytes, lengths and the values a correct parser reads."""
    rng = np.random.default_rng([seed, 7])
    p, rows, vals = case["p"], [], []
    E, F, G, H, cot, Ic, K = _luts()
    mu = 10.0 ** rng.uniform(0, 4, p)
    for _ in range(4096):
        f, v = [], []
        if case["style"] == "table1":
            b, c, d = rng.integers(0, 6), rng.integers(0, 10), rng.integers(0, 100)
            t = [b + 3, c + 1, d + 1, E[b * 10 + c], F[b * 100 + d], G[c], H[d], cot[c], Ic[c], K[c * 100 + d]]
            t += list(rng.integers(0, 101, 8))
            for k in range(1, p):
                s = "%.17g" % t[k - 1] if k == REAL_COL else "%d" % t[k - 1]
                f.append(s)
                v.append(float(s))
        else:  # general decimals: fixed point, %.17g and exponent forms, signs
            z = rng.standard_normal(p)
            for k in range(1, p):
                s = ("%.6f", "%.17g", "%.3f", "%.8e")[k % 4] % (mu[k] * z[k])
                f.append(s)
                v.append(float(s))
        rows.append(("," + ",".join(f) + "\n").encode())
        vals.append(v)
    width = max(map(len, rows))
    tab = np.zeros((4096, width), np.uint8)
    for i, r in enumerate(rows):
        tab[i, :len(r)] = np.frombuffer(r, np.uint8)
    return (torch.from_numpy(tab).to(DEV), torch.tensor([len(r) for r in rows], device=DEV),
            torch.tensor(vals, dtype=torch.float64, device=DEV))


def _text(case, seed):
    """CSV text of n lines (identifier 1..n first) and the index of each line's tail."""
    n = case["n"]
    tab, lens, vals = _text_table(case, seed)
    gen = _gen(seed)
    which = torch.randint(0, 4096, (n,), generator=gen, device=DEV)
    parts = []
    powers = torch.tensor([10 ** k for k in range(7, -1, -1)], device=DEV)
    step = 1 << 20
    for r in range(0, n, step):
        m = min(step, n - r)
        ids = torch.arange(r + 1, r + m + 1, device=DEV)[:, None]
        digits = (ids // powers) % 10 + 48
        w = which[r:r + m]
        line = torch.cat([digits.to(torch.uint8), tab[w]], dim=1)
        keep = torch.cat([ids >= powers, torch.arange(tab.shape[1], device=DEV) < lens[w][:, None]], dim=1)
        parts.append(line[keep])
    return torch.cat(parts), which, vals


def _text_is_int(case):
    return [k == 0 or (case["style"] == "table1" and k != REAL_COL) for k in range(case["p"])]


def _group_offsets(case, seed):
    rng = np.random.default_rng([seed, 4])
    sizes = np.floor(np.exp(rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["ngroups"]))).astype(np.int64)
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _inputs(case, seed):
    kind, p = case["kind"], case["p"]
    gen = _gen(seed)
    if kind == "rows":
        return [_table1_rows(gen, case["n"], p)]
    if kind == "planes":
        n, step = case["n"], 1 << 24
        planes = [torch.empty(n, dtype=torch.float64 if k == REAL_COL else torch.int32, device=DEV) for k in range(p)]
        for r in range(0, n, step):
            m = min(step, n - r)
            for k, col in enumerate(_table1_cols(gen, r, m, p)):
                planes[k][r:r + m] = col.to(planes[k].dtype)
        return planes
    if kind == "f32rows":
        return [_gauss(gen, case["n"], p, torch.float32)]
    if kind == "wide32":
        return [_gauss(gen, case["n"], p - 1, torch.float32),
                torch.arange(1, case["n"] + 1, device=DEV, dtype=torch.int32)]
    if kind == "wide64":
        return [_gauss(gen, case["n"], p, torch.float64)]
    if kind == "groups":
        off = _group_offsets(case, seed)
        return [_table1_rows(gen, int(off[-1]), p)]
    if kind == "pairwise":
        x = _gauss(gen, case["n"], p, torch.float64)
        step = 1 << 22
        for r in range(0, case["n"], step):
            u = torch.rand(x[r:r + step].shape, generator=gen, device=DEV)
            x[r:r + step][u < 0.05] = math.nan
        return [x]
    raise ValueError(kind)


# ---- handle and pass --------------------------------------------------------

def _table1_flags(k):
    return (0 if k == REAL_COL else INT) | (IDENT if k == 0 else 0)


def _config(case):
    kind, p = case["kind"], case["p"]
    stream = torch.cuda.current_stream().cuda_stream
    if kind in ("rows", "groups"):
        cols, strides = [(L.STATS_F64, 0, 8 * k, _table1_flags(k)) for k in range(p)], [8 * p]
    elif kind == "planes":
        cols = [(L.STATS_F64, k, 0, 0) if k == REAL_COL else (L.STATS_I32, k, 0, IDENT if k == 0 else 0) for k in range(p)]
        strides = [8 if k == REAL_COL else 4 for k in range(p)]
    elif kind == "f32rows":
        cols, strides = [(L.STATS_F32, 0, 4 * k, 0) for k in range(p)], [4 * p]
    elif kind == "wide32":
        cols = [(L.STATS_F32, 0, 4 * k, 0) for k in range(p - 1)] + [(L.STATS_I32, 1, 0, IDENT)]
        strides = [4 * (p - 1), 4]
    elif kind in ("wide64", "pairwise"):
        cols, strides = [(L.STATS_F64, 0, 8 * k, 0) for k in range(p)], [8 * p]
    else:  # text, convert: FP64 rows
        cols = [(L.STATS_F64, 0, 8 * k, (INT if i else 0) | (IDENT if k == 0 else 0))
                for k, i in enumerate(_text_is_int(case))]
        strides = [8 * p]
    return L.make_config(cols, strides, stream=stream, pairwise=kind == "pairwise")


class State:
    """Inputs and the open handle; the handle is closed with the state."""

    def __init__(self, case, seed):
        self.case = case
        if case["kind"] in ("text", "convert"):
            self.data = [_text(case, seed)[0]]
            self.out = torch.zeros((case["n"], case["p"]), dtype=torch.float64, device=DEV) if case["kind"] == "convert" else None
        else:
            self.data = _inputs(case, seed)
        torch.cuda.synchronize()
        self.offsets = _group_offsets(case, seed) if case["kind"] == "groups" else None
        cfg = _config(case)
        self.h = L.stats_open_groups(cfg, case["ngroups"]) if case["kind"] == "groups" else L.stats_open(cfg)

    def chunks(self):
        """(planes, rows) of each chunk; chunk starts fall on whole 16-byte units."""
        n, k = self.case["n"], self.case["chunks"]
        step = -(-n // (4 * k)) * 4
        return [([x[r:r + step] for x in self.data], min(step, n - r)) for r in range(0, n, step)]

    def __del__(self):
        if getattr(self, "h", None):
            L.stats_close(self.h)


def prepare(case, seed):
    return State(case, seed)


def run(state):
    case, h = state.case, state.h
    kind, p = case["kind"], case["p"]
    if kind == "convert":
        buf = state.data[0]
        rows, used = L.stats_text_to_binary(h, buf, buf.numel(), [state.out], case["n"], is_last=True)
        return {"rows": rows, "used": used, "out": state.out}
    L.stats_reset(h)
    if kind == "text":
        L.stats_accumulate_text(h, state.data[0], state.data[0].numel(), is_last=True)
        return L.stats_finalize(h, p)
    if kind == "groups":
        L.stats_accumulate_segmented(h, state.data, state.offsets)
        return L.stats_finalize_groups(h, case["ngroups"], p)
    for planes, rows in state.chunks():
        L.stats_accumulate(h, planes, rows)
    if kind == "pairwise":
        return L.stats_finalize_pairwise(h, p)
    return L.stats_finalize(h, p)


# ---- what a pass cannot do without -------------------------------------------

def _rows_of(case):
    if case["kind"] != "groups":
        return case["n"]
    lo, hi = case["lo"], case["hi"]
    return int(case["ngroups"] * (hi - lo) / math.log(hi / lo))  # mean of a log-uniform size


def work(case):
    kind, p, n = case["kind"], case["p"], _rows_of(case)
    out = 8 * (3 * p * p + 4 * p)
    if kind in ("rows", "wide64", "pairwise"):
        row = 8 * p
    elif kind == "groups":
        row, out = 8 * p, 8 * case["ngroups"] * (1 + p + p * p)
    elif kind == "planes":
        row = 4 * p + (4 if p > REAL_COL else 0)
    elif kind in ("f32rows", "wide32"):
        row = 4 * p
    else:  # mean characters per line: the identifier and the other fields
        row = 6 + (3.5 * p + (16 if p > REAL_COL else 0) if case["style"] == "table1" else 13.0 * p)
        if kind == "convert":
            out = 8 * p * n
    flops = p * (p + 1.0) * n * (4 if kind == "pairwise" else 1)
    if kind == "convert":
        flops = 0.0
    return {"bytes": float(row * n + out), "flops": float(flops)}


# ---- the same in 64 bits, without the library ---------------------------------

def _moments(blocks, p):
    """n, mean and centred cross products of the FP64 rows that blocks() yields (two passes)."""
    n, s, shift = 0, torch.zeros(p, dtype=torch.float64, device=DEV), None
    for x in blocks():
        if shift is None:
            shift = x[0].clone()
        n += x.shape[0]
        s += (x - shift).sum(0)
    mean = shift + s / n
    M, e = torch.zeros((p, p), dtype=torch.float64, device=DEV), torch.zeros(p, dtype=torch.float64, device=DEV)
    for x in blocks():
        d = x - mean
        e += d.sum(0)
        M += d.T.contiguous() @ d
    M -= torch.outer(e, e) / n
    return n, (mean + e / n).cpu().numpy(), M.cpu().numpy()


def _finished(n, mean, M, keep):
    mean, cov = mean[keep], (M / (n - 1))[np.ix_(keep, keep)]
    sd = np.sqrt(np.diag(cov))
    corr = cov / np.outer(sd, sd)
    np.fill_diagonal(corr, 1.0)
    w, v = np.linalg.eigh(corr)
    w, v = w[::-1], v[:, ::-1].T
    big = np.argmax(np.abs(v), axis=1)
    v = v * np.sign(v[np.arange(len(w)), big])[:, None]
    pct = 100.0 * w / w.sum()
    return {"mean": mean, "cov": cov, "corr": corr, "eigval": w.copy(), "eigvec": v, "var_pct": pct,
            "cum_pct": np.cumsum(pct)}


def exact(case, seed):
    kind, p = case["kind"], case["p"]
    step = max(1, (1 << 27) // p)
    if kind in ("text", "convert"):
        _, which, vals = _text(case, seed)
        ids = torch.arange(1, case["n"] + 1, device=DEV, dtype=torch.float64)
        x = torch.cat([ids[:, None], vals[which]], dim=1)
        if kind == "convert":
            return {"rows": None, "used": None, "out": x}
        data = [x]
    else:
        data = _inputs(case, seed)
    n = data[0].shape[0]
    if kind == "pairwise":
        x = data[0]
        have = ~torch.isnan(x)
        first = torch.stack([x[:, k][have[:, k]][0] for k in range(p)])
        d, v = torch.where(have, x - first, 0.0), have.double()
        N, S, C = v.T.contiguous() @ v, d.T.contiguous() @ v, d.T.contiguous() @ d
        Q = (d * d).T.contiguous() @ v
        cov = (C - S * S.T / N) / (N - 1)
        var = Q - S * S / N
        corr = (C - S * S.T / N) / torch.sqrt(var * var.T)
        corr.fill_diagonal_(1.0)
        mean = first + S.diagonal() / N.diagonal()
        return {"n": None, "mean": mean, "cov": cov, "corr": corr}
    if kind == "groups":
        off = _group_offsets(case, seed)
        keep = np.arange(1, p)
        mean, cov = np.zeros((len(off) - 1, p - 1)), np.zeros((len(off) - 1, p - 1, p - 1))
        for g in range(len(off) - 1):
            m, mu, M = _moments(lambda: iter([data[0][off[g]:off[g + 1]]]), p)
            mean[g], cov[g] = mu[keep], (M / (m - 1))[np.ix_(keep, keep)]
        return {"n": None, "mean": mean, "cov": cov}

    def blocks():
        for r in range(0, n, step):
            part = [x[r:r + step] if x.ndim == 2 else x[r:r + step, None] for x in data]
            yield torch.cat([x.double() for x in part], dim=1) if len(part) > 1 else part[0].double()

    drop = {"rows": 0, "planes": 0, "text": 0, "wide32": p - 1}.get(kind)
    keep = np.array([k for k in range(p) if k != drop])
    m, mean, M = _moments(blocks, p)
    return _finished(m, mean, M, keep)
