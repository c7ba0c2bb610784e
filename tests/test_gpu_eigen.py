"""Principal components of given correlation matrices (restored as checkpoints
with unit variances) against LAPACK: sizes at the edges of each solver's range,
separated, clustered, repeated and vanishing eigenvalues.

Tolerance: the solvers' backward error is a small multiple of q u ||A||
(u = 2^-53: q reflectors or rotations per entry, each within a few u); 20 q u
||A|| for eigenvalues and residuals, 20 q u for orthogonality."""
import struct

import numpy as np
import pytest

from helpers import current_stream, lib

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def finalize_of(A, **kw):
    """Finalize of a state with N = 2 and co-moments A (unit variances)."""
    L = lib()
    p = A.shape[0]
    T = p * (p + 1) // 2
    state = np.zeros(2 + 3 * p + 3 * T, dtype=np.uint64)
    state[0] = 2
    state[2 + 2 * p + 2 * T + p:] = np.ascontiguousarray(A[np.triu_indices(p)]).view(np.uint64)
    hdr = b"STSTATS1" + struct.pack("<q", p) + struct.pack("<ii", L.STATS_F64, 0) * p
    cfg = L.make_config([(L.STATS_F64, 0, 8 * c, 0) for c in range(p)], [8 * p], stream=current_stream())
    h = L.stats_deserialize(hdr + state.tobytes(), cfg)
    try:
        return L.stats_finalize(h, p, **kw)
    finally:
        L.stats_close(h)


def unit(A):
    d = 1.0 / np.sqrt(np.diag(A))
    A = A * np.outer(d, d)
    A = 0.5 * (A + A.T)
    np.fill_diagonal(A, 1.0)
    return A


def matrix(kind, q):
    rng = np.random.default_rng([q, len(kind)])
    if kind == "random":
        G = rng.standard_normal((q, 2 * q))
        return unit(G @ G.T)
    if kind == "identity":
        return np.eye(q)
    if kind == "rank1":  # +-1 everywhere
        s = np.where(rng.random(q) < 0.5, -1.0, 1.0)
        return np.outer(s, s)
    if kind == "equi":  # one eigenvalue of multiplicity q - 1
        return np.full((q, q), 0.25) + 0.75 * np.eye(q)
    if kind == "near":  # nearly collinear columns: eigenvalues down to 1e-12
        G = rng.standard_normal((q, 1)) + 1e-6 * rng.standard_normal((q, 2 * q))
        return unit(G @ G.T)
    if kind == "twins":  # every column twice: half of the eigenvalues vanish
        G = rng.standard_normal(((q + 1) // 2, 2 * q))
        B = unit(G @ G.T)
        i = np.arange(q) // 2
        return B[np.ix_(i, i)]
    if kind == "blocks":  # decoupled equal blocks
        i = np.arange(q) // 3
        return np.where(i[:, None] == i[None, :], 0.5, 0.0) + 0.5 * np.eye(q)
    raise ValueError(kind)


def check(A, fin):
    q = A.shape[0]
    lam, V = fin["eigval"], fin["eigvec"]
    assert np.array_equal(fin["corr"], A)
    ref = np.linalg.eigvalsh(A)[::-1]
    norm = max(1.0, ref[0])
    assert np.all(np.diff(lam) <= 0)
    assert np.max(np.abs(lam - ref)) <= 20 * q * U * norm
    assert np.max(np.abs(V @ V.T - np.eye(q))) <= 20 * q * U
    assert np.max(np.abs(A @ V.T - V.T * lam)) <= 20 * q * U * norm
    big = np.argmax(np.abs(V), axis=1)
    assert np.all(V[np.arange(q), big] > 0)


@pytest.mark.parametrize("kind", ["random", "identity", "rank1", "equi", "near", "twins", "blocks"])
@pytest.mark.parametrize("q", [1, 2, 3, 9, 15, 16, 17, 31, 32, 33, 59, 60])
def test_one_workgroup(kind, q):
    print(f"eigen {kind} q={q}", flush=True)
    A = matrix(kind, q)
    check(A, finalize_of(A))


@pytest.mark.parametrize("kind", ["random", "identity", "rank1", "equi", "near", "twins", "blocks"])
@pytest.mark.parametrize("q", [61, 64, 100, 128, 129, 192, 256, 257])
def test_whole_gpu(kind, q):
    print(f"eigen {kind} q={q}", flush=True)
    A = matrix(kind, q)
    check(A, finalize_of(A))


@pytest.mark.parametrize("q", [513, 1024])
def test_whole_gpu_largest(q):
    print(f"eigen random q={q}", flush=True)
    A = matrix("random", q)
    check(A, finalize_of(A))


@pytest.mark.parametrize("q", [5, 61, 130])
def test_covariance_stays_graded(q):
    # eigenvalues of a covariance matrix over 12 decades keep their relative
    # accuracy (the Jacobi method); a zero variance gives NaN eigenpairs
    s = 10.0 ** np.linspace(0, -6, q)
    A = matrix("random", q) * np.outer(s, s)
    A = 0.5 * (A + A.T)
    lam = finalize_of(A, pca_on=1)["eigval"]
    # bounds from the scaled matrix: lambda_k / s_k^2 within its extreme eigenvalues
    w = np.linalg.eigvalsh(unit(A))
    assert np.all(lam / (s * s) >= w[0] * (1 - 1e-9)) and np.all(lam / (s * s) <= w[-1] * (1 + 1e-9))
    A[1] = A[:, 1] = 0.0
    for on in (0, 1):
        fin = finalize_of(A, pca_on=on)
        assert np.all(np.isnan(fin["corr"][1])) and np.all(np.isnan(fin["eigval"])) == (on == 0)
