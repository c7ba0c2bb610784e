"""Eigenpairs of correlation matrices near the identity, in one workgroup: with
F = A - I (exact: the diagonal is 1) every error is a small multiple of q u ||F||
(u = 2^-53), over the gap for an eigenvector, however weak the correlations; 20 q u
||F|| as for the residuals of any matrix, plus the roundings of the results."""
import numpy as np
import pytest

import oracle
from test_gpu_eigen import U, finalize_of, matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1.0, 1e-2, 1e-4, 1e-6])
@pytest.mark.parametrize("q", [3, 5, 9, 16, 17, 24])
def test_near_identity(q, scale):
    A = matrix("random", q) * scale
    np.fill_diagonal(A, 1.0)
    fin = finalize_of(A)
    lam, V = oracle.eig_sym(A)  # 50 digits, rounded
    norm = float(np.max(np.abs(lam - 1.0)))
    assert np.max(np.abs(fin["eigval"] - lam)) <= 20 * q * U * norm + 2 * U * lam[0]
    for k in range(q):
        gap = min(abs(lam[k] - lam[j]) for j in range(q) if j != k)
        v = fin["eigvec"][k]
        err = min(np.max(np.abs(v - V[k])), np.max(np.abs(v + V[k])))
        assert err <= 20 * q * U * norm / gap + 64 * U, k
