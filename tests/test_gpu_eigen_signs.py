"""Sign of eigenvectors whose largest entries tie: the entry of lowest index is
positive and tied entries are equal, at every size (one rotation, QL, the
whole-GPU solver and both Jacobi forms, and the sizes around their limits)."""
import numpy as np
import pytest

from test_gpu_eigen import U, finalize_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [s * v for s in (1, -1) for v in (0.7313, 0.5, 0.1, 3e-3, 1e-4, 1e-8, 2e-12, 1 - 1e-9)])
@pytest.mark.parametrize("pca_on", [0, 1])
def test_two_columns(r, pca_on):
    # (1, 1) and (1, -1) over sqrt 2 whatever the correlation
    fin = finalize_of(np.array([[1.0, r], [r, 1.0]]), pca_on=pca_on)
    plus, minus = [1.0, 1.0], [1.0, -1.0]
    want = np.sqrt(0.5) * np.array([plus, minus] if r > 0 else [minus, plus])
    assert np.array_equal(fin["eigval"], [1 + abs(r), 1 - abs(r)])
    assert np.max(np.abs(fin["eigvec"] - want)) <= 4 * U  # a root, a quotient and a product
    assert np.all(np.abs(fin["eigvec"]) == np.abs(fin["eigvec"][0, 0]))


@pytest.mark.parametrize("kind", ["rank1", "equi"])
@pytest.mark.parametrize("pca_on", [0, 1])
@pytest.mark.parametrize("q", [3, 4, 9, 16, 17, 24, 25, 31, 60, 61, 100])
def test_collinear_and_equicorrelated(kind, pca_on, q):
    # columns equal or equicorrelated up to their signs s: the first component is s / sqrt q
    for seed in range(4):
        s = np.where(np.random.default_rng([q, seed]).random(q) < 0.5, -1.0, 1.0)
        A = np.outer(s, s) if kind == "rank1" else 0.5 * np.outer(s, s) + 0.5 * np.eye(q)
        v = finalize_of(A, pca_on=pca_on)["eigvec"][0]
        # backward error 20 q u ||A|| over a gap of at least ||A|| (2 - 1/q) / 3
        assert np.max(np.abs(v - s[0] * s / np.sqrt(q))) <= 60 * q * U
        assert np.all(np.abs(v) == v[0])
