"""Accuracy of the p x p eigensolver in units of the last place."""
import numpy as np
import pytest

from oracle import gsi_oracle as O
from paper_2306_10379_amd import inputs

pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.mark.parametrize("p", [8, 16, 32, 48, 64, 80, 128])
def test_first_step_length(p):
    """The first step length follows from the eigenvalues of P^T P. It is well conditioned here (a
    relative error of the terms grows by 4 to 9), so eigenvalues good to an ulp or two put it within
    10 eps of the oracle's; norms that drift with the number of rotations do not."""
    from paper_2306_10379_amd import gsi
    A = inputs.spiked_sparse(1500, 6, p, seed=1)
    X0 = np.random.default_rng(1).standard_normal((1500, p))
    with gsi.Solver(A, X0, p, tol=0.0, max_iter=10) as s:
        s.step(1)
        mu = s.history()["mu"][0]
    ref = O.rcg(A, X0, tol=0.0, max_iter=1).mu[0]
    assert abs(mu - ref) <= 10 * EPS * ref


@pytest.mark.parametrize("p", [16, 31, 64, 80, 128])
def test_ritz_vectors_are_orthogonal(p):
    """Columns of the eigensolver are left as they are up to a cosine of eps; the cosine's own
    rounding, that of the product X U and of the start block add as much again each, and the
    largest of the p^2 entries is some standard deviations out: 6 eps."""
    from paper_2306_10379_amd import gsi
    A = inputs.spiked_sparse(1500, 6, p, seed=1)
    X0 = np.random.default_rng(1).standard_normal((1500, p))
    with gsi.Solver(A, X0, p, tol=0.0, max_iter=10) as s:
        s.step(1)
        s.residuals()
        U = s.get_x().cpu().numpy().astype(np.longdouble)
    off = U.T @ U
    np.fill_diagonal(off, 0.0)
    assert np.max(np.abs(off)) <= 6 * EPS


def _graded(n, p, sign=1.0):
    """Diagonal matrix whose first p entries fall over 12 decades, these entries in descending
    order, and their eigenvectors."""
    d = np.concatenate([sign * np.logspace(0, -12, p), -np.linspace(1.0, 0.5, n - p)])
    A = inputs.CSR(n=n, rowptr=np.arange(n + 1, dtype=np.int32), colind=np.arange(n, dtype=np.int32), vals=d)
    return A, np.sort(d[:p])[::-1], np.eye(n)[:, :p].copy()


@pytest.mark.parametrize("p", [3, 16, 20, 64, 100])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_small_ritz_values_beside_large_ones(p, sign):
    """The projected matrix of exact eigenvectors is diagonal: each Ritz value is right to the
    rounding of its own vector's normalization (8 eps), however small it is. sign = -1 makes the
    projected matrix negative."""
    from paper_2306_10379_amd import gsi
    A, w, X0 = _graded(300, p, sign)
    with gsi.Solver(A, X0, p) as s:
        ritz = s.residuals()[0]
    np.testing.assert_allclose(ritz, w, rtol=8 * EPS)


def test_small_ritz_values_of_a_batch():
    from paper_2306_10379_amd import gsi
    sizes = [(300, 3), (200, 16), (400, 20), (100, 32)]
    mats, ws, xs = zip(*[_graded(n, p) for n, p in sizes])
    b = gsi.BatchedSolver(list(mats), list(xs), [p for _, p in sizes], which=1, precision="fp64", max_iter=5)
    b.solve()
    for i in range(len(sizes)):
        np.testing.assert_allclose(b.results(i)[0], ws[i], rtol=8 * EPS)


@pytest.mark.parametrize("p", [2, 18])
@pytest.mark.parametrize("e1", [1e-4, 1e-5, 1e-6])
def test_long_step_keeps_the_block_orthonormal(p, e1):
    """A start column nearly orthogonal to the eigenvector it moves to takes a step with mu^2 b up to
    1e12, beside columns whose b are 1e-16 of the largest: each column is scaled by its own
    (1 + mu^2 b)^-1/2. Column norms and cosines carry the rounding of some products: 8 eps."""
    from paper_2306_10379_amd import gsi
    n = 80
    d = np.concatenate([[3.0], np.linspace(2.5, 1.5, p - 1), np.linspace(0.5, -1.0, n - p)])
    A = inputs.CSR(n=n, rowptr=np.arange(n + 1, dtype=np.int32), colind=np.arange(n, dtype=np.int32), vals=d)
    X0 = np.zeros((n, p))
    X0[p, 0], X0[0, 0] = 1.0, e1
    for j in range(1, p):
        X0[j, j], X0[p + 10 + j, j] = 1.0, 3e-8 * e1
    with gsi.Solver(A, X0, p, tol=0.0, max_iter=10) as s:
        s.step(1)
        X = s.get_x().cpu().numpy()
        mu = s.history()["mu"][0]
    assert mu * mu * (e1 * (d[0] - d[p])) ** 2 > 1e6, "no longer a long step"
    assert np.max(np.abs(X.T @ X - np.eye(p))) <= 8 * EPS
