"""Weakly coupled rows in the eigensolvers: one row and column of a matrix times
s, from far above to far below the size whose square leaves the range of a
double (1e-154 of the largest entry), where a reflector formed from squares
that have lost their bits is not orthogonal. The whole spectrum by whole rows
and by tiles, of matrices near 1 and far from it, and the Rayleigh-Ritz kernel.
Bounds: the backward error of a Householder reduction, n eps times the norm at
worst, as 1e-12 max(1, n / 100) (the whole spectrum) and 1e-13 (Rayleigh-Ritz,
n <= 96), for the residual, the eigenvalues and the orthonormality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _weak(n, row, s, seed):
    M = np.random.default_rng(seed).standard_normal((n, n))
    M = M + M.T
    d = M[row, row]
    M[row, :] *= s
    M[:, row] *= s
    M[row, row] = d
    return M


def _check(M, w, V, tol):
    wl = np.linalg.eigvalsh(M)
    scale = np.abs(wl).max()
    assert np.abs(w - wl).max() <= tol * scale
    assert np.abs(V @ V.T - np.eye(M.shape[0])).max() <= 10 * tol
    assert np.abs(M @ V.T - V.T * w[None, :]).max() <= tol * scale


@pytest.mark.parametrize("s", [1e-120, 1e-150, 1e-154, 1e-156, 1e-158, 1e-159, 1e-160, 1e-161, 1e-162, 1e-200, 1e-240,
                               1e-300])
@pytest.mark.parametrize("n,row", [(2, 0), (3, 0), (8, 0), (8, 3), (150, 0), (150, 148)])
def test_whole_spectrum(n, row, s):
    import paper_1709_03005_amd as cc
    M = _weak(n, row, s, n + row)
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(M)
    _check(M, w, V, 1e-12 * max(1.0, n / 100))


@pytest.mark.parametrize("power,s", [(-300, 1e-40), (-200, 1e-120), (-97, 1e-150), (-96, 1e-160), (96, 1e-160),
                                     (97, 1e-230), (300, 1e-160), (1000, 1e-160), (-1000, 1e-161)])
@pytest.mark.parametrize("n", [40, 150])
def test_whole_spectrum_scaled(n, power, s):
    # 2^power times a matrix has 2^power times its eigenvalues and the same vectors
    import paper_1709_03005_amd as cc
    M = np.ldexp(_weak(n, 0, s, n), power)
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(M)
    _check(np.ldexp(M, -power), np.ldexp(w, -power), V, 1e-12 * max(1.0, n / 100))


@pytest.mark.parametrize("s", [1e-154, 1e-158, 1e-160, 1e-161])
def test_whole_spectrum_by_tiles(s):
    import paper_1709_03005_amd as cc
    n = 3100
    M = _weak(n, 0, s, 5)
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(M)
    _check(M, w, V, 1e-12 * n / 100)


@pytest.mark.parametrize("s", [1e-150, 1e-156, 1e-158, 1e-160, 1e-161, 1e-162, 1e-200])
@pytest.mark.parametrize("n,row", [(8, 0), (40, 5), (80, 0), (96, 50)])
def test_rayleigh_ritz(n, row, s):
    import paper_1709_03005_amd as cc
    M = _weak(n, row, s, n + row)
    with cc.Context(0) as ctx:
        th, Y, nf = ctx.subspace_eig(M)
    _check(M, th, Y.T, 1e-13)
    assert nf == 0


@pytest.mark.parametrize("n", [33, 64, 150])
def test_graded_over_150_decades(n):
    # every column is weaker than the one before it, down through the window
    import paper_1709_03005_amd as cc
    s = np.logspace(0, -150, n)
    M = np.random.default_rng(n).standard_normal((n, n))
    M = (M + M.T) * s[:, None] * s[None, :]
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(M)
    _check(M, w, V, 1e-12 * max(1.0, n / 100))
