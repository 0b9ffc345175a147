"""The reduction to tridiagonal form at the edges of its launch shapes: row
blocks of 128, columns from the 16-aligned one on, panels of 32, the switch of
the product from whole rows to tiles at 3072 trailing rows, odd sizes (vectors
at odd offsets), and the lane counts of the eigenvalue search (up to 1024, up
to 3072, above). Against LAPACK: residual, orthonormality and eigenvalues within
1e-12 of the spectral radius times n / 100 (the backward error of a Householder
reduction grows as n eps at worst)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(M, w, V):
    n = M.shape[0]
    wl = np.linalg.eigvalsh(M)
    scale = np.abs(wl).max()
    tol = 1e-12 * max(1.0, n / 100)
    assert np.all(np.diff(w) >= 0)
    assert np.abs(w - wl).max() <= tol * scale
    assert np.abs(V @ V.T - np.eye(n)).max() <= 10 * tol
    assert np.abs(M @ V.T - V.T * w[None, :]).max() <= tol * scale


@pytest.mark.parametrize("n", [15, 16, 17, 63, 65, 127, 128, 255, 256, 258, 1023, 1024, 1025, 3071, 3072, 3073, 3201])
def test_sizes_at_launch_edges(n):
    import paper_1709_03005_amd as cc
    rng = np.random.default_rng(n)
    M = rng.standard_normal((n, n))
    M = M + M.T
    print(f"[eig_all] edge n = {n}", flush=True)
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(M)
    _check(M, w, V)


@pytest.mark.parametrize("power", [-100, 0, 100, 150])
@pytest.mark.parametrize("n", [150, 3100])
def test_scaled_matrices(n, power):
    # entries far from 1 (their squares are in range), by whole rows and by
    # tiles: a power of two times the matrix multiplies the eigenvalues by it
    import paper_1709_03005_amd as cc
    rng = np.random.default_rng(3)
    B = rng.standard_normal((n, n))
    B = B + B.T
    f = 2.0 ** int(power * np.log2(10.0))
    with cc.Context(0) as ctx:
        w, V, _ = ctx.eig_all(B * f)
    _check(B, w / f, V)


def test_not_finite_is_refused():
    import paper_1709_03005_amd as cc
    n = 40
    with cc.Context(0) as ctx:
        for bad in (np.nan, np.inf):
            M = np.eye(n)
            M[5, 3] = M[3, 5] = bad
            with pytest.raises(cc.CchError):
                ctx.eig_all(M)
