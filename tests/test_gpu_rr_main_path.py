"""The Rayleigh-Ritz kernel's main path, with no Jacobi fallback, on what its search
has to bracket again: pairs of eigenvalues 1e-4 to 1e-10 apart (far above the
rounding of the norm, so the twisted vectors stay independent), direct sums
(couplings that vanish), a diagonal matrix with a border of a few rows, as a
restarted solve has, and a matrix with one eigenvalue far from the rest. Bounds
of tests/test_gpu_rr.py: 1e-13 times the norm."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(G):
    import paper_1709_03005_amd as cc
    n = G.shape[0]
    with cc.Context() as ctx:
        th, Y, nf = ctx.subspace_eig(G)
    w = np.linalg.eigvalsh(G)
    nrm = np.abs(w).max()
    assert np.abs(th - w).max() <= 1e-13 * nrm
    assert np.abs(Y.T @ Y - np.eye(n)).max() <= 1e-13
    assert np.abs(G @ Y - Y * th[None, :]).max() <= 1e-13 * nrm
    assert nf == 0


@pytest.mark.parametrize("n", [24, 64, 72, 96])
@pytest.mark.parametrize("gap", [1e-4, 1e-7, 1e-10])
def test_close_pairs(n, gap):
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    ev = np.repeat(np.sort(rng.uniform(-3, 3, n // 2)), 2) + gap * (np.arange(n) % 2)
    G = (Q * ev) @ Q.T
    _run(0.5 * (G + G.T))


@pytest.mark.parametrize("n", [30, 90])
def test_direct_sums(n):
    rng = np.random.default_rng(n)
    G = np.zeros((n, n))
    for b in range(0, n, 6):
        B = rng.standard_normal((6, 6))
        G[b:b + 6, b:b + 6] = B + B.T
    _run(G)


@pytest.mark.parametrize("n,border", [(20, 5), (64, 10), (80, 10), (96, 16)])
@pytest.mark.parametrize("size", [1.0, 1e-3, 1e-8])
def test_diagonal_with_border(n, border, size):
    rng = np.random.default_rng(n)
    G = np.diag(np.sort(rng.uniform(-10, 30, n)))
    B = rng.standard_normal((border, n))
    G[n - border:, :] += size * B
    G[:, n - border:] += size * B.T
    _run(G)


@pytest.mark.parametrize("n", [16, 65, 96])
def test_one_far(n):
    M = np.random.default_rng(n).standard_normal((n, n))
    G = M + M.T
    G[n // 2, n // 2] = 1e6
    _run(G)
