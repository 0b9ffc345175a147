"""The Rayleigh-Ritz eigensolver at the edges of its thread layout: the rows
come in groups of 14 and the columns in groups of 32, with two column groups
held up to 64; and with what its search has to bracket again: pairs of close
eigenvalues, a matrix of exact direct sums (zero couplings), a graded one.
Against LAPACK with the bounds of tests/test_gpu_rr.py."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(G, fallback=0):
    import paper_1709_03005_amd as cc
    n = G.shape[0]
    with cc.Context() as ctx:
        th, Y, nf = ctx.subspace_eig(G)
    w = np.linalg.eigvalsh(G)
    nrm = np.abs(w).max()
    assert np.abs(th - w).max() <= 1e-13 * nrm
    assert np.abs(Y.T @ Y - np.eye(n)).max() <= 1e-13
    assert np.abs(G @ Y - Y * th[None, :]).max() <= 1e-13 * nrm
    assert fallback is None or nf == fallback


@pytest.mark.parametrize("n", [13, 14, 15, 27, 28, 29, 32, 33, 42, 43, 56, 57, 62, 66, 70, 71, 84, 85, 94])
def test_group_edges(n):
    M = np.random.default_rng(n).standard_normal((n, n))
    _run(M + M.T)


@pytest.mark.parametrize("n", [24, 64, 72, 96])
@pytest.mark.parametrize("gap", [1e-4, 1e-7, 1e-10])
def test_close_pairs(n, gap):
    rng = np.random.default_rng(n)
    Q, _ = np.linalg.qr(rng.standard_normal((n, n)))
    ev = np.repeat(np.sort(rng.uniform(-3, 3, n // 2)), 2) + gap * (np.arange(n) % 2)
    G = (Q * ev) @ Q.T
    _run(0.5 * (G + G.T), None)


@pytest.mark.parametrize("n", [30, 90])
def test_direct_sums_and_grading(n):
    rng = np.random.default_rng(n)
    G = np.zeros((n, n))
    for b in range(0, n, 6):
        B = rng.standard_normal((6, 6))
        G[b:b + 6, b:b + 6] = B + B.T
    _run(G, None)
    s = np.logspace(0, -12, n)
    M = rng.standard_normal((n, n))
    _run((M + M.T) * s[:, None] * s[None, :], None)
