"""Orthonormalisation of the Davidson blocks at the widths where its kernel
changes (8, 16 and 32 columns): first blocks of 2k = 2 to 32 columns, in a
space hardly wider than the block, where directions drop out, and in a wide
one. Eigenvalues against the host's (a residual below tol puts each within tol
of one), vectors against orthonormality and their own residuals."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
TOL = 1e-8


@pytest.mark.parametrize("D", [35, 700])
@pytest.mark.parametrize("k", [1, 3, 4, 5, 8, 9, 15, 16])
def test_pairs_at_block_widths(k, D):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(20, 6, 1, 5, [0], 12, 2, D - 10, 10)
    assert inst.dim() == D
    with cc.from_instance(inst) as ctx:
        ctx.build()
        H = ctx.get_matrix()
        ev, vec, info, rc = ctx.davidson(k, tol=TOL)
    assert rc == cc.CCH_OK
    w = np.linalg.eigvalsh(H)
    assert np.abs(ev - w[:k]).max() < 2 * TOL
    assert np.linalg.norm(H @ vec.T - vec.T * ev[None, :], axis=0).max() < 2 * TOL
    assert np.abs(vec @ vec.T - np.eye(k)).max() < 1e-10
