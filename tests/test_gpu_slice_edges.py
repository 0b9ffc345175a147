"""The split-BF16 slices of the integral rows at the edges of their tiles: column
counts around 64 (with a remainder), depths below, at and above a tile of 64, one
to eight slices (the two LDS sizes), a column of zeros. The matrix of seven
slices or more against the FP64 one within 1e-12 of its largest entry, with fewer
within 4 K 2^-8s of it (each of the K terms of an entry is cut at 2^-8s), and
two builds bit for bit."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_o,n_c", [(2, 7), (5, 8), (6, 9), (8, 16), (9, 13)])
@pytest.mark.parametrize("slices", [1, 3, 4, 5, 8])
def test_slices(n_o, n_c, slices):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(n_o, 2, 1, n_c, [0], min(4, n_o), 2, 2, 3, e_core=0.5)
    # two orbitals without two-electron integrals: their columns are zero
    inst.ttcc[:, :, -1, :] = 0.0
    inst.ttcc[:, :, :, -1] = 0.0
    inst.tctc[:, -1, :, :] = 0.0
    inst.tctc[:, :, :, -1] = 0.0
    with cc.from_instance(inst) as ctx:
        ctx.build()
        H = ctx.get_matrix()
    with cc.from_instance(inst, precision=cc.CCH_PREC_SPLIT_BF16, split_slices=slices) as ctx:
        ctx.build()
        S = ctx.get_matrix()
        ctx.build()
        assert np.array_equal(ctx.get_matrix(), S)
    K = 2 * n_o * n_o
    bound = max(4.0 * K * 2.0 ** (-8 * slices), 1e-12)
    assert np.abs(S - H).max() <= bound * np.abs(H).max()
