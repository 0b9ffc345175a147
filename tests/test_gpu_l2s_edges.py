"""The sparse L2 block at the edges of its passes: function counts around the
eight rows of a wave, the 32 of a workgroup and the 64 columns of a step, rows
with more low-degree entries than one list of 64 holds (a full space of few
electrons in few orbitals, where a large share of a row is single
substitutions), one to three words. Bit for bit against the dense build, whose
values come from the same pairs."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_o,n_elec,n_l2", [(8, 2, 1), (8, 2, 7), (8, 2, 8), (8, 2, 9), (8, 2, 31), (8, 2, 33), (8, 2, 63),
                                             (8, 2, 64), (8, 2, 65), (8, 2, 127), (8, 2, 129), (12, 2, 790), (33, 2, 300),
                                             (66, 2, 200), (9, 6, 500)])
def test_equals_dense(n_o, n_elec, n_l2):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(n_o, n_elec, 1, 2, [0], 8, 2, n_l2, 21, e_core=0.5)
    with cc.from_instance(inst) as dense, cc.from_instance(inst, sparse_l2=True) as sp:
        dense.build()
        sp.build()
        G = dense.get_matrix()
        assert np.array_equal(sp.get_matrix(), G)
        assert np.array_equal(sp.get_diagonal(), dense.get_diagonal())
        x = np.random.default_rng(1).standard_normal((3, G.shape[0]))
        w = sp.apply(x)
    assert np.abs(w - x @ G).max() <= 1e-13 * np.abs(G).sum(1).max() * np.abs(x).max()
