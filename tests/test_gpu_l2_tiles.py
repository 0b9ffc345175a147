"""The L2 block at the edges of its tiles: 16-row tiles around 16 and 64
functions (every element against the oracle), and both tile heights around
the count where they change (2880 functions) against the sparse build, which
evaluates each pair on its own, bit for bit."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_l2", [1, 15, 16, 17, 63, 64, 65, 130])
@pytest.mark.parametrize("n_o", [8, 34])
def test_every_element(n_l2, n_o):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(n_o, 4, 1, 3, [0], 10, 2, n_l2, 9, e_core=0.25)
    H, A, K = oracle.Oracle(inst).build(with_abs=True)
    with cc.from_instance(inst) as ctx:
        ctx.build()
        G = ctx.get_matrix()
    ok, _ = oracle.tolerance_ok(G, H, A, K)
    assert ok.all()
    assert np.array_equal(G, G.T)


@pytest.mark.parametrize("n_l2", [2815, 2880, 2881, 3009])
def test_tile_heights_equal_the_sparse_build(n_l2):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(20, 6, 1, 5, [0], 12, 2, n_l2, 10)
    with cc.from_instance(inst) as ctx, cc.from_instance(inst, sparse_l2=True) as sp:
        ctx.build()
        sp.build()
        assert np.array_equal(ctx.get_matrix(), sp.get_matrix())
