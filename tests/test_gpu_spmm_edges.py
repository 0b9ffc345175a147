"""The sparse-L2 product at its edges: vector counts around the record lengths
(4, 8, 16 and 17), rows shorter and longer than a wave, continuum columns
around the strip and block sizes of the lower-triangle part (none, 1, 15, 16,
63, 65, 512, 513), against the host product of the read-out matrix."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
U = np.finfo(np.float64).eps / 2


@pytest.mark.parametrize("n_c,n_l2", [(0, 40), (1, 5), (15, 63), (16, 64), (63, 65), (65, 700), (512, 33), (513, 900),
                                      (30, 1)])
def test_sparse_product(n_c, n_l2):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(14, 6, 1, n_c, [0], 12, 1, n_l2, 10)
    D = inst.dim()
    rng = np.random.default_rng(D)
    with cc.from_instance(inst, sparse_l2=True) as ctx:
        ctx.build()
        H = ctx.get_matrix()
        for b in (1, 4, 5, 8, 9, 16, 17):
            V = rng.standard_normal((b, D))
            tol = 2 * D * U * (np.abs(V) @ np.abs(H)) + 1e-300
            W = ctx.apply(V)
            assert (np.abs(W - V @ H) <= tol).all(), b
            assert np.array_equal(W, ctx.apply(V))
