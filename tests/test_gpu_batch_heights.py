"""A batch whose products take tiles of every height in one launch (1, 15, 16,
17, 28, 45, 66 and 136 rows, squares and rectangles, several symmetries): each
instance bit for bit as its own build."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("autotune", [False, True])
def test_heights(autotune):
    import paper_1709_03005_amd as cc
    insts = [synth.make_instance(8, 4, 1, 9 + i, [0], 30, s, 20 + i, 31 + i, e_core=0.5, packed=True)
             for i, s in enumerate([1, 5, 16, 7, 9, 11])]
    insts.append(synth.make_instance(8, 4, 2, [7, 12], [0, 1], 20, [5, 4], 25, 41, e_core=0.5, packed=True))
    insts.append(synth.make_instance(8, 4, 2, [5, 9], [0, 0, 1], 20, [3, 17, 2], 25, 42, e_core=0.5, packed=True))
    ctxs = [cc.from_instance(i) for i in insts]
    b = cc.Batch(ctxs, autotune=autotune)
    b.build()
    got = [c.get_matrix() for c in ctxs]
    b.close()
    for i, g in zip(insts, got):
        with cc.from_instance(i) as c:
            c.build()
            assert np.array_equal(c.get_matrix(), g)
