"""A vector that is not finite in one L2 component: the sparse-L2 product is not
finite only in the rows that hold a non-zero in that column (and in the
continuum rows, which are dense); every other row has the bits of the product
with that component zero. The first component of the L2 block, one in the
middle and the last, at each record length."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_c", [0, 9])
@pytest.mark.parametrize("at", ["first", "middle", "last"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_reaches_connected_rows_only(n_c, at, bad):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(14, 6, 1, n_c, [0], 12, 1, 700, 10)
    inst.l2_dets = inst.l2_dets[::-1].copy()   # (the reference, connected to every double, goes last)
    D = inst.dim()
    Dc = D - 700
    with cc.from_instance(inst, sparse_l2=True) as ctx:
        ctx.build()
        H = ctx.get_matrix()
        for b in (1, 4, 7, 16):
            V = np.random.default_rng(b).standard_normal((b, D))
            c = {"first": Dc, "middle": Dc + 350, "last": D - 1}[at]
            V[:, c] = 0.0
            W0 = ctx.apply(V)
            V[b - 1, c] = bad
            W = ctx.apply(V)
            assert np.array_equal(W[:b - 1], W0[:b - 1])
            free = np.flatnonzero(H[Dc:, c] == 0.0) + Dc
            assert free.size < 700 and (free.size > 0 or at == "last")
            assert np.array_equal(W[b - 1, free], W0[b - 1, free])
            assert not np.isfinite(W[b - 1, np.flatnonzero(H[Dc:, c]) + Dc]).any()
