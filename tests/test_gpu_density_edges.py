"""Target-space sums of a build at the edges of their launch shapes: batches of
64 pairs over the eight waves of a workgroup (determinant counts around 64 and
512, every determinant in the slots P = Q and in the rows of the aufbau one),
states around 16 and 32 of the bra and the ket (also more than 64), symmetries
with themselves and with each other, reduced precision's slot order. Every
element against the oracle with its own bounds."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


CASES = [
    (1, [0], 3, 1), (1, [0], 63, 5), (1, [0], 64, 16), (1, [0], 65, 17), (1, [0], 511, 2), (1, [0], 513, 33),
    (1, [0], 784, 32), (1, [0], 130, 66), (2, [0, 1], [300, 65], [15, 31]), (2, [0, 0, 1], [64, 129, 257], [1, 17, 33]),
]


@pytest.mark.parametrize("n_irrep,syms,n_det,n_states", CASES)
def test_every_element(n_irrep, syms, n_det, n_states):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(8, 4, n_irrep, 2, syms, n_det, n_states, 20, 7, e_core=0.5)
    H, A, K = oracle.Oracle(inst).build(with_abs=True)
    with cc.from_instance(inst) as ctx:
        ctx.build()
        G = ctx.get_matrix()
        ctx.build()
        assert np.array_equal(ctx.get_matrix(), G)   # sums in a fixed order
    ok, _ = oracle.tolerance_ok(G, H, A, K)
    assert ok.all()
    assert np.array_equal(G, G.T)
    with cc.from_instance(inst, plan=False) as ctx:
        ctx.plan(precision=cc.CCH_PREC_SPLIT_BF16, split_slices=4)
        ctx.build()
        S = ctx.get_matrix()
    # four 8-bit slices: 2^-24 of the row and column norms or better
    assert np.abs(S - H).max() <= 2.0 ** -20 * np.abs(H).max()
