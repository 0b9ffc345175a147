"""The split-BF16 slices value by value. One target determinant in one state has
the transition densities 0, 1 and 2, which one slice holds, so the continuum
block differs from the FP64 one by exactly what the s slices of each integral
cut off: a column of the integral rows over the power of two at or above its
largest entry, truncated to 8 s bits. Column counts around 64, depths around the
64-deep tile, one to eight slices. Bound: the FP64 rounding of the sums over at
most 2 n_o^2 rows, 4 n_o^2 eps times the largest entry."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _cut(B, s):
    m = np.abs(B).max(axis=0)
    f, e = np.frexp(np.where(m > 0.0, m, 1.0))
    sg = np.ldexp(1.0, np.where(f == 0.5, e - 1, e))
    x, v = B / sg, np.zeros_like(B)
    for t in range(1, s + 1):
        a = np.trunc(x * 256.0)
        x = x * 256.0 - a
        v += a * 256.0 ** -t
    return v * sg


@pytest.mark.parametrize("n_o,n_c", [(2, 7), (5, 8), (6, 9), (8, 16), (9, 13), (12, 1)])
@pytest.mark.parametrize("slices", [1, 2, 3, 4, 5, 8])
def test_cut_integrals(n_o, n_c, slices):
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(n_o, 2, 1, n_c, [0], 1, 1, 2, 19, e_core=0.5)
    occ = synth.det_to_occ(inst.syms[0].dets[0])
    J, K = np.zeros((n_o, n_o)), np.zeros((n_o, n_o))
    for k in occ:
        J[k // 2, k // 2] += 1.0
        K[k // 2, k // 2] += k % 2 == 0
    A = np.concatenate([J.ravel(), K.ravel()])
    # rows (P Q | j j') and -(P j' | Q j)
    B = np.concatenate([inst.ttcc.reshape(n_o * n_o, -1),
                        -inst.tctc.transpose(0, 2, 3, 1).reshape(n_o * n_o, -1)])
    with cc.from_instance(inst) as ctx:
        ctx.build()
        H = ctx.get_matrix()
    with cc.from_instance(inst, precision=cc.CCH_PREC_SPLIT_BF16, split_slices=slices) as ctx:
        ctx.build()
        S = ctx.get_matrix()
    lost = (A @ (B - _cut(B, slices))).reshape(n_c, n_c)
    tol = 4 * n_o * n_o * np.finfo(np.float64).eps * np.abs(H).max()
    low = np.tril_indices(n_c)
    assert np.abs((H[:n_c, :n_c] - S[:n_c, :n_c] - lost)[low]).max() <= tol
    if slices == 1:
        assert np.abs(lost).max() > 1e6 * tol
    assert np.abs((H - S)[n_c:]).max() <= tol   # (class 4 and the L2 block are not sliced)
