"""Two-continuum integrals given without the symmetries of real orbitals: the FP64
build then reads every value as given, (PQ|jj') for the label PQ and -(Pj'|jQ),
as the eight-slice split-BF16 build does (within 1e-12 of the largest entry), in
one pass and in several. A single pair of values that differ, in any of the
symmetries, at the corners of the blocks and beside the edges of the 32-wide
tiles, is found; values that agree to a few rounding errors are taken as equal
(the folded product's smaller operation count)."""
import copy

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _instance(n_irrep, n_c=35):
    return synth.make_instance(8, 4, n_irrep, n_c, list(range(n_irrep)), 12, 3, 10, 21)


def _flops(inst, **plan):
    import paper_1709_03005_amd as cc
    with cc.from_instance(inst, **plan) as ctx:
        return ctx.work_counts()["gemm_flops"]


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("n_irrep", [1, 2, 4])
def test_every_value_is_read(n_irrep, packed):
    import paper_1709_03005_amd as cc
    inst = copy.deepcopy(_instance(n_irrep))
    rng = np.random.default_rng(5)
    inst.ttcc = inst.ttcc * rng.uniform(0.5, 1.5, inst.ttcc.shape)
    inst.tctc = inst.tctc * rng.uniform(0.5, 1.5, inst.tctc.shape)
    if packed:
        inst = synth.pack_integrals(inst)
    with cc.from_instance(inst, precision=cc.CCH_PREC_SPLIT_BF16, split_slices=8) as ctx:
        ctx.build()
        S = ctx.get_matrix()
        plain = ctx.work_counts()["gemm_flops"]
    with cc.from_instance(inst) as ctx:
        ctx.build()
        H = ctx.get_matrix()
        size = ctx.plan_info()[0]
        rows = ctx.work_counts()["relayout_bytes"] / 2
        assert ctx.work_counts()["gemm_flops"] == plain
    assert np.abs(H - S).max() <= 1e-12 * np.abs(H).max()
    with cc.from_instance(inst, plan=False) as ctx:
        ctx.plan(max_device_bytes=int(size - rows + rows // (4 * n_irrep * n_irrep)))
        assert ctx.plan_info()[1] > 1
        ctx.build()
        assert np.array_equal(ctx.get_matrix(), H)


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("P,Q", [(0, 0), (6, 6), (6, 2), (0, 4)])
@pytest.mark.parametrize("j,k", [(0, 1), (31, 32), (32, 31), (34, 0), (3, 34), (33, 34)])
@pytest.mark.parametrize("which", ["ttcc", "tctc"])
def test_one_value_off_is_found(which, j, k, P, Q, packed):
    import paper_1709_03005_amd as cc
    inst = _instance(2)
    plain = _flops(inst, precision=cc.CCH_PREC_FP32)
    first = int(inst.n_c[0])   # j and k in the second irrep's range, P and Q of one irrep
    for err, found in ((1e-12, True), (2.0 ** -52, False)):
        y = copy.deepcopy(inst)
        v = y.ttcc if which == "ttcc" else y.tctc.transpose(0, 2, 1, 3)
        assert y.n_c[1] == 35 and v[P, Q, first + j, first + k] != 0.0
        v[P, Q, first + j, first + k] *= 1.0 + err
        if packed:
            y = synth.pack_integrals(y)
        assert (_flops(y) == plain) == found, err


def test_batch_of_both_layouts():
    import paper_1709_03005_amd as cc
    a, b = copy.deepcopy(_instance(2)), _instance(4, 20)
    a.ttcc = a.ttcc * np.random.default_rng(3).uniform(0.5, 1.5, a.ttcc.shape)
    single = []
    for inst in (a, b):
        with cc.from_instance(inst) as ctx:
            ctx.build()
            single.append(ctx.get_matrix())
    with cc.from_instance(a) as x, cc.from_instance(b) as y:
        batch = cc.Batch([x, y])
        for _ in range(2):
            batch.build()
            x.sync()
            assert np.array_equal(x.get_matrix(), single[0])
            assert np.array_equal(y.get_matrix(), single[1])
        batch.close()
