"""The tables of a build's launches are part of the plan's memory: budgets from the
whole of it down, a few bytes at a time, where the table of the expansion
products goes first (a launch each then), then the single pass. Every plan
stays within its budget and gives the same bits; the bytes of many symmetry
pairs hold their tables."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_budgets_around_the_tables():
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(9, 4, 4, 11, [0, 1, 2, 3], 14, 3, 30, 41)
    with cc.from_instance(inst) as ref:
        ref.build()
        G = ref.get_matrix()
        whole = ref.plan_info()[0]
        rows = int(ref.work_counts()["relayout_bytes"] / 2)   # bytes of the integral rows
    seen = set()
    for less in (0, 1, 8, 300, 900, 1500, 2100, 3000, 6000, rows // 2, rows - rows // 24):
        with cc.from_instance(inst, plan=False) as ctx:
            ctx.plan(max_device_bytes=whole - less)
            got, passes = ctx.plan_info()
            assert got <= whole - less
            seen.add((got < whole, passes > 1))
            ctx.build()
            assert np.array_equal(ctx.get_matrix(), G)
    assert {(False, False), (True, False), (True, True)} <= seen


def test_pairs_pay_for_their_tables():
    # two counts of symmetries alike but for the pairs: each pair adds its lists (of
    # known sizes, one determinant and one state a symmetry) and its table entries
    import paper_1709_03005_amd as cc
    n_o, k = 2, (10, 30)
    got = []
    for n in k:
        inst = synth.make_instance(n_o, 2, 1, 1, [0] * n, [1] * n, [1] * n, 0, 3)
        with cc.from_instance(inst, precision=cc.CCH_PREC_FP32) as ctx:
            got.append(ctx.plan_info()[0])
    pairs = [n * (n + 1) // 2 for n in k]
    per_pair = (got[1] - got[0]) / (pairs[1] - pairs[0])
    slots, pr = n_o * n_o, 1   # (every label; one connected determinant pair at most)
    lists = (8 + 8 + 8) + pr * (4 + 4 + 1 + 1 + 8) + slots * 8 + n_o * n_o * 4 + 8 + pr * (8 + 4 + 8 + 8) + 8 * 4
    lists += 2 * slots * 8 + 3 * (slots + 1) * 8 + 8 + 2 * slots * (8 + 4 + 4) + 4
    print(f"[tables] {per_pair:.1f} bytes a pair, lists {lists}", flush=True)
    assert per_pair >= lists + 300
