"""More symmetry pairs than one launch's grid takes along z: 128 target symmetries
(8256 pairs), one of them with 256 states, which the densities take in eight
groups a pair. The matrix against the CPU oracle within its rounding bound."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def test_pairs_beyond_one_grid():
    import paper_1709_03005_amd as cc
    k = 127
    inst = synth.make_instance(8, 4, 1, 1, [0] * (k + 1), [260] + [2] * k, [256] + [1] * k, 20, 77)
    print(f"[symmetries] {k + 1} symmetries, {(k + 1) * (k + 2) // 2} pairs, D = {inst.dim()}", flush=True)
    H, A, K = oracle.Oracle(inst).build(with_abs=True)
    with cc.from_instance(inst) as ctx:
        ctx.build()
        G = ctx.get_matrix()
    ok, _ = oracle.tolerance_ok(G, H, A, K)
    assert ok.all()
