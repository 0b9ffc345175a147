"""Class 4 (continuum x L2) at the edges of its split: states around the quads
and instances of the matrix-core product (and more than 64: two passes),
continuum orbitals around the tiles of 32, a workgroup's four tiles and 1 (no
pair of orbitals to load), odd counts (rows that begin 8 bytes off a 16-byte
boundary), functions one and four to a workgroup, several irreps, and L2
functions whose pairs and terms exceed one list (189 pairs, 441 terms). Every
element against the oracle with its own bounds."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def _check(inst):
    import paper_1709_03005_amd as cc
    H, A, K = oracle.Oracle(inst).build(with_abs=True)
    with cc.from_instance(inst) as ctx:
        ctx.build()
        G = ctx.get_matrix()
    ok, _ = oracle.tolerance_ok(G, H, A, K)
    assert ok.all()
    assert np.array_equal(G, G.T)


@pytest.mark.parametrize("n_states", [1, 4, 5, 8, 9, 13, 17, 24, 29, 37, 41, 53, 61, 65, 70])
@pytest.mark.parametrize("n_c", [1, 3])
def test_states(n_states, n_c):
    _check(synth.make_instance(8, 4, 1, n_c, [0], 100, n_states, 30, 11, e_core=0.5))


@pytest.mark.parametrize("n_c", [1, 2, 31, 32, 33, 65, 127, 129, 161])
def test_orbitals(n_c):
    _check(synth.make_instance(6, 4, 1, n_c, [0], 40, 3, 30, 12, e_core=0.5))


@pytest.mark.parametrize("n_irrep,n_c,syms,n_det,n_states", [(2, [5, 34], [0, 1], 60, 6), (4, [3, 1, 35, 2], [0, 1, 2, 3], 30, 2)])
def test_irreps(n_irrep, n_c, syms, n_det, n_states):
    _check(synth.make_instance(8, 4, n_irrep, n_c, syms, n_det, n_states, 40, 13, e_core=0.5))


def test_many_functions():
    # four L2 functions a workgroup, a remainder of one
    _check(synth.make_instance(14, 4, 1, 33, [0], 50, 2, 4097, 14, e_core=0.5))


def test_long_lists():
    _check(synth.make_instance(10, 16, 1, 3, [0], 2025, 3, 21, 15, e_core=0.5))
