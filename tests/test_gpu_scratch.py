"""The work space a context keeps between calls: results of calls that reuse
blocks other calls have written equal those of a fresh context bit for bit,
and the memory comes back at the end (at once under a memory budget)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _calls(ctx, V, A):
    """One pass over the calls that take work space, small and large ones in turn."""
    out = [ctx.apply(V[:1])]
    w, Z, _ = ctx.eig_all(A)
    out += [w, Z, ctx.apply(V)]
    ev, vec, _, _ = ctx.davidson(5, tol=1e-9)
    out += [ev, vec, *ctx.subspace_eig(A[:40, :40])[:2]]
    w, Z, _ = ctx.eig_all(A[:70, :70])
    return out + [w, Z]


@pytest.mark.parametrize("name,budget", [("tiny", 0), ("small", 0), ("small", 1 << 34)])
def test_reused_work_space_gives_the_same_bits(name, budget):
    import torch
    import paper_1709_03005_amd as cc
    inst = synth.CONFIGS[name]()
    rng = np.random.default_rng(3)
    V = rng.standard_normal((20, inst.dim()))
    A = rng.standard_normal((333, 333))
    A = A + A.T
    torch.cuda.synchronize()
    with cc.from_instance(inst, plan=False) as ctx:
        ctx.plan(max_device_bytes=budget)
        ctx.build()
        free0 = torch.cuda.mem_get_info()[0]
        first = _calls(ctx, V, A)
        second = _calls(ctx, V, A)
        third = _calls(ctx, V, A)
        kept = free0 - torch.cuda.mem_get_info()[0]
    for a, b, c in zip(first, second, third):
        assert np.array_equal(a, b) and np.array_equal(a, c)
    # idle blocks: none under a budget, a bounded amount without (1/64 of the device)
    assert kept <= (16 << 20 if budget else torch.cuda.mem_get_info()[1] // 64)
    assert np.allclose(first[3], V @ oracle_matrix(inst), rtol=0, atol=1e-9)


def oracle_matrix(inst):
    import oracle
    return oracle.Oracle(inst).build()
