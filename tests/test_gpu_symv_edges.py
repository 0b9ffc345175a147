"""The lower-triangle product at its edges: dimensions around the threshold
(2048), strip ends (512 columns), blocks of 16 and 32 rows and one last row or
column, group counts of one to four, device vectors with odd leading
dimensions (no 16-byte alignment), against the host product elementwise."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
U = np.finfo(np.float64).eps / 2


@pytest.mark.parametrize("D", [2047, 2048, 2049, 2063, 2079, 2080, 2081, 2559, 2560, 2561, 3073])
def test_product_at_tile_edges(D):
    import torch
    import paper_1709_03005_amd as cc
    inst = synth.make_instance(20, 6, 1, 5, [0], 12, 2, D - 10, 10)
    assert inst.dim() == D
    rng = np.random.default_rng(D)
    with cc.from_instance(inst) as ctx:
        ctx.build()
        H = ctx.get_matrix()
        for b in (1, 4, 5, 12, 13, 16):
            V = rng.standard_normal((b, D))
            ref = V @ H
            tol = 2 * D * U * (np.abs(V) @ np.abs(H)) + 1e-300
            ldv, ldw = D + 3, D + 1
            dV = torch.full((b * ldv + 1,), float("nan"), dtype=torch.float64, device="cuda")
            dW = torch.full((b * ldw + 1,), -7.0, dtype=torch.float64, device="cuda")
            dV[1:].view(b, ldv)[:, :D] = torch.from_numpy(V).cuda()
            torch.cuda.synchronize()
            ctx._ck(cc.lib.cch_apply(ctx.h, dV.data_ptr() + 8, ldv, b, dW.data_ptr() + 8, ldw, cc.CCH_MEM_DEVICE))
            W = dW[1:].view(b, ldw).cpu().numpy()
            assert (np.abs(W[:, :D] - ref) <= tol).all(), (D, b, np.abs(W[:, :D] - ref).max())
            assert (W[:, D:] == -7.0).all() and float(dW[0]) == -7.0
