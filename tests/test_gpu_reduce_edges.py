"""The reductions where they change from one launch to two (two chunks of
4096 partials) and at chunk ends: sums of whole numbers, exact in any order."""

import numpy as np
import pytest
import torch

import paper_1105_2279_amd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zt", [(2, 2), (63, 65), (64, 64), (17, 241), (64, 128), (3, 2731)])
@pytest.mark.parametrize("prec", [q.F64, q.F32])
def test_norm_of_whole_numbers(zt, prec):
    L = (8, 8) + zt  # as many 64-site groups (partials) as z times t
    V = int(np.prod(L))
    ctx = q.Context(0)
    aos = torch.from_numpy(np.random.default_rng(V).integers(-3, 4, (V, 12, 2)).astype(np.float64)).cuda()
    phi, U = q.alloc_fermion(L, prec), torch.zeros(q.qdpx_links_bytes(L, prec, q.LINK18), dtype=torch.uint8, device="cuda")
    q.qdpx_pack_fermion(ctx, L, aos, prec, phi)
    chi, norm = torch.zeros_like(phi), torch.zeros(1, dtype=torch.float64, device="cuda")
    q.qdpx_eval_shift_mul_axpy(ctx, L, prec, q.LINK18, U, phi, phi, 1.0, chi, norm,
                               q.alloc_workspace(q.OP_SHIFT, L, prec, q.LINK18), dir_mask=0)
    assert norm.item() == aos.square().sum().item()


@pytest.mark.parametrize("zt", [(2, 2), (35, 39), (2, 683)])
def test_plaquette_of_unit_links(zt):
    L = (8, 8) + zt  # three partials per group and component
    ctx = q.Context(0)
    aos = torch.zeros((int(np.prod(L)), 4, 3, 3, 2), dtype=torch.float64, device="cuda")
    for a in range(3):
        aos[:, :, a, a, 0] = 1.0
    U, plaq = q.alloc_links(L, q.F64, q.LINK18), torch.zeros(3, dtype=torch.float64, device="cuda")
    q.qdpx_pack_links(ctx, L, aos, q.F64, q.LINK18, U)
    q.qdpx_plaquette(ctx, L, q.F64, q.LINK18, U, plaq, q.alloc_workspace(q.OP_PLAQ, L, q.F64, q.LINK18))
    assert plaq.tolist() == [1.0, 1.0, 1.0]
