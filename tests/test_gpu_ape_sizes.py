"""The smearing step on both sides of the size where three waves share a
link's staples (128 groups of 64 sites in FP64, 384 in FP32): against the
oracle, with partial masks and the plaquettes, and every launch geometry with
the same bits above it; below it the persistent batched kernel, which never
splits a link, gives the bits to match."""

import numpy as np
import pytest
import torch

import latgen
import oracle
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev, link_err, tol

pytestmark = pytest.mark.gpu

# groups: 1, 5 (ragged), 128, 130, 384, 408, 403 (ragged)
LATTICES = [(4, 4, 2, 2), (3, 5, 4, 5), (8, 8, 16, 8), (8, 8, 13, 10), (16, 16, 12, 8), (16, 16, 6, 17), (13, 9, 11, 20)]


def _smear(c, L, Ud, prec, fmt, n, mask, with_plaq=True):
    out = torch.zeros_like(Ud)
    plaq = torch.zeros(3 * (n + 1), dtype=torch.float64, device=dev()) if with_plaq else None
    q.qdpx_ape_smear(c, L, prec, fmt, Ud, out, 0.5, n, plaq, q.alloc_workspace(q.OP_APE, L, prec, fmt, n, dev()),
                     smear_mask=mask)
    return out, plaq


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", LATTICES, ids=lambda L: "x".join(map(str, L)))
def test_step_sizes_against_oracle(L, prec, fmt):
    U = latgen.haar_links(L, 7500 + sum(L))
    c = q.Context(0)
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    for mask in (0xF, 0x7, 0xA, 0x1):
        out, plaq = _smear(c, L, Ud, prec, fmt, 1, mask)
        V = q.links_to_host(c, L, out, prec, fmt)
        torch.cuda.synchronize()
        ref = oracle.ape_step(U, 0.5, mask)
        assert link_err(V, ref) < tol(prec), mask
        p = plaq.cpu().numpy().reshape(2, 3)
        assert np.abs(p[0] - oracle.plaquette(U)).max() < tol(prec)
        assert np.abs(p[1] - oracle.plaquette(ref)).max() < tol(prec)
        # the links do not depend on whether the plaquettes are taken
        assert torch.equal(out.view(torch.int64), _smear(c, L, Ud, prec, fmt, 1, mask, False)[0].view(torch.int64))
    c.close()


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
def test_split_links_equal_the_batched_kernels(prec, fmt):
    Ls = [(4, 4, 2, 2), (3, 5, 4, 5), (8, 8, 8, 8), (8, 8, 16, 8), (16, 16, 12, 8), (13, 9, 11, 20)]
    c = q.Context(0)
    Us = [q.links_to_device(c, L, latgen.haar_links(L, 7600 + i), prec, fmt, dev()) for i, L in enumerate(Ls)]
    outs = [torch.zeros_like(u) for u in Us]
    q.qdpx_ape_smear_batched(c, Ls, prec, fmt, Us, outs, 0.5, 3, None, q.alloc_workspace(q.OP_BATCHED, Ls, prec, fmt))
    for L, u, o in zip(Ls, Us, outs):
        one, _ = _smear(c, L, u, prec, fmt, 3, 0xF, False)
        torch.cuda.synchronize()
        assert torch.equal(one.view(torch.int64), o.view(torch.int64)), L
    c.close()


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", [(16, 16, 6, 17), (13, 9, 11, 20)], ids=lambda L: "x".join(map(str, L)))
@pytest.mark.parametrize("mask", [0xF, 0x7])
def test_geometries_above_the_split_give_the_same_bits(L, prec, fmt, mask):
    U = latgen.haar_links(L, 7700)
    c = q.Context(0)
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    want = None
    for block, ns, xcd in ((256, 1, 1), (512, 1, 0), (256, 2, 2), (512, 4, 2)):
        for lds in range(5) if prec == q.F32 else (0,):
            q.qdpx_tune_set(c, q.OP_APE, L, prec, fmt, block, ns, xcd, 1, lds)
            out, plaq = _smear(c, L, Ud, prec, fmt, 2, mask)
            got = (out.view(torch.int64).clone(), plaq.clone())
            want = want or got
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (block, ns, xcd, lds)
    c.close()
