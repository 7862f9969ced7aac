"""Launch geometries of the smearing step, and block orders of the shift and the
hop, on lattices above the size where the step's split kernel ends (which takes
no geometry): t windows, LDS tiles, blocks with a group past the end and tiles
with blocks that have none give the same bits, for full and partial direction
masks; and the step on both sides of that size against the oracle and the
batched kernel, which never splits a link."""

import os
import re

import numpy as np
import pytest
import torch

import latgen
import oracle
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev, link_err, tol

pytestmark = pytest.mark.gpu

with open(os.path.join(os.path.dirname(q.__file__), "csrc", "ape.hip")) as fh:
    SPLIT = [int(n) for n in re.search(r"kSplitGroups64 = (\d+), kSplitGroups32 = (\d+);", fh.read()).groups()]

# groups: 400, four t ranges of one tile each, 16 blocks without a group; 324, two
# t ranges, 12 without; 400 and no whole groups in an xy plane; 403, no columns,
# the last ragged
ABOVE = [(20, 16, 5, 16), (16, 12, 9, 12), (20, 8, 10, 16), (13, 9, 11, 20)]
# (block, groups a wave, order, t window, LDS tile)
GEOMETRIES = [(256, 1, 1, 1, 0), (256, 1, 0, 2, 1), (512, 2, 1, 4, 0), (256, 4, 0, 8, 2), (256, 2, 2, 1, 0),
              (512, 1, 2, 1, 1), (512, 2, 2, 1, 2), (256, 1, 1, 16, 3), (512, 1, 2, 1, 3), (512, 2, 0, 2, 3),
              (256, 4, 1, 1, 3), (256, 1, 2, 1, 4), (512, 2, 1, 1, 4), (512, 1, 0, 8, 4), (512, 4, 1, 2, 4)]


def _groups(L):
    return (int(np.prod(L)) + 63) // 64


def _smear(c, L, Ud, prec, fmt, n, mask):
    out = torch.zeros_like(Ud)
    plaq = torch.zeros(3 * (n + 1), dtype=torch.float64, device=dev())
    q.qdpx_ape_smear(c, L, prec, fmt, Ud, out, 0.5, n, plaq, q.alloc_workspace(q.OP_APE, L, prec, fmt, n, dev()),
                     smear_mask=mask)
    return out, plaq


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", ABOVE, ids=lambda L: "x".join(map(str, L)))
def test_geometries_give_the_same_links(L, prec, fmt):
    assert _groups(L) > max(SPLIT)
    U = latgen.haar_links(L, 8000 + sum(L))
    c = q.Context(0)
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    for mask in (0xF, 0x7, 0x5):
        want = None
        for block, ns, xcd, tw, lds in GEOMETRIES:
            while L[3] % tw:
                tw //= 2
            q.qdpx_tune_set(c, q.OP_APE, L, prec, fmt, block, ns, xcd, tw, lds if prec == q.F32 else 0)
            out, plaq = _smear(c, L, Ud, prec, fmt, 2, mask)
            got = (out.view(torch.int64).clone(), plaq.clone())
            if want is None:
                want = got
                one, _ = _smear(c, L, Ud, prec, fmt, 1, mask)
                V = q.links_to_host(c, L, one, prec, fmt)
                torch.cuda.synchronize()
                assert link_err(V, oracle.ape_step(U, 0.5, mask)) < tol(prec), mask
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), (mask, block, ns, xcd, tw, lds)
    c.close()


# the last size that is split and the first that is not, whole and ragged
EDGES = [(8, 8, 16, 8), (13, 9, 10, 7), (4, 8, 6, 43), (8, 5, 5, 41), (16, 16, 10, 8), (11, 10, 6, 31), (4, 16, 3, 107),
         (10, 10, 5, 41)]


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
def test_split_edges(prec, fmt):
    assert sorted(_groups(L) for L in EDGES) == sorted(2 * [SPLIT[0], SPLIT[0] + 1, SPLIT[1], SPLIT[1] + 1])
    c = q.Context(0)
    Us = [latgen.haar_links(L, 8100 + i) for i, L in enumerate(EDGES)]
    Ud = [q.links_to_device(c, L, U, prec, fmt, dev()) for L, U in zip(EDGES, Us)]
    outs = [torch.zeros_like(u) for u in Ud]
    q.qdpx_ape_smear_batched(c, EDGES, prec, fmt, Ud, outs, 0.5, 1, None,
                             q.alloc_workspace(q.OP_BATCHED, EDGES, prec, fmt))
    for L, U, u, o in zip(EDGES, Us, Ud, outs):
        one, plaq = _smear(c, L, u, prec, fmt, 1, 0xF)
        V = q.links_to_host(c, L, one, prec, fmt)
        torch.cuda.synchronize()
        assert torch.equal(one.view(torch.int64), o.view(torch.int64)), L
        ref = oracle.ape_step(U, 0.5)
        assert link_err(V, ref) < tol(prec), L
        p = plaq.cpu().numpy().reshape(2, 3)
        assert np.abs(p[0] - oracle.plaquette(U)).max() < tol(prec)
        assert np.abs(p[1] - oracle.plaquette(ref)).max() < tol(prec)
    c.close()


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", ABOVE, ids=lambda L: "x".join(map(str, L)))
def test_given_orders_with_partial_masks(L, prec, fmt):
    """A geometry of qdpx_tune_set keeps its block order for every mask."""
    c = q.Context(0)
    Ud = q.links_to_device(c, L, latgen.haar_links(L, 8200), prec, fmt, dev())
    p, f = (q.fermion_to_device(c, L, latgen.dirac_field(L, 8201 + i), prec, dev()) for i in range(2))
    work = q.alloc_workspace(q.OP_SHIFT, L, prec, fmt, 1, dev())
    for mask in (0xF, 0x7, 0x8, 0x4, 0x0):
        want = None
        for ns, xcd, tw in ((1, 1, 1), (1, 0, 4), (2, 2, 1), (8, 2, 1), (1, 2, 1)):
            for op in (q.OP_SHIFT, q.OP_JACOBI):
                q.qdpx_tune_set(c, op, L, prec, fmt, 256, ns, xcd, tw)
            out = [torch.zeros_like(p) for _ in range(3)]
            n2 = torch.zeros(2, dtype=torch.float64, device=dev())
            for k, sign in enumerate((1, -1)):
                q.qdpx_eval_shift_mul_axpy(c, L, prec, fmt, Ud, p, f, 0.3, out[k], n2[k:], work, dir_mask=mask, sign=sign)
            q.qdpx_eval_hop(c, L, prec, fmt, Ud, p, out[2], dir_mask=mask)
            torch.cuda.synchronize()
            got = [t.view(torch.int64).clone() for t in (*out, n2)]
            want = want or got
            assert all(torch.equal(a, b) for a, b in zip(got, want)), (mask, ns, xcd, tw)
    c.close()
