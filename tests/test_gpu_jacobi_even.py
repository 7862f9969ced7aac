"""Jacobi smearing with an even number of iterations: the first hop reads the
caller's field itself and keeps the copy the later ones add.  The workspace
starts as NaN, so that a component that copy misses shows, on lattices of
linear, ragged and plane-filling extents, for full, sparse and spatial masks,
against the oracle."""

import pytest
import torch

import latgen
import oracle
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, ctx, dev, need_gpu, rel_err, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", [(3, 5, 4, 7), (8, 8, 4, 4), (2, 2, 3, 5)], ids=lambda L: "x".join(map(str, L)))
@pytest.mark.parametrize("n,mask", [(2, 0xF), (4, 0x5), (6, 0x7)])
def test_even_iterations_match_oracle(L, prec, fmt, n, mask):
    need_gpu()
    U, chi = latgen.haar_links(L, 5100 + sum(L)), latgen.dirac_field(L, 5200 + sum(L))
    c = ctx()
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    cd = q.fermion_to_device(c, L, chi, prec, dev())
    work = q.alloc_workspace(q.OP_JACOBI, L, prec, fmt, n, dev())
    work.view(dtype=torch.uint8).fill_(0xFF)
    q.qdpx_jacobi_smear(c, L, prec, fmt, Ud, cd, 0.21, n, 1.5, mask, work)
    got = q.fermion_to_host(c, L, cd, prec)
    nrm, mx = rel_err(got, oracle.jacobi_smear(U, chi, 0.21, n, 1.5, mask))
    assert nrm < n * tol(prec) and mx < n * tol(prec), (nrm, mx)  # one tolerance per iteration
