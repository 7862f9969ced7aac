"""Every operation in the slab-walk order against the contiguous one, bit for
bit, on lattices whose tiles leave blocks without a group, whose t range is
cut, and which have no tiles."""

import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev

pytestmark = pytest.mark.gpu

LATTICES = [(8, 8, 9, 8), (16, 12, 9, 8), (20, 16, 5, 12), (12, 12, 12, 24), (24, 8, 4, 4), (6, 5, 4, 7)]


def _bits(t):
    return t.view(torch.int64).clone()


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", LATTICES, ids=lambda L: "x".join(map(str, L)))
def test_slab_walk_gives_the_same_bits(L, prec, fmt):
    U = latgen.haar_links(L, 7100 + sum(L))
    psi, phi = latgen.dirac_field(L, 7101), latgen.dirac_field(L, 7102)
    c = q.Context(0)
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    p, f = q.fermion_to_device(c, L, psi, prec, dev()), q.fermion_to_device(c, L, phi, prec, dev())
    c.close()
    got = []
    for xcd, ns in ((1, 1), (2, 1), (2, 4)):
        c = q.Context(0)
        for op in (q.OP_APE, q.OP_SHIFT, q.OP_CHAIN, q.OP_JACOBI):
            q.qdpx_tune_set(c, op, L, prec, fmt, 256, ns, xcd)
        out = [torch.zeros_like(Ud), torch.zeros_like(p), p.clone(), p.clone()]
        plaq, n1, nk = (torch.zeros(n, dtype=torch.float64, device=dev()) for n in (9, 1, 2))
        q.qdpx_ape_smear(c, L, prec, fmt, Ud, out[0], 0.5, 2, plaq, q.alloc_workspace(q.OP_APE, L, prec, fmt, 2, dev()))
        q.qdpx_eval_shift_mul_axpy(c, L, prec, fmt, Ud, p, f, 0.3, out[1], n1,
                                   q.alloc_workspace(q.OP_SHIFT, L, prec, fmt, 1, dev()))
        q.qdpx_shift_chain(c, L, prec, fmt, Ud, out[2], f, 0.3, 0.1, 2, nk,
                           q.alloc_workspace(q.OP_CHAIN, L, prec, fmt, 2, dev()))
        q.qdpx_jacobi_smear(c, L, prec, fmt, Ud, out[3], 0.21, 3, 1.5, 0xF,
                            q.alloc_workspace(q.OP_JACOBI, L, prec, fmt, 1, dev()))
        torch.cuda.synchronize()
        got.append([_bits(t) for t in (*out, plaq, n1, nk)])
        c.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert torch.equal(a, b)
