"""The batched smearing at the edges of its phase bookkeeping and launch rule:
few phases (every ticket counter on a line of its own) up to the 1024 the call
takes (counters side by side), and batches on both sides of the size from
which blocks of 256 threads are used.  Links and plaquettes are those of the
single-lattice call, bit for bit."""

import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import ctx, dev, need_gpu

pytestmark = pytest.mark.gpu

TYPES = [(q.F64, q.LINK18), (q.F32, q.LINK12), (q.F32, q.LINK18)]
TYPE_IDS = ["f64_18", "f32_12", "f32_18"]


def check(Ls, Uds, prec, fmt, n):
    """Each lattice against qdpx_ape_smear on it (once per lattice and input)."""
    c = ctx()
    outs = [q.alloc_links(L, prec, fmt, dev()) for L in Ls]
    plaq = torch.zeros(3 * len(Ls), dtype=torch.float64, device=dev())
    work = q.alloc_workspace(q.OP_BATCHED, Ls, prec, fmt, len(Ls), dev())
    q.qdpx_ape_smear_batched(c, Ls, prec, fmt, Uds, outs, 0.5, n, plaq, work)
    torch.cuda.synchronize()
    assert int(work[4:8].view(torch.int32)[0]) == 0  # no wait ran out
    seen = {}
    for i, (L, U) in enumerate(zip(Ls, Uds)):
        if (L, U.data_ptr()) not in seen:
            out = q.alloc_links(L, prec, fmt, dev())
            p = torch.zeros(3 * (n + 1), dtype=torch.float64, device=dev())
            q.qdpx_ape_smear(c, L, prec, fmt, U, out, 0.5, n, None, q.alloc_workspace(q.OP_APE, L, prec, fmt, n, dev()))
            q.qdpx_plaquette(c, L, prec, fmt, out, p, q.alloc_workspace(q.OP_PLAQ, L, prec, fmt, 1, dev()))
            seen[(L, U.data_ptr())] = q.links_to_host(c, L, out, prec, fmt), p[:3].cpu()
        links, p = seen[(L, U.data_ptr())]
        assert (q.links_to_host(c, L, outs[i], prec, fmt) == links).all(), (i, L)
        assert torch.equal(plaq[3 * i:3 * i + 3].cpu(), p), (i, L)


@pytest.mark.parametrize("prec,fmt", TYPES, ids=TYPE_IDS)
@pytest.mark.parametrize("n", [1, 34, 35, 140, 1024])
def test_phase_counts(prec, fmt, n):
    need_gpu()
    Ls = [(2, 2, 2, 2), (3, 5, 4, 7), (8, 8, 8, 4)]
    Uds = [q.links_to_device(ctx(), L, latgen.haar_links(L, 5300 + i), prec, fmt, dev()) for i, L in enumerate(Ls)]
    check(Ls, Uds, prec, fmt, n)


@pytest.mark.parametrize("prec,fmt", TYPES, ids=TYPE_IDS)
@pytest.mark.parametrize("copies", [15, 17])
def test_both_sides_of_the_size_rule(prec, fmt, copies):
    """15 or 17 lattices of 16^4 (1024 groups each; the rule changes at 16384)."""
    need_gpu()
    L = (16, 16, 16, 16)
    U = q.links_to_device(ctx(), L, latgen.haar_links(L, 5400), prec, fmt, dev())
    check([L] * copies, [U] * copies, prec, fmt, 3)
