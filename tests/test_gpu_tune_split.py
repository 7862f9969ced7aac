"""qdpx_tune on lattices where the Gram-Schmidt step has no launch geometry: the
polar step is timed, so no LDS tile is chosen among equal ones, and its links do
not depend on what was chosen."""

import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", [(4, 4, 4, 4), (8, 8, 8, 16)], ids=lambda L: "x".join(map(str, L)))
def test_tuned_geometry_of_few_groups(L, prec, fmt):
    c = q.Context(0)
    Ud = q.links_to_device(c, L, latgen.haar_links(L, 8400), prec, fmt, dev())
    out = [torch.zeros_like(Ud) for _ in range(4)]

    def smear(k):
        for p in (q.PROJ_POLAR, q.PROJ_GRAM_SCHMIDT):
            q.qdpx_ape_smear(c, L, prec, fmt, Ud, out[2 * k + (p == q.PROJ_POLAR)], 0.5, 1, projection=p)

    smear(0)
    q.qdpx_tune(c, q.OP_APE, L, prec, fmt)
    assert q.qdpx_tune_source(c, q.OP_APE, L, prec, fmt) == "tuned"
    block, ns, xcd, tw, lds = q.qdpx_tune_get(c, q.OP_APE, L, prec, fmt)
    assert block in (256, 512) and ns in (1, 2, 4) and xcd in (0, 1, 2) and L[3] % tw == 0
    assert lds == (4 if prec == q.F32 else 0)
    smear(1)
    torch.cuda.synchronize()
    assert torch.equal(out[0].view(torch.int64), out[2].view(torch.int64))
    assert torch.equal(out[1].view(torch.int64), out[3].view(torch.int64))
    c.close()
