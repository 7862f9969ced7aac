"""FP64 smearing steps with every smear mask, whose planes lie in one, two,
three or none of the step's phases, above the size where the split kernel ends
(128 groups), ragged and not, with one and four groups a wave: against the
oracle, the other directions bit for bit."""

import numpy as np
import pytest
import torch

import latgen
import oracle
import paper_1105_2279_amd as q
from gpuhelp import dev, link_err, tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ns", [1, 4])
@pytest.mark.parametrize("L", [(8, 8, 13, 10), (13, 9, 11, 7)], ids=lambda L: "x".join(map(str, L)))
def test_every_mask(L, ns):
    assert np.prod(L) > 128 * 64
    U = latgen.haar_links(L, 7900 + sum(L))
    c = q.Context(0)
    q.qdpx_tune_set(c, q.OP_APE, L, q.F64, q.LINK18, 256, ns, 1, 1)
    Ud = q.links_to_device(c, L, U, q.F64, q.LINK18, dev())
    for mask in range(16):
        out = torch.zeros_like(Ud)
        q.qdpx_ape_smear(c, L, q.F64, q.LINK18, Ud, out, 0.5, 1, smear_mask=mask)
        V = q.links_to_host(c, L, out, q.F64, q.LINK18)
        torch.cuda.synchronize()
        assert link_err(V, oracle.ape_step(U, 0.5, mask)) < tol(q.F64), mask
        for mu in range(4):
            if not (mask >> mu) & 1:
                assert np.array_equal(V[..., mu, :, :].view(np.float64), U[..., mu, :, :].view(np.float64)), (mask, mu)
    c.close()
