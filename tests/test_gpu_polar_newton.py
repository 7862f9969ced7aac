"""The polar projection over the condition numbers of W: the Newton iteration
stops lane by lane, so well and ill conditioned links share waves here, and
the first step of a lane may start at any norm.  Reference: singular vectors
of the oracle's W, the determinant's phase removed on the principal branch."""

import numpy as np
import pytest

import latgen
import oracle
import paper_1105_2279_amd as q
import torch
from gpuhelp import ctx, dev

pytestmark = pytest.mark.gpu


# alpha 1: W is the staple sum alone (condition numbers of several thousand);
# 0.02: next to the link, all singular values near 1; -3, 40: far from norm 3
@pytest.mark.parametrize("alpha", [1.0, 0.5, 0.02, -3.0, 40.0])
@pytest.mark.parametrize("mask", [0xF, 0x7])
def test_polar_over_condition_numbers(alpha, mask):
    L = (8, 8, 6, 9)
    U = latgen.haar_links(L, 5400)
    c = ctx()
    Ud = q.links_to_device(c, L, U, q.F64, q.LINK18, dev())
    out = q.alloc_links(L, q.F64, q.LINK18, dev())
    q.qdpx_ape_smear(c, L, q.F64, q.LINK18, Ud, out, alpha, 1, None, None, smear_mask=mask, projection=q.PROJ_POLAR)
    got = q.links_to_host(c, L, out, q.F64, q.LINK18)
    torch.cuda.synchronize()
    dirs = [mu for mu in range(4) if mask >> mu & 1]
    W = oracle.ape_w(U, alpha, mask)[..., dirs, :, :].reshape(-1, 3, 3)
    u, s, vh = np.linalg.svd(W)
    V = u @ vh
    V *= np.exp(-1j * np.angle(np.linalg.det(W)) / 3)[:, None, None]
    err = np.abs(got[..., dirs, :, :].reshape(-1, 3, 3) - V).max((1, 2))
    # a change dW of W moves the factor and the phase by about |dW| / s_min;
    # |dW| is some tens of roundings of the largest singular value
    assert (err < 100 * np.finfo(float).eps * s[:, 0] / s[:, 2]).all(), (err * s[:, 2] / s[:, 0]).max()
