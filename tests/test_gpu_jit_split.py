"""Generated kernels whose sum is split over the waves of a group, and ones
whose sum is not, in the contiguous and the tile block order and on lattices
ending inside a group, with the norm, against the reference evaluator."""

import numpy as np
import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev, rel_err, tol
from oracle import expr

pytestmark = pytest.mark.gpu

EXPRS = [
    # split: a partial mask between plain terms on both sides, a double shift
    "(sub (add (shift (shift f1 + 3) - 0) (scale s0 (sum 0xB (uadj m (shift f0 - m))))) (scale s1 f0))",
    # split: nothing around the sum; a link and a field of the sum at one site
    "(sum 0x6 (sub (umul m (shift f0 + m)) (shift (uadj m f1) - m)))",
    # not split: a link outside the sum; two sums; one direction
    "(add f1 (umul 2 (scale s0 (sum 0xF (umul m (shift f0 + m))))))",
    "(add (sum 0x3 (umul m (shift f0 + m))) (scale s1 (sum 0xC (uadj m f1))))",
    "(add f1 (scale s0 (sum 0x4 (umul m (shift f0 + m)))))",
]
# one group, a ragged end, and two beyond the size from which the tile order
# is taken (FP64 88 K sites, FP32-12 175 K): with columns, and without
LATTICES = [(4, 4, 2, 2), (3, 5, 4, 7), (24, 16, 24, 20), (14, 18, 22, 34)]


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", LATTICES, ids=lambda L: "x".join(map(str, L)))
def test_split_sums(L, prec, fmt, tmp_path, monkeypatch):
    monkeypatch.setenv("QDPX_JIT_CACHE", str(tmp_path))
    c, sc = q.Context(0), [0.6, -1.7]
    U = latgen.haar_links(L, 7300 + sum(L))
    fields = [latgen.dirac_field(L, 7301 + i) for i in range(2)]
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    fd = [q.fermion_to_device(c, L, f, prec, dev()) for f in fields]
    for e in EXPRS if np.prod(L) < 10000 else EXPRS[:3]:
        k = q.qdpx_jit_compile(c, e, prec, fmt, 2, 2)
        out, n2 = q.alloc_fermion(L, prec, dev()), torch.zeros(1, dtype=torch.float64, device=dev())
        q.qdpx_jit_eval(c, k, L, Ud, fd, sc, out, n2, q.alloc_workspace(q.OP_SHIFT, L, prec, fmt, 1, dev()))
        got = q.fermion_to_host(c, L, out, prec)
        torch.cuda.synchronize()
        nrm, mx = rel_err(got, expr.evaluate(e, U, fields, sc))
        assert nrm < tol(prec) and mx < tol(prec), (e, nrm, mx)
        # the norm is of the stored values, every product and sum in FP64
        assert abs(n2.item() / np.sum(np.abs(got) ** 2) - 1.0) < 1e-12, e
    c.close()
