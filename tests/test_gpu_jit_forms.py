"""Generated kernels by form against the reference evaluator: two waves a group
(a block of two groups, the second past the end or ragged, in contiguous and
tile order) and flat kernels in ranges and in dispatch order (FP64 fields of
more than 256 MB in all), with the norm."""

import numpy as np
import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import FORMAT_IDS, FORMATS, dev, rel_err, tol
from oracle import expr

pytestmark = pytest.mark.gpu

TWO = ["(sum 0x9 (umul m (shift f0 + m)))",
       "(sub (shift f1 - 2) (scale s0 (sum 0x6 (add (umul m (shift f0 + m)) (shift (uadj m f0) - m)))))",
       # three fields around it: a loop in FP32
       "(add (sum 0x3 (umul m (shift f0 + m))) (sub (scale s0 f1) (add f0 (shift f1 + 3))))"]
FLAT = ["(umul 3 (shift f0 + 3))", "(add f0 (scale s0 (shift (uadj 0 f1) - 0)))"]
# 1 group; 3 and 7, the last ragged; 2 and 130 of columns; the tile order in
# FP64 (from 88 K sites on) and in all formats (175 K), and FP64 fields of 270 MB
LATTICES = [(4, 4, 2, 2), (3, 5, 4, 3), (3, 5, 4, 7), (4, 4, 4, 2), (8, 8, 13, 10), (24, 16, 24, 20)]


@pytest.mark.parametrize("prec,fmt", FORMATS, ids=FORMAT_IDS)
@pytest.mark.parametrize("L", LATTICES, ids=lambda L: "x".join(map(str, L)))
def test_forms(L, prec, fmt, tmp_path, monkeypatch):
    monkeypatch.setenv("QDPX_JIT_CACHE", str(tmp_path))
    c, sc, n_fields = q.Context(0), [0.6], 7 if np.prod(L) > 100000 else 2
    U = latgen.haar_links(L, 7800 + sum(L))
    fields = [latgen.dirac_field(L, 7801 + i) for i in range(2)]
    Ud = q.links_to_device(c, L, U, prec, fmt, dev())
    fd = [q.fermion_to_device(c, L, f, prec, dev()) for f in fields]
    for e in TWO + FLAT:
        k = q.qdpx_jit_compile(c, e, prec, fmt, n_fields, 1)
        out, n2 = q.alloc_fermion(L, prec, dev()), torch.zeros(1, dtype=torch.float64, device=dev())
        q.qdpx_jit_eval(c, k, L, Ud, fd + [fd[1]] * (n_fields - 2), sc, out, n2,
                        q.alloc_workspace(q.OP_SHIFT, L, prec, fmt, 1, dev()))
        got = q.fermion_to_host(c, L, out, prec)
        torch.cuda.synchronize()
        nrm, mx = rel_err(got, expr.evaluate(e, U, fields, sc))
        assert nrm < tol(prec) and mx < tol(prec), (e, nrm, mx)
        assert abs(n2.item() / np.sum(np.abs(got) ** 2) - 1.0) < 1e-12, e
    c.close()
