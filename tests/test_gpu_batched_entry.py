"""Which batches a stored batched geometry is used for.  The groups per ticket
of a call show in the device table it builds: a later call in a given geometry
may be captured exactly when an eager one took the same number."""

import json

import pytest
import torch

import latgen
import paper_1105_2279_amd as q
from gpuhelp import dev

pytestmark = pytest.mark.gpu

LS = [(8, 8, 8, 8), (4, 4, 4, 6)]  # 70 groups: the default is 2 a ticket


def _captured(c, Us, outs, work, chunk):
    q.qdpx_tune_set(c, q.OP_BATCHED, LS[0], q.F64, q.LINK18, 256, chunk, 1)
    s, g, err = torch.cuda.Stream(), torch.cuda.CUDAGraph(), None
    with torch.cuda.graph(g, stream=s):
        try:
            q.qdpx_ape_smear_batched(c, LS, q.F64, q.LINK18, Us, outs, 0.5, 1, None, work, stream=s)
        except q.QdpxError as e:
            err = e
    assert err is None or err.code == -6
    return err is None


@pytest.mark.parametrize("groups,chunk", [(225168, 2), (16385, 2), (16384, 4), (None, 4)])
def test_entry_of_a_large_batch_is_not_for_a_small_one(tmp_path, groups, chunk):
    table = str(tmp_path / "table.json")
    entry = {"op": "BATCHED", "prec": "F64", "fmt": "LINK18", "L": [8, 8, 8, 8], "launch": [256, 4, 1, 1, 0]}
    with open(table, "w") as fh:
        json.dump({"device": torch.cuda.get_device_properties(0).gcnArchName,
                   "entries": [dict(entry, **({} if groups is None else {"groups": groups}))]}, fh)
    c = q.Context(0, tune_cache=table)
    assert q.qdpx_tune_get(c, q.OP_BATCHED, LS[0], q.F64, q.LINK18) == (256, 4, 1, 1, 0)
    Us = [q.links_to_device(c, L, latgen.haar_links(L, 8300), q.F64, q.LINK18, dev()) for L in LS]
    outs = [torch.zeros_like(u) for u in Us]
    work = q.alloc_workspace(q.OP_BATCHED, LS, q.F64, q.LINK18, device=dev())
    q.qdpx_ape_smear_batched(c, LS, q.F64, q.LINK18, Us, outs, 0.5, 1, None, work)
    torch.cuda.synchronize()
    took = [n for n in (1, 2, 4) if _captured(c, Us, outs, work, n)]
    assert took == [chunk]
    c.close()


def test_tuned_geometry_keeps_its_batch_size(tmp_path):
    table = str(tmp_path / "table.json")
    c = q.Context(0, tune_cache=table)
    q.qdpx_tune_batched(c, LS, q.F64, q.LINK18, 2)
    c.close()
    with open(table) as fh:
        assert json.load(fh)["entries"][0]["groups"] == 70
