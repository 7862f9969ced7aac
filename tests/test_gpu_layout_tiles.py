"""Layout conversion at the edges of its site tiles: lattices smaller than a
tile, ending inside one and filling tiles exactly, against the documented
layout formed with numpy; what lies behind the last site stays untouched."""

import numpy as np
import pytest
import torch

import paper_1105_2279_amd as q

pytestmark = pytest.mark.gpu

LATTICES = [(2, 2, 2, 2), (3, 3, 3, 3), (4, 4, 4, 2), (5, 3, 5, 7), (4, 4, 4, 4), (3, 7, 6, 3)]
FORMATS = [(q.F64, q.LINK18), (q.F32, q.LINK18), (q.F32, q.LINK12)]


def _guarded(nbytes, fill):
    return torch.full((nbytes + 4096,), fill, dtype=torch.uint8, device="cuda")


def _soa(cols, S, paired, fill):
    """(components, V, 2) values in the SoA layout as bytes, holes holding `fill`."""
    n, V, _ = cols.shape
    parts, at = [], 0
    while at < n:
        w = 2 if paired and at + 1 < n else 1
        a = np.frombuffer(bytes([fill]) * (S * w * 2 * cols.itemsize), dtype=cols.dtype).copy().reshape(S, w, 2)
        a[:V] = cols[at:at + w].transpose(1, 0, 2)
        parts.append(a.reshape(-1))
        at += w
    return np.concatenate(parts)


@pytest.mark.parametrize("L", LATTICES)
@pytest.mark.parametrize("prec,fmt", FORMATS)
def test_links_tile_edges(L, prec, fmt):
    V, S = int(np.prod(L)), q.qdpx_site_stride(L)
    dt = np.float64 if prec == q.F64 else np.float32
    rows = 2 if fmt == q.LINK12 else 3
    aos = np.random.default_rng(V).standard_normal((V, 4, 9, 2))
    ctx = q.Context(0)
    nb = q.qdpx_links_bytes(L, prec, fmt)
    soa = _guarded(nb, 0x5A)
    q.qdpx_pack_links(ctx, L, torch.from_numpy(aos).cuda(), prec, fmt, soa)
    want = np.concatenate([_soa(aos[:, mu, :3 * rows].transpose(1, 0, 2).astype(dt), S, prec == q.F32, 0x5A)
                           for mu in range(4)])
    got = soa.cpu().numpy()
    assert (got[:nb].view(dt).view(np.uint8) == want.view(np.uint8)).all()
    assert (got[nb:] == 0x5A).all()
    back = _guarded(V * 4 * 144, 0x33)
    q.qdpx_unpack_links(ctx, L, soa, prec, fmt, back)
    back = back.cpu().numpy()
    assert (back[V * 576:] == 0x33).all()
    m = back[:V * 576].view(np.float64).reshape(V, 4, 9, 2)
    held = aos.astype(dt).astype(np.float64)
    assert (m[:, :, :3 * rows] == held[:, :, :3 * rows]).all()
    if rows == 2:
        z = held[..., 0] + 1j * held[..., 1]
        r2 = np.cross(z[:, :, 0:3], z[:, :, 3:6]).conj()
        # four products and three sums of doubles below about 10 x 10
        assert np.abs((m[..., 6:, 0] + 1j * m[..., 6:, 1]) - r2).max() < 1e-13


@pytest.mark.parametrize("L", LATTICES)
@pytest.mark.parametrize("prec", [q.F64, q.F32])
def test_fermion_tile_edges(L, prec):
    V, S = int(np.prod(L)), q.qdpx_site_stride(L)
    dt = np.float64 if prec == q.F64 else np.float32
    aos = np.random.default_rng(V + 1).standard_normal((V, 12, 2))
    ctx = q.Context(0)
    nb = q.qdpx_fermion_bytes(L, prec)
    soa = _guarded(nb, 0x5A)
    q.qdpx_pack_fermion(ctx, L, torch.from_numpy(aos).cuda(), prec, soa)
    want = _soa(aos.transpose(1, 0, 2).astype(dt), S, prec == q.F32, 0x5A)
    got = soa.cpu().numpy()
    assert (got[:nb].view(dt).view(np.uint8) == want.view(np.uint8)).all()
    assert (got[nb:] == 0x5A).all()
    back = _guarded(V * 192, 0x33)
    q.qdpx_unpack_fermion(ctx, L, soa, prec, back)
    back = back.cpu().numpy()
    assert (back[V * 192:] == 0x33).all()
    assert (back[:V * 192].view(np.float64).reshape(V, 12, 2) == aos.astype(dt).astype(np.float64)).all()
