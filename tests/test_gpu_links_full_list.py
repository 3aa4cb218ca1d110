"""LINKS bins of more pieces of large triangles than their list holds (65,536):
the rest is done by the waves that found them.  The triangles are halves of
axis-aligned faces of boxes nested closely, with thousands of candidate blocks
each; the blocks that each one meets are known in closed form."""
import numpy as np
import pytest
import torch

from synth import meshes
from test_gpu_links_pieces import _met

pytestmark = pytest.mark.gpu

LIST_CAP, STEP, PIECES = 65536, 256, 64  # the list's entries; candidates that a wave does itself; most pieces


def _pieces(P, nb):
    """Pieces of triangles P [t, 3, 3]: the blocks whose widened box meets the bounding box, cut in multiples of 256."""
    lo = np.maximum(np.ceil((P.min(1) - 4.5) / 4 - 1e-7), 0)
    hi = np.minimum(np.floor((P.max(1) + 0.5) / 4 + 1e-7), nb - 1)
    n = (hi - lo + 1).prod(1).astype(np.int64)
    piece = ((n + PIECES - 1) // PIECES + STEP - 1) // STEP * STEP
    return np.where(n > STEP, (n + piece - 1) // piece, 0)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_more_pieces_than_the_list_holds(dtype):
    import paper_2512_01251_amd as geo
    n, n0, nb, boxes = 256, (256, 256, 256), 64, 400
    k = np.arange(boxes)
    lo = np.stack([4.03 + 0.0131 * k, 4.07 + 0.0137 * k, 4.11 + 0.0139 * k], 1)
    m = meshes.merge([meshes.box(a, n - a) for a in lo])
    nt = 12 * boxes
    verts = m.verts.astype(dtype)
    P = verts[m.tris].astype(np.float64)
    assert _pieces(P, nb).sum() > 1.2 * LIST_CAP
    V, T = torch.from_numpy(verts).cuda(), torch.from_numpy(m.tris).cuda()
    coord = torch.empty((nb ** 3, 3), dtype=torch.int32, device="cuda")
    geo.geo_level0_blocks(n0, coord)
    cap = nt * 2 * nb * nb
    off = torch.empty(nb ** 3 + 1, dtype=torch.int32, device="cuda")
    val = torch.empty(cap, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    bins = geo.make_bins(geo.GEO_BINS_LINKS, nb ** 3, off, val, cap, cnt)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_BINS_LINKS, nb ** 3, cap), dtype=torch.uint8, device="cuda")
    geo.geo_build_bins(geo.make_mesh(V, T), geo.make_level(n0, 0, coord, []), geo.GEO_BINS_LINKS, geo.GEO_PREC_F64,
                       bins, None, ws)
    total = int(cnt.item())
    assert total <= cap and int(off[-1]) == total
    block = torch.repeat_interleave(torch.arange(nb ** 3, device="cuda"), torch.diff(off.long()))
    got = torch.sort(block * nt + val[:total].long())[0]
    assert torch.all(got[1:] > got[:-1])  # none twice
    want, most = [], []
    for t in range(nt):
        for keep, grow in ((want, 0.0), (most, 1e-3)):
            b = _met(P[t], nb, grow)
            keep.append((b[:, 0] + nb * (b[:, 1] + nb * b[:, 2])) * nt + t)
    got = got.cpu().numpy()
    assert np.isin(np.concatenate(want), got).all()
    assert np.isin(got, np.concatenate(most)).all()
