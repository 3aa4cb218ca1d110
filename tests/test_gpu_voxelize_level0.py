"""Voxelization of level 0, whose blocks are no families of 8 children: 4 blocks
to a wave, also where that leaves a remainder.  A box against its closed form."""
import numpy as np
import pytest
import torch

from synth import meshes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n0", [(4, 4, 4), (8, 4, 4), (12, 4, 4), (16, 4, 4), (20, 4, 4), (12, 20, 4), (36, 20, 28),
                                (132, 124, 140)])
def test_box(n0):
    import paper_2512_01251_amd as geo
    lo, hi = np.array([0.8, 1.2, 0.9]), np.array(n0) - np.array([0.7, 1.3, 1.6])
    m = meshes.box(lo, hi)
    V, T = torch.from_numpy(m.verts).cuda(), torch.from_numpy(m.tris).cuda()
    nb = [v // 4 for v in n0]
    nk, cap = n0[1] * n0[2], 4 * n0[1] * n0[2]
    coord = torch.empty((nb[0] * nb[1] * nb[2], 3), dtype=torch.int32, device="cuda")
    geo.geo_level0_blocks(n0, coord)
    lv = geo.make_level(n0, 0, coord, [])
    off = torch.empty(nk + 1, dtype=torch.int32, device="cuda")
    val = torch.empty(cap, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    rows = geo.make_bins(geo.GEO_BINS_ROWS, nk, off, val, cap, cnt)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_BINS_ROWS, nk, cap), dtype=torch.uint8, device="cuda")
    geo.geo_build_bins(geo.make_mesh(V, T), lv, geo.GEO_BINS_ROWS, geo.GEO_PREC_F64, rows, None, ws)
    n = coord.shape[0]
    solid = torch.full((n + 8,), -7, dtype=torch.int64, device="cuda")
    geo.geo_voxelize(lv, rows, solid)
    assert int(cnt.item()) <= cap and (solid[n:] == -7).all()
    ins = [(np.arange(s) + 0.5 > a) & (np.arange(s) + 0.5 < b) for s, a, b in zip(n0, lo, hi)]
    c = ins[2][:, None, None] & ins[1][:, None] & ins[0]  # [z, y, x]
    c = c.reshape(nb[2], 4, nb[1], 4, nb[0], 4).transpose(0, 2, 4, 1, 3, 5).reshape(-1, 64).astype(np.uint64)
    ref = (c << np.arange(64, dtype=np.uint64)).sum(1, dtype=np.uint64)
    assert np.array_equal(solid[:n].cpu().numpy().view(np.uint64), ref)
