"""The device-wide exclusive scan at the edges of its tiles (4,096 values) and
of its three ways: one tile, tiles that read the values before them (up to 4
tiles), tiles that add up the tiles' sums.  Seen through the dense layout's
block map and boundary-block count, which are the scan of the blocks' flags."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb", [1, 63, 4095, 4096, 4097, 8192, 16383, 16384, 16385, 20480, 20481, 1100003])
def test_block_map_is_the_scan_of_the_flags(nb):
    import paper_2512_01251_amd as geo
    rng = np.random.default_rng(nb)
    has = rng.random(nb) < 0.4
    has[-1] = True  # the last value counts in the total only
    b = np.flatnonzero(has)
    cell = torch.from_numpy((64 * b + rng.integers(0, 64, len(b))).astype(np.int32)).cuda()
    dr = torch.full((len(b),), 14, dtype=torch.uint8, device="cuda")
    q = torch.rand(len(b), device="cuda")
    tri = torch.arange(len(b), dtype=torch.int32, device="cuda")
    lv = geo.geo_level()
    coord = torch.zeros((nb, 3), dtype=torch.int32, device="cuda")
    for a in range(3):
        lv.n0[a] = 4
    lv.level, lv.nblocks, lv.bcoord = 0, nb, coord.data_ptr()
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_LINKS_DENSE, nb, 0), dtype=torch.uint8, device="cuda")
    bmap = torch.full((nb,), -7, dtype=torch.int32, device="cuda")
    d_n = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    dq = torch.empty((1, 18, 64), device="cuda")
    dt = torch.empty((1, 18, 64), dtype=torch.int32, device="cuda")
    geo.geo_links_dense(lv, len(b), cell, dr, q, tri, 19, 1, bmap, dq, dt, d_n, ws)
    assert int(d_n.item()) == len(b)
    assert np.array_equal(bmap.cpu().numpy(), np.where(has, np.cumsum(has) - 1, -1))
