"""The device-wide exclusive scan of large arrays: up to 8,192 tiles of 4,096
values each tile adds up the sums of the tiles before it, above that the sums
are scanned first.  Seen through ROWS bins of small boxes scattered over a
plane of lines: a line has two entries per box that it crosses (no face lies
on a plane of centres)."""
import numpy as np
import pytest
import torch

from synth import meshes

pytestmark = pytest.mark.gpu


def _boxes(ny, nz, count):
    rng = np.random.default_rng(ny + nz)
    lo = np.stack([np.full(count, 1.125), rng.integers(1, ny - 9, count) + 0.125,
                   rng.integers(1, nz - 9, count) + 0.375], 1)
    hi = lo + np.stack([np.full(count, 1.25), rng.integers(1, 8, count), rng.integers(1, 8, count)], 1)
    lo[-1, 1:], hi[-1, 1:] = (ny - 2.125, nz - 2.125), (ny - 0.125, nz - 0.125)  # the last line counts too
    m = meshes.merge([meshes.box(a, b) for a, b in zip(lo, hi)])
    V = torch.from_numpy(m.verts).cuda()
    return lo, hi, V, torch.from_numpy(m.tris).cuda()


def _bins(geo, nk, cap):
    off = torch.full((nk + 1,), -7, dtype=torch.int32, device="cuda")
    val = torch.empty(cap, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -7, dtype=torch.int64, device="cuda")
    return geo.make_bins(geo.GEO_BINS_ROWS, nk, off, val, cap, cnt), off, val, cnt


def _offsets(lo, hi, ny, nz, L):
    inside = []
    for a, n in ((1, ny << L), (2, nz << L)):
        c = (np.arange(n) + 0.5) / 2 ** L
        inside.append(torch.from_numpy(((lo[:, a, None] < c) & (c < hi[:, a, None])).astype(np.float32)).cuda())
    per_line = 2 * (inside[1].T @ inside[0]).reshape(-1).long()  # key = j + ny k
    return torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(per_line, 0)])


@pytest.mark.parametrize("ny,nz,lf", [(4096, 8192, 0),    # 8,192 tiles: the last without a scan of the sums
                                      (4096, 8196, 0),    # 8,196, the first with one
                                      (4100, 2052, 1),    # a level of 2,054 tiles beside one of 8,216, both part-filled
                                      (16384, 16380, 0)])  # 65,520
def test_offsets(ny, nz, lf):
    import paper_2512_01251_amd as geo
    lo, hi, V, T = _boxes(ny, nz, 2000)
    cap = 400000
    per = [_bins(geo, (ny << L) * (nz << L), cap) for L in range(lf + 1)]
    nk = sum(p[1].numel() - 1 for p in per)
    call = geo.GEO_CALL_BINS_ROWS_LEVELS
    ws = torch.empty(geo.geo_workspace_size(call, nk, cap * len(per)), dtype=torch.uint8, device="cuda")
    geo.geo_build_row_bins_levels(geo.make_mesh(V, T), (4, ny, nz), 0, geo.GEO_PREC_F64, [p[0] for p in per], None, ws)
    for L, (_, off, _, cnt) in enumerate(per):
        want = _offsets(lo, hi, ny, nz, L)
        assert int(cnt.item()) == int(want[-1]) <= cap
        assert torch.equal(off.long(), want)


def test_time_grows_like_the_array():
    import paper_2512_01251_amd as geo
    ms = []
    for n in (6144, 24576):  # 16 times the lines
        _, _, V, T = _boxes(n, n, 1)
        bins, *keep = _bins(geo, n * n, 4096)
        lv = geo.make_level((4, n, n), 0, torch.empty((0, 3), dtype=torch.int32, device="cuda"), [])
        ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_BINS_ROWS, n * n, 4096), dtype=torch.uint8, device="cuda")
        best = float("inf")
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                geo.geo_build_bins(geo.make_mesh(V, T), lv, geo.GEO_BINS_ROWS, geo.GEO_PREC_F64, bins, None, ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 5)
        ms.append(best)
        del bins, keep, ws
    assert ms[1] < 24 * ms[0], ms
