"""LINKS bins of large triangles, which are cut into pieces, and of more pieces
than their list holds (65,536), which the waves that found them do in place
(560 boxes: about 80,000 pieces).  The triangles are halves of axis-aligned
faces of nested boxes, so the blocks that each one meets are known in closed
form; the bins may hold more only where a block misses by a rounding margin."""
import numpy as np
import pytest
import torch

from synth import meshes

pytestmark = pytest.mark.gpu


def _met(P, nb, grow):
    """Blocks [k, 3] whose box [4b - 1/2, 4b + 4.5] grown by `grow` meets the
    closed axis-aligned right triangle P."""
    lo, hi = P.min(0), P.max(0)
    r = [np.arange(max(0, int(np.ceil((lo[a] - 4.5 - grow) / 4))),
                   min(nb - 1, int(np.floor((hi[a] + 0.5 + grow) / 4))) + 1) for a in range(3)]
    b = np.stack(np.meshgrid(*r, indexing="ij"), 3).reshape(-1, 3)
    flat = int(np.argmin(hi - lo))
    u, w = [a for a in range(3) if a != flat]
    # the hypotenuse's side on which the right-angle vertex lies
    corner = next(i for i in range(3) if all((P[i] == P[(i + 1) % 3])[a] or (P[i] == P[(i + 2) % 3])[a] for a in (u, w)))
    A, B = P[(corner + 1) % 3], P[(corner + 2) % 3]
    n = np.array([B[w] - A[w], A[u] - B[u]])
    if n @ (P[corner][[u, w]] - A[[u, w]]) > 0:
        n = -n
    box0, box1 = 4.0 * b - 0.5 - grow, 4.0 * b + 4.5 + grow
    # the box's nearest corner along -n must be on the triangle's side
    near = np.where(n > 0, box0[:, [u, w]], box1[:, [u, w]])
    return b[(near - A[[u, w]]) @ n <= 1e-9 * grow]


@pytest.mark.parametrize("boxes", [1, 560])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_nested_boxes(boxes, dtype):
    import paper_2512_01251_amd as geo
    n, n0, nb = 128, (128, 128, 128), 32
    k = np.arange(boxes)
    lo = np.stack([8.03 + 0.0931 * k, 8.07 + 0.0937 * k, 8.11 + 0.0939 * k], 1)
    hi = np.stack([119.91 - 0.0941 * k, 119.95 - 0.0943 * k, 119.97 - 0.0949 * k], 1)
    m = meshes.merge([meshes.box(a, b) for a, b in zip(lo, hi)])
    verts = m.verts.astype(dtype)
    V, T = torch.from_numpy(verts).cuda(), torch.from_numpy(m.tris).cuda()
    coord = torch.empty((nb ** 3, 3), dtype=torch.int32, device="cuda")
    geo.geo_level0_blocks(n0, coord)
    lv = geo.make_level(n0, 0, coord, [])
    cap = 12 * boxes * 2 * nb * nb
    off = torch.empty(nb ** 3 + 1, dtype=torch.int32, device="cuda")
    val = torch.empty(cap, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    bins = geo.make_bins(geo.GEO_BINS_LINKS, nb ** 3, off, val, cap, cnt)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_BINS_LINKS, nb ** 3, cap), dtype=torch.uint8, device="cuda")
    geo.geo_build_bins(geo.make_mesh(V, T), lv, geo.GEO_BINS_LINKS, geo.GEO_PREC_F64, bins, None, ws)
    total = int(cnt.item())
    assert total <= cap
    o = off.cpu().numpy().astype(np.int64)
    assert o[-1] == total
    block = np.repeat(np.arange(nb ** 3), np.diff(o))
    got = np.sort(block * (12 * boxes) + val[:total].cpu().numpy())
    assert len(np.unique(got)) == total
    want, most = [], []
    for t in range(12 * boxes):
        P = verts[m.tris[t]].astype(np.float64)
        for keep, grow in ((want, 0.0), (most, 1e-3)):
            b = _met(P, nb, grow)
            keep.append((b[:, 0] + nb * (b[:, 1] + nb * b[:, 2])) * (12 * boxes) + t)
    assert np.isin(np.concatenate(want), got).all()
    assert np.isin(got, np.concatenate(most)).all()
