"""The backward pass at the edges of its runs and tables: runs of 256 and up to
2,048 links, a table of 512 triangles emptied when another 256 might not fit,
then of up to 511 vertices, past which contributions go to memory at once.
Links of random cells, directions and triangles of a random soup (every
triangle distinct, a few triangles, one triangle), against the formula in
float64.  Each vertex sums at most a few hundred float32 additions here: the
tolerance is 256 float32 roundings of the sum of its terms' magnitudes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 255, 256, 257, 2047, 2048, 2049, 3000000])
@pytest.mark.parametrize("tris", [1, 40, 20000])
def test_against_the_formula(n, tris, dtype):
    import paper_2512_01251_amd as geo
    rng = np.random.default_rng(n + tris)
    n0, nb = (64, 64, 64), 4096
    nv = 3 * tris if tris < 1000 else tris // 2
    V = rng.uniform(4, 60, (nv, 3)).astype(dtype)
    T = rng.integers(0, nv, (tris, 3)).astype(np.int32)
    if tris < 1000:
        T = np.arange(3 * tris, dtype=np.int32).reshape(-1, 3)
    cell = np.sort(rng.integers(0, 64 * nb, n)).astype(np.int32)
    k = rng.integers(0, 26, n)
    k = (k + (k >= 13)).astype(np.uint8)
    tri = rng.integers(0, tris, n).astype(np.int32)
    tri[rng.random(n) < 0.01] = -1  # no hit
    g = (rng.uniform(-1, 1, n) * (rng.random(n) > 0.05)).astype(np.float32)
    t = lambda a: torch.from_numpy(a).cuda()
    tv, tt = t(V), t(T)
    coord = torch.empty((nb, 3), dtype=torch.int32, device="cuda")
    geo.geo_level0_blocks(n0, coord)
    lv = geo.make_level(n0, 0, coord, [])
    grad = torch.zeros((nv, 3), dtype=torch.float32, device="cuda")
    geo.geo_cutlinks_backward(geo.make_mesh(tv, tt), lv, n, t(cell), t(k), t(tri), t(g), grad)
    bc = coord.cpu().numpy()[cell >> 6]
    tc = cell & 63
    X = 4 * bc + np.stack([tc & 3, tc >> 2 & 3, tc >> 4], 1) + 0.5
    d = np.stack([k.astype(int) % 3 - 1, k.astype(int) // 3 % 3 - 1, k.astype(int) // 9 - 1], 1).astype(np.float64)
    P = V.astype(np.float64)[T[np.maximum(tri, 0)]]
    N = np.cross(P[:, 1] - P[:, 0], P[:, 2] - P[:, 0])
    nd, nn = (N * d).sum(1), (N * N).sum(1)
    ok = (tri >= 0) & (nd != 0) & (nn != 0)
    with np.errstate(divide="ignore", invalid="ignore"):
        H = X + ((N * (P[:, 0] - X)).sum(1) / nd)[:, None] * d
        f = [(N * np.cross(P[:, (j + 1) % 3] - H, P[:, (j + 2) % 3] - H)).sum(1) / nn * g / nd for j in range(3)]
    ref, mag = np.zeros((nv, 3)), np.zeros((nv, 3))
    for j in range(3):
        term = f[j][ok, None] * N[ok]
        np.add.at(ref, T[tri[ok], j], term)
        np.add.at(mag, T[tri[ok], j], np.abs(term))
    err = np.abs(grad.cpu().numpy() - ref)
    assert (err <= 256 * 2.0 ** -24 * mag).all(), float((err / np.maximum(mag, 1e-300)).max())
