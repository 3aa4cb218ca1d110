"""Voxelization of block lists that are not made of whole families of 8
children, and of lines with many entries: the same blocks as in the forest's
own list, permuted, cut short or with a family broken up, get the same masks."""
import numpy as np
import pytest
import torch

from synth import configs, meshes
from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu


def _nested(n=20):  # lines with 40 crossings
    return configs.Workload("nested", meshes.merge([meshes.box((4.1 + 0.53 * k,) * 3, (27.9 - 0.51 * k,) * 3)
                                                    for k in range(n)]), (32, 32, 32), 1, 19)


@pytest.mark.parametrize("name", ["star", "nested"])
def test_any_block_list(name):
    import paper_2512_01251_amd as geo
    from paper_2512_01251_amd import pipeline
    w = configs.star_small(lf=2) if name == "star" else _nested()
    V, T = to_gpu(w.mesh)
    emb = pipeline.Embedder().embed(V, T, w.n0, w.lf, w.lattice, w.d_spec, "f32", with_links=False)
    rec = emb.levels[-1]
    maps = [lv.child_map for lv in emb.levels[:-1]]
    nb, n = int(rec.bcoord.shape[0]), int(rec.rows_val.numel())
    nk = (w.n0[1] << w.lf) * (w.n0[2] << w.lf)
    cnt = torch.full((1,), n, dtype=torch.int64, device="cuda")
    rows = geo.make_bins(geo.GEO_BINS_ROWS, nk, rec.rows_off, rec.rows_val, n, cnt)
    rng = np.random.default_rng(5)
    swap = np.arange(nb)
    swap[[3, 8 * 20 + 6]] = swap[[8 * 20 + 6, 3]]
    for order in (np.arange(nb), np.arange(nb)[4:], np.arange(nb)[:13], rng.permutation(nb), swap, np.arange(nb)[::-1],
                  np.array([0])):
        i = torch.from_numpy(np.ascontiguousarray(order)).cuda()
        coord = rec.bcoord[i].contiguous()
        solid = torch.full((len(order),), 7, dtype=torch.int64, device="cuda")
        geo.geo_voxelize(geo.make_level(w.n0, w.lf, coord, maps), rows, solid)
        assert torch.equal(solid, rec.solid[i])
