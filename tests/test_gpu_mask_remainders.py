"""The link-mask pass where no chunk length divides the number of blocks: 31 x 33
blocks per layer and odd layers, so that the last chunk of every length is
part-filled, with a body in the last blocks of the level and one in the first.
The bodies' links must be those of the smallest grid, which is checked against
the oracle, those of the last blocks shifted by the layers added between."""
import dataclasses

import numpy as np
import pytest

import oracle
from synth import configs, meshes
from gpu_helpers import compare, gpu_embed, say

pytestmark = pytest.mark.gpu

NX, NY, LAYER = 124, 132, 31 * 33
_base = []


def _work(layers):
    star = configs.star_small(n0=96)
    top = np.array([NX, NY, 4 * layers], dtype=np.float64)
    box = meshes.box(top - (14.375, 12.75, 15.125), top - (0.6875, 0.8125, 1.4375))  # its last block is the level's
    return dataclasses.replace(star, mesh=meshes.merge([star.mesh, box]), n0=(NX, NY, 4 * layers), lf=0)


def _table(emb):
    k = emb.links
    return [x.cpu().numpy() for x in (k.cell, k.dir, k.q, k.tri, k.mask)]


@pytest.mark.parametrize("layers,chunk", [(27, 2), (33, 4), (65, 8), (129, 16), (257, 32), (513, 64)])
def test_links_with_a_part_filled_last_chunk(layers, chunk):
    if not _base:
        w = _work(27)
        emb, _, _ = gpu_embed(w, "f32")
        compare(w, emb, oracle.embed(w.mesh, w.n0, w.lf, w.lattice, w.d_spec))
        _base.append(_table(emb))
    nb = LAYER * layers
    assert 8192 * chunk <= nb < 16384 * chunk or chunk == 64 and nb >= 8192 * 64 or chunk == 2 and nb < 32768
    assert nb % chunk
    emb, _, _ = gpu_embed(_work(layers), "f32")
    cell, dr, q, tri, mask = _table(emb)
    say(f"[mask remainders] {nb} blocks ({chunk} per wave, {nb % chunk} in the last): {len(cell)} links")
    cell0, dr0, q0, tri0, mask0 = _base[0]
    shift = 64 * LAYER * (layers - 27)
    split = 64 * LAYER * 23  # the box's links are in the last 4 layers
    assert cell0.max() >> 6 == LAYER * 27 - 1
    assert np.array_equal(cell, np.where(cell0 < split, cell0, cell0 + shift))
    assert np.array_equal(dr, dr0) and np.array_equal(q, q0) and np.array_equal(tri, tri0)
    assert np.array_equal(mask[:split], mask0[:split]) and np.array_equal(mask[split + shift:], mask0[split:])
    assert not mask[split:split + shift].any()
