"""The link-mask pass takes 64 blocks per wave on large levels and fewer on
small ones.  The grid of one body is extended along z, which leaves the block
indices of its lower part as they are: at level sizes on every chunk length (2
to 64 blocks, the last one part-filled) the link table and the masks must stay
those of the smallest grid, which are checked against the oracle."""
import dataclasses

import numpy as np
import pytest

import oracle
from synth import configs
from gpu_helpers import compare, gpu_embed, say

pytestmark = pytest.mark.gpu

_base = []


def _work(layers):
    return dataclasses.replace(configs.star_small(n0=128), n0=(128, 128, 4 * layers), lf=0)


def _table(emb):
    k = emb.links
    return [x.cpu().numpy() for x in (k.cell, k.dir, k.q, k.tri, k.mask)]


@pytest.mark.parametrize("layers,chunk", [(31, 2), (33, 4), (65, 8), (129, 16), (257, 32), (513, 64)])
def test_links_whatever_the_chunk(layers, chunk):
    if not _base:
        w = _work(31)
        emb, _, _ = gpu_embed(w, "f32")
        compare(w, emb, oracle.embed(w.mesh, w.n0, w.lf, w.lattice, w.d_spec))
        _base.append(_table(emb))
    emb, _, _ = gpu_embed(_work(layers), "f32")
    *links, mask = _table(emb)
    say(f"[mask chunks] {layers} layers of 1,024 blocks ({chunk} per wave): {len(links[0])} links")
    for got, ref in zip(links, _base[0]):
        assert np.array_equal(got, ref)
    n = len(_base[0][4])
    assert np.array_equal(mask[:n], _base[0][4]) and not mask[n:].any()
