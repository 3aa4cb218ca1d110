"""The children of refined blocks are placed tile by tile: a tile is one pass
of 256 blocks, several where a level has more than 2,048 x 256 blocks.  On
level 0, with one block, at the edges of a tile and with two passes per tile,
classes, marks, child maps and children must equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _words(nb, bits, dt):
    """Solid words: blocks partly solid with a probability that falls along the
    list from 0.3 (nearly every block refined) to 0 (none)."""
    rng = np.random.default_rng(nb)
    some = rng.random(nb) < 0.3 * np.maximum(1 - np.arange(nb) / (0.75 * nb), 0)
    some[0] = True
    return np.where(some, rng.integers(1, 2 ** (bits - 1), nb), 0).astype(dt)


def _check(r, nb, bclass, refine, cmap, child, d_n):
    n = int(d_n.item())
    assert n == len(r["children"])
    assert np.array_equal(bclass.cpu().numpy(), r["bclass"])
    assert np.array_equal(refine.cpu().numpy(), r["refine"])
    assert np.array_equal(cmap.cpu().numpy(), r["child_map"])
    assert np.array_equal(child[:n].cpu().numpy(), r["children"])


def _outputs(nb, d):
    return (torch.empty(nb, dtype=torch.uint8, device="cuda"), torch.empty(nb, dtype=torch.uint8, device="cuda"),
            torch.empty(nb, dtype=torch.int32, device="cuda"),
            torch.empty((2 ** d * nb, d), dtype=torch.int32, device="cuda"),
            torch.full((1,), -1, dtype=torch.int64, device="cuda"))


@pytest.mark.parametrize("n_prop", [0, 1])
@pytest.mark.parametrize("blocks", [(1, 1, 1), (255, 1, 1), (256, 1, 1), (257, 1, 1), (83, 83, 83)])
def test_children_of_a_level(blocks, n_prop):
    import paper_2512_01251_amd as geo
    n0 = tuple(4 * k for k in blocks)
    bc = oracle.level0_blocks(n0)
    nb = len(bc)
    words = _words(nb, 64, np.int64)
    cells = ((words.view(np.uint64)[:, None] >> np.arange(64, dtype=np.uint64)[None, :]) & np.uint64(1)).astype(np.uint8)
    r = oracle.refine(n0, 0, bc, cells, n_prop)
    say(f"[children] 3D {blocks}, n_prop {n_prop}: {int(r['refine'].sum())} of {nb} refined")
    dbc = torch.from_numpy(np.ascontiguousarray(bc, dtype=np.int32)).cuda()
    out = _outputs(nb, 3)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_REFINE, nb, 0), dtype=torch.uint8, device="cuda")
    geo.geo_refine_flags(geo.make_level(n0, 0, dbc, []), torch.from_numpy(words).cuda(), n_prop, *out, ws)
    torch.cuda.synchronize()
    _check(r, nb, *out)


@pytest.mark.parametrize("blocks", [(1, 1), (255, 1), (256, 1), (257, 1), (730, 731)])
def test_children_of_a_level_2d(blocks):
    import paper_2512_01251_amd as geo
    n0 = tuple(4 * k for k in blocks)
    bc = oracle.level0_blocks2d(n0)
    nb = len(bc)
    words = _words(nb, 16, np.int16)
    cells = ((words.view(np.uint16)[:, None] >> np.arange(16, dtype=np.uint16)[None, :]) & np.uint16(1)).astype(np.uint8)
    r = oracle.refine2d(n0, 0, bc, cells, 1)
    say(f"[children] 2D {blocks}: {int(r['refine'].sum())} of {nb} refined")
    dbc = torch.from_numpy(np.ascontiguousarray(bc, dtype=np.int32)).cuda()
    out = _outputs(nb, 2)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL2_REFINE, nb, 0), dtype=torch.uint8, device="cuda")
    geo.geo2_refine_flags(geo.make_level2(n0, 0, dbc, []), torch.from_numpy(words).cuda(), 1, *out, ws)
    torch.cuda.synchronize()
    _check(r, nb, *out)
