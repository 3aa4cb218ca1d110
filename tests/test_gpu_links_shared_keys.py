"""LINKS bins of triangles that outnumber the blocks: four rows of staged pairs
share a key's atomic, where otherwise each row takes its own.  The bins of a
triangle do not depend on the others, so those of the whole set must be the
union of the bins of parts that are no larger than the number of blocks.
Small triangles in one block, in a few and in all of them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N0, NB = (32, 32, 32), 512


def _bins(geo, V, T, first):
    coord = torch.empty((NB, 3), dtype=torch.int32, device="cuda")
    geo.geo_level0_blocks(N0, coord)
    cap = 40 * T.shape[0]
    off = torch.empty(NB + 1, dtype=torch.int32, device="cuda")
    val = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int64, device="cuda")
    bins = geo.make_bins(geo.GEO_BINS_LINKS, NB, off, val, cap, cnt)
    ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_BINS_LINKS, NB, cap), dtype=torch.uint8, device="cuda")
    geo.geo_build_bins(geo.make_mesh(V, T), geo.make_level(N0, 0, coord, []), geo.GEO_BINS_LINKS, geo.GEO_PREC_F64,
                       bins, None, ws)
    n = int(cnt.item())
    assert n <= cap
    o = off.cpu().numpy().astype(np.int64)
    assert o[0] == 0 and o[-1] == n and (np.diff(o) >= 0).all()
    v = val[:n].cpu().numpy().astype(np.int64)
    assert v.min() >= 0 and v.max() < T.shape[0]
    return np.repeat(np.arange(NB), np.diff(o)) * 2 ** 32 + v + first


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("spread", [1.5, 9.0, 27.0])
@pytest.mark.parametrize("nt", [513, 1000, 9001, 140003])
def test_whole_is_the_union_of_its_parts(nt, spread, dtype):
    import paper_2512_01251_amd as geo
    rng = np.random.default_rng(nt)
    at = 17.1 + spread / 2 * rng.uniform(-1, 1, (nt, 1, 3))
    P = (at + rng.uniform(-0.3, 0.3, (nt, 3, 3))).astype(dtype).reshape(-1, 3)
    V = torch.from_numpy(P).cuda()
    T = torch.arange(3 * nt, dtype=torch.int32, device="cuda").reshape(-1, 3)
    whole = np.sort(_bins(geo, V, T, 0))
    assert len(np.unique(whole)) == len(whole)
    step = NB if nt < 20000 else 100 * NB  # (the largest: parts that share keys too, of other sizes)
    parts = np.sort(np.concatenate([_bins(geo, V, T[f:f + step].contiguous(), f) for f in range(0, nt, step)]))
    assert np.array_equal(whole, parts)
