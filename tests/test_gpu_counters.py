"""Counters of the q kernel, which its workgroups add into slots of the
workspace (2 slots for 8 blocks, 64 from 2,048 blocks on) and the call's last
kernel adds to the caller's array.  Tasks follow from the bins and the table;
the other counters must not depend on the number of slots, on earlier contents
of the array (they accumulate) or on whether a table is written."""
import numpy as np
import pytest
import torch

from synth import configs, meshes
from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu

CASES = {
    "8_blocks": lambda: configs.Workload("tiny", meshes.icosphere(2, 2.0, (4.1, 3.9, 4.2)), (8, 8, 8), 0, 27),
    "icosphere64": lambda: configs.icosphere64(),
    "star_small": lambda: configs.star_small(lf=2),
}


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("name", list(CASES))
def test_q_counters(name, precision):
    import paper_2512_01251_amd as geo
    from paper_2512_01251_amd import pipeline
    w = CASES[name]()
    V, T = to_gpu(w.mesh)
    emb = pipeline.Embedder().embed(V, T, w.n0, w.lf, w.lattice, w.d_spec, precision)
    rec, k = emb.levels[-1], emb.links
    nb = int(rec.bcoord.shape[0])
    off = k.bins_off.cpu().numpy().astype(np.int64)
    nc = off[1:] - off[:-1]
    nl = np.bincount(k.cell.cpu().numpy() // 64, minlength=nb)
    tasks = int((-(-nl // 64) * np.maximum(1, -(-nc // 64)) * (nl > 0)).sum())

    mesh = geo.make_mesh(V, T)
    lvd = geo.make_level(w.n0, w.lf, rec.bcoord, [lv.child_map for lv in emb.levels[:-1]])
    cnt = torch.tensor([rec.rows_val.numel(), k.bins_val.numel()], dtype=torch.int64, device="cuda")
    nk = (w.n0[1] << w.lf) * (w.n0[2] << w.lf)
    rows = geo.make_bins(geo.GEO_BINS_ROWS, nk, rec.rows_off, rec.rows_val, rec.rows_val.numel(), cnt[:1])
    links = geo.make_bins(geo.GEO_BINS_LINKS, nb, k.bins_off, k.bins_val, k.bins_val.numel(), cnt[1:])
    prec = pipeline.PRECISIONS[precision]
    d_n = torch.zeros(1, dtype=torch.int64, device="cuda")

    def call(stats, cap):
        ws = torch.empty(geo.geo_workspace_size(geo.GEO_CALL_CUTLINKS, nb, cap), dtype=torch.uint8, device="cuda")
        o = [torch.empty(max(cap, 1), dtype=t, device="cuda") for t in (torch.int32, torch.uint8, torch.float32,
                                                                       torch.int32)]
        geo.geo_cutlinks(mesh, lvd, rows, links, w.lattice, prec, None, cap, d_n, *o, stats, ws)
        torch.cuda.synchronize()
        assert int(d_n.item()) == k.n
        return o

    stats = torch.zeros(geo.GEO_NSTATS, dtype=torch.int64, device="cuda")
    call(stats, k.n)
    one = stats.cpu().numpy()
    assert one[geo.GEO_STAT_TASKS] == tasks
    assert one[geo.GEO_STAT_STAGED] > 0 and one[geo.GEO_STAT_PAIRS] > 0
    call(stats, k.n)
    assert np.array_equal(stats.cpu().numpy(), 2 * one)
    none = torch.zeros_like(stats)
    call(none, 0)  # counting only: no table, no exact pass
    none = none.cpu().numpy()
    for s in (geo.GEO_STAT_TASKS, geo.GEO_STAT_STAGED, geo.GEO_STAT_PAIRS, geo.GEO_STAT_F32_TO_F64):
        assert none[s] == one[s]
    q = call(None, k.n)[2]
    assert torch.equal(q, k.q)


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n_theta", [4, 12, 40, 160])
def test_groups_of_blocks_and_chunks(n_theta, dtype, precision):
    """Candidates staged for several blocks at once and for blocks with more
    than 64 (the poles of the finer meshes), against the oracle: from a few
    candidates per block, where a group spans 64 blocks, to hundreds."""
    import oracle
    from gpu_helpers import compare, gpu_embed
    w = configs.star_small(n_theta=n_theta, n_phi=2 * n_theta, lf=1, lattice=27, dtype=dtype)
    ref = oracle.embed(w.mesh, w.n0, w.lf, w.lattice, w.d_spec)
    emb, _, _ = gpu_embed(w, precision)
    compare(w, emb, ref)
    nc = np.diff(emb.links.bins_off.cpu().numpy())
    assert nc.max() > 64 if n_theta >= 40 else nc.max() < 64
