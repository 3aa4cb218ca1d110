"""The 2D cut links with few and many candidate edges per block: a lane per
link while the edges of a chunk of 64 take no more tests in a row than the
block's links, else a lane per edge, and both in one block where the last chunk
is short.  Polygons from 4 edges over the whole grid to 20,000 edges in a few
blocks, against the 2D oracle."""
import numpy as np
import pytest

import oracle
from synth import configs, polygons
from gpu_helpers import say
from test_gpu_2d import _compare, _gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lf", [0, 2])
@pytest.mark.parametrize("edges", [4, 24, 200, 500, 1000, 4000, 20000])
def test_against_the_oracle(edges, lf):
    if edges == 4:  # faces through cell centres: hits at both ends of links, and ties at the corners
        poly = polygons.rectangle((9.5, 11.5), (52.5, 41.25))
    else:
        poly = polygons.circle(edges, (31.3, 32.1), 17.3, noise=0.2 / edges, seed=edges)
    w = configs.Workload2D("polygon", poly, (64, 64), lf)
    ref = oracle.embed2d(w.poly, w.n0, w.lf, w.d_spec)
    emb = _gpu(w)
    err = _compare(w, emb, ref)
    say(f"[2d] {edges} edges, {emb.links.n} links on level {lf}: max |dq| {err:.2e}")
