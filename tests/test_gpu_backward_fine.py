"""The backward pass on meshes with fewer than 8 links per triangle, whose runs
are of 256 or 512 links: nearly every link has a triangle of its own, and a
round has more vertices than its table holds.  Against the formula in float64,
with the tolerance of the other table tests."""
import numpy as np
import pytest

from test_gpu_backward_tables import test_against_the_formula as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n,tris", [(256, 33), (257, 400000), (511, 400000), (524288, 400000), (524289, 400000),
                                    (600001, 80000), (600001, 60000)])
def test_fine_meshes(n, tris, dtype):
    check(n, tris, dtype)
