"""Every grid sub-step variant, and the one chosen by the grid's size, gives
the bits of variant 4 (several nodes per lane, lanes dealt afresh each
sub-step) on grids that end inside, at and just past the tiles' edges, with a
last launch of fewer sub-steps than the others."""
import numpy as np
import pytest

from paper_2006_13631_amd import hlbm
from paper_2006_13631_amd.workloads import random_populations

pytestmark = pytest.mark.gpu
W9 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nux,nuy", [(17, 12), (24, 16), (25, 18), (32, 16), (33, 34), (64, 16), (97, 50), (140, 40)])
def test_variants_on_tile_edges(nux, nuy, storage):
    b = float(2 * max(1, nux // 6))
    c = dict(nx=nux + 30, ny=nuy + 26, nux=nux, nuy=nuy, b=b, tau=0.75, kc=0.3, beta=20.0, n_sub=6, max_steps=3)
    ref = None
    for v in (4, -1, 0, 1, 2, 3, 8, 9, 10):
        s = hlbm.Case(storage=storage, **c)
        s.set_grid(random_populations((9, s.nnode), 7, np.array(W9)))
        s.tune(variant=v)
        s.step(3)
        got = (s.grid(), s.lattice(), s.history())
        s.close()
        if ref is None:
            ref = got
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), v
