"""Grids with enough large tiles (more than 160 of 24 x 16 nodes, 320 of 32 x
16) that schedules 3 and 0 run them, ending inside, at and past a tile's edge;
with fewer they stand for smaller tiles. Single cases against variant 4
(several nodes per lane), a batch against the same cases alone: the same bits,
with a last launch of fewer sub-steps than the others. And the benchmark-size
comparison with the oracle with one sub-step per launch (variant 8)."""
import numpy as np
import pytest

from paper_2006_13631_amd import hlbm
from paper_2006_13631_amd.workloads import random_populations
from tests.test_gpu_parity import test_full_size_in_benchmark_configuration as full_size

pytestmark = pytest.mark.gpu
W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


def _config(nux, nuy):
    return dict(nx=nux + 30, ny=nuy + 26, nux=nux, nuy=nuy, b=float(2 * (nux // 6)), tau=0.75, kc=0.3, beta=20.0,
                n_sub=6, max_steps=2)


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("nux,nuy", [(337, 180), (336, 176), (641, 260), (640, 272)])
def test_large_tiles(nux, nuy, storage):
    ref = None
    for v in (4, 3, 0, 9, -1):
        s = hlbm.Case(storage=storage, **_config(nux, nuy))
        s.set_grid(random_populations((9, s.nnode), 7, W9))
        s.tune(variant=v)
        s.step(2)
        got = (s.grid(), s.history())
        s.close()
        if ref is None:
            ref = got
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), v


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("ncases,variant", [(2, -1), (2, 3), (2, 0), (20, -1), (20, 3), (20, 0)])
def test_batch_tiles(ncases, variant, storage):
    cfgs = [_config(170 + i % 3, 40) for i in range(ncases)]
    b = hlbm.Batch(cfgs, storage=storage)
    if variant >= 0:
        b.tune(schedule=dict(substep_variant=variant))
    for m in b.cases:
        m.set_grid(random_populations((9, m.nnode), 7, W9))
    b.step(2)
    for i in (0, 1, ncases - 1):
        s = hlbm.Case(storage=storage, **cfgs[i])
        s.set_grid(random_populations((9, s.nnode), 7, W9))
        s.tune(variant=4)
        s.step(2)
        assert np.array_equal(b[i].grid(), s.grid()) and np.array_equal(b[i].history(), s.history()), i
        s.close()
    b.close()


def test_one_substep_per_launch_at_full_size(oracle):
    full_size(oracle, "lamina_4096", 26, dict(variant=8, lattice=(256, 1), order=2))
