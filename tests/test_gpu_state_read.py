"""A lattice that is set and read back without a step in between equals the
host's own rounding through the storage type (FP32; FP16 of the deviation
from the rest weights): lattices that one piece of the read holds, that take a
piece per plane, and whose planes take several pieces with a ragged last one,
for single cases and refinement levels. Values differ from node to node and
from plane to plane, so a wrong offset or a wrong plane's weight shows."""
import numpy as np
import pytest

from paper_2006_13631_amd import hlbm
from paper_2006_13631_amd.workloads import random_populations

pytestmark = pytest.mark.gpu
W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


def _stored(f, storage):
    if storage == "f64":
        return f
    f = f.astype(np.float32)
    if storage == "f32":
        return f.astype(np.float64)
    w = W9.astype(np.float32)[:, None, None]
    return ((f - w).astype(np.float16).astype(np.float32) + w).astype(np.float64)


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("nx,ny", [(131, 77), (521, 450), (2311, 1013)])
def test_lattice_read_back(nx, ny, storage):
    case = hlbm.Case(nx=nx, ny=ny, tau=0.8, storage=storage, max_steps=2)
    f = random_populations((9, ny, nx), seed=5, base=W9, spread=0.05)
    case.set_lattice(f)
    want = _stored(f, storage)
    for _ in range(2):  # the second read through the buffer the first one left
        assert np.array_equal(case.lattice(), want)
    case.close()


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
def test_level_read_back(storage):
    m = hlbm.MultiLevel(2311, 1013, [(12, 12, 48, 44)], max_steps=64, storage=storage, nux=40, nuy=24, b=10.0,
                        beta=20.0, kc=0.5, tau=0.7)
    for l in (0, 1):
        nx, ny = m.shapes[l]
        f = random_populations((9, ny, nx), seed=6 + l, base=W9, spread=0.05)
        m.set_level(l, f)
        assert np.array_equal(m.level(l), _stored(f, storage))
    m.close()
