"""Steps taken in one call, where a step's refill also writes the next one's
lattice interpolation nodes, against the same steps taken one call at a time,
where it may not: the same bits, whatever the grid's spacing, storage and
boundaries, and also when the state is read or replaced in between."""
import numpy as np
import pytest

from paper_2006_13631_amd import hlbm
from paper_2006_13631_amd.workloads import graded_nodes, preset

pytestmark = pytest.mark.gpu


def _cfg(name):
    if name == "graded":
        return dict(nx=160, ny=96, nux=41, nuy=20, b=14.0, tau=0.7, kc=0.7, beta=40.0,
                    x_nodes=graded_nodes(41, 1.0, 1.05, 2.0, 8.0), y_nodes=graded_nodes(20, 1.0, 1.06, 2.0, 3.0))
    c = preset("tiny_fine_grid" if name == "fine" else "tiny_ragged")
    c.pop("steps")
    if name == "paper_bc":
        c.update(bc=hlbm.BC_PAPER)
    if name == "large":  # the two-step path with a grid of several tiles
        c.update(nx=190, ny=141, nux=97, nuy=46, b=30.0, beta=60.0)
    return c


@pytest.mark.parametrize("storage", ["f64", "f32", "f16dev"])
@pytest.mark.parametrize("name", ["ragged", "paper_bc", "fine", "graded", "large"])
def test_steps_in_one_call_equal_single_calls(name, storage):
    c = _cfg(name)
    n = 21
    a = hlbm.Case(max_steps=n, storage=storage, **c)
    b = hlbm.Case(max_steps=n, storage=storage, **c)
    a.step(11)
    for _ in range(11):
        b.step(1)
    # a read between the calls sees no interpolation nodes of the next step
    assert np.array_equal(a.lattice(), b.lattice())
    f = b.lattice()
    f[:, 2:9, 3:11] *= 1.001
    a.set_lattice(f)
    b.set_lattice(f)
    a.step(10)
    for _ in range(5):
        b.step(2)
    assert np.array_equal(a.history(), b.history())
    assert np.array_equal(a.grid(), b.grid())
    assert np.array_equal(a.lattice(), b.lattice())
    ia, ib = a.info(), b.info()
    assert (ia.n_type1, ia.n_type2, ia.n_type3) == (ib.n_type1, ib.n_type2, ib.n_type3)
