"""The adjoint's gathers with sixteen, four and one lane per grid node and
thirty-two, sixteen and one per lattice node (chosen by their number: up to
8192, 49 152 grid nodes, 4096, 24 576 lattice nodes), on uniform and graded
grids, against the oracle's complex step; and the reduced-precision reverse
sub-steps in 16 x 16 tiles (grids of more than 512 8 x 8 tiles) against the
FP64 adjoint, whose tiles are 8 x 8 at every size."""
import numpy as np
import pytest

from paper_2006_13631_amd import hlbm
from paper_2006_13631_amd.workloads import graded_nodes
from tests.test_gpu_adjoint import _compare, _gpu_derivatives, _oracle_derivatives, _random_state, _say, _weights

pytestmark = pytest.mark.gpu


def _uniform(nux, nuy, bc=0):
    return dict(nx=nux + 31, ny=nuy + 27, nux=nux, nuy=nuy, b=float(2 * (nux // 7)), tau=0.7, kc=0.2, beta=12.0,
                n_sub=5, bc=bc)


def _graded(nux, nuy):
    x, y = graded_nodes(nux, 0.5, 1.02, 1.5, fine=18.0), graded_nodes(nuy, 0.5, 1.05, 1.5)
    return dict(nx=int(x[-1] - x[0]) + 32, ny=int(y[-1] - y[0]) + 28, nux=nux, nuy=nuy, b=30.0, thickness=0.5,
                tau=0.8, kc=0.3, beta=20.0, n_sub=5, x_nodes=x, y_nodes=y)


@pytest.mark.parametrize("name,c", [("4096 nodes", _uniform(128, 32)), ("9100 nodes", _uniform(130, 70, 2)),
                                    ("51000 nodes", _uniform(300, 170)), ("graded, 9170 nodes", _graded(131, 70)),
                                    ("graded, 51170 nodes", _graded(301, 170))])
def test_adjoint_lanes(oracle, name, c):
    _say("adjoint lanes", name)
    n = 2
    f0, g0, dirs = _random_state(oracle, c, 37)
    w = _weights(n, 6)
    ref = _oracle_derivatives(oracle, c, n, w, f0, g0, dirs)
    gpu, _ = _gpu_derivatives(c, n, w, f0, g0, dirs, ckpt=2)
    _compare(gpu, ref)


@pytest.mark.parametrize("storage,tol", [(hlbm.FP32, 2e-3), (hlbm.FP16_DEV, 5e-2)])
def test_reduced_precision_large_tiles(storage, tol):
    _say("reduced precision adjoint, large tiles", storage)
    c = _uniform(272, 136)
    n = 60
    w = _weights(n, 18)
    g64, _ = _gpu_derivatives(c, n, w, ckpt=20)
    glo, _ = _gpu_derivatives(c, n, w, ckpt=20, storage=storage)
    rel = np.abs(glo - g64) / np.abs(g64)
    _say("f64", g64, "reduced", glo, "rel", rel)
    assert np.all(rel <= tol), rel
