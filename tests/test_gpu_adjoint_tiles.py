"""The reverse sub-steps in either tile (8 x 8 on small grids, 16 x 16 on
grids of more than 512 such tiles) on widths that end inside, at and past a
tile's edge, with a last launch of fewer sub-steps: dJ/d(A, omega, tau) and
the initial state's adjoint against the oracle's complex step."""
import pytest

from paper_2006_13631_amd import hlbm
from tests.test_gpu_adjoint import _compare, _gpu_derivatives, _oracle_derivatives, _random_state, _weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nux,nuy,bc", [(40, 16, 0), (41, 18, 2), (272, 136, 0), (257, 146, 0)])
def test_adjoint_tiles(oracle, nux, nuy, bc):
    c = dict(nx=nux + 31, ny=nuy + 27, nux=nux, nuy=nuy, b=float(2 * (nux // 7)), tau=0.7, kc=0.2, beta=12.0,
             n_sub=6, bc=bc)
    n = 2
    f0, g0, dirs = _random_state(oracle, c, 91)
    w = _weights(n, 5)
    ref = _oracle_derivatives(oracle, c, n, w, f0, g0, dirs)
    gpu, _ = _gpu_derivatives(c, n, w, f0, g0, dirs, ckpt=2, storage=hlbm.FP64)
    _compare(gpu, ref)
