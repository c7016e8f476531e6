"""Residual adjoint at the edges of its tiles of 16 x 4 cells on the ghosted grid:
the ghosted width one short of, at and past a multiple of 16, heights of every
remainder and
the smallest grid.  Oracle and bound are those of
the dot-product test (double rounding of a sum over the grid)."""

import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import workloads  # noqa: E402
from test_gpu_vjp import dot_test, rel  # noqa: E402

pytestmark = pytest.mark.gpu

WALLS = ('outflow', 'slip', 'noslip', 'outflow')


@pytest.mark.parametrize('bc', [('periodic',) * 4, WALLS])
@pytest.mark.parametrize('nx,ny', [(4, 4), (23, 5), (24, 4), (25, 7), (26, 6), (57, 5), (8, 33)])
def test_dot_product_at_tile_edges(nx, ny, bc):
    U = workloads.random_smooth_2d(nx, ny, seed=21, noise=1e-3)
    lhs, rhs, mref, mub, _ = dot_test(U, bc, seed=nx + ny, mu=0.02)
    print('%dx%d: rel %.2e mu rel %.2e' % (nx, ny, rel(lhs, rhs), rel(mref, mub)))
    assert rel(lhs, rhs) < 1e-10
    assert rel(mref, mub) < 1e-10

