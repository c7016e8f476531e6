"""Weak moments formed inside the gradient kernel (every forward launch) against the
kernel of their own that a recorded step runs, where the fields are rough: shocks,
the positivity limiter acting, walls inside the grid, periodic and inflow sides, on
tiles ragged in x, in y or both and on both sides of the line between the gradient
kernel's tiles.  The arithmetic is the same, so every comparison is exact."""

import numpy as np
import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import hweno, workloads  # noqa: E402

pytestmark = pytest.mark.gpu


def compare(s, U, nsteps):
    """Steps of s from U, each against the recorded step of the same size; the
    limiter's cells and the restarts on the way."""
    s.set_record(1)
    s.set_state(U)
    pp = restarts = 0
    for _ in range(nsteps):
        d = s.rk_step(0.0)
        a = s.get_state()[0]
        assert bool(torch.isfinite(a).all())
        for grad in (32, 64):
            s.set_tiles(recon=32, grad=grad, flux=0)
            assert torch.equal(s.rk_step_record(0, U, d['dt']), a)
        U, pp, restarts = a, pp + d['pp_cells'], restarts + d['restarts']
    return pp, restarts


def dev(U):
    return torch.from_numpy(np.ascontiguousarray(U)).cuda()


@pytest.mark.parametrize('shape', [(4, 4), (33, 9), (37, 13), (64, 16), (100, 41)])
@pytest.mark.parametrize('mu_exp', [0.0, 0.7])
def test_periodic(shape, mu_exp):
    nx, ny = shape
    print('periodic %dx%d' % shape, flush=True)
    s = hweno.Solver(nx, ny, mu_ref=0.01, mu_exp=mu_exp, T_ref=1.0 / 1.4)
    compare(s, dev(workloads.random_smooth_2d(nx, ny, seed=nx * 7 + ny, noise=1e-3)), 2)


# (1534 + 2) x (127 + 2) cells are more than 6144 blocks of 16 x 2
@pytest.mark.parametrize('shape', [(120, 60), (1534, 127)])
def test_shock_tube(shape):
    nx, ny = shape
    print('shock tube %dx%d' % shape, flush=True)
    s = hweno.Solver(nx, ny, extent=(0.0, 1.0, 0.0, 0.5), mu_ref=1.0 / 200.0, bc=('noslip',) * 4)
    compare(s, dev(workloads.viscous_shock_tube_2d(nx, ny, seed=5, amp=0.02)), 2)


@pytest.mark.parametrize('n', [40, 45])
def test_sedov_start(n):
    """The limiter acts and the first steps restart."""
    print('Sedov %d' % n, flush=True)
    s = hweno.Solver(n, n, extent=(0.0, 1.1, 0.0, 1.1), bc=('slip', 'outflow', 'slip', 'outflow'),
                     gamma=1.4, Pr=0.72, mu_ref=1e-4)
    pp, restarts = compare(s, dev(workloads.sedov_2d(n)), 4)
    assert pp > 0 and restarts > 0


def test_limited_cells_in_every_tile_place():
    """Near-vacuum cells spread over the tiles, so that limited traces enter the
    weak moments of tile edges and corners too."""
    nx, ny = 61, 35
    U = workloads.random_smooth_2d(nx, ny, seed=9, noise=1e-3)
    for k, (j, i) in enumerate([(0, 0), (3, 8), (4, 7), (9, 31), (10, 32), (17, 16), (34, 60)]):
        U[:, :, j, i] = 0.0
        U[0, 0, j, i], U[0, 3, j, i] = 1e-3 * (1 + k), 2e-3
    s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('inflow', 'outflow', 'slip', 'noslip'),
                     inflow={0: (1.1, 0.6, 0.1, 1.2)})
    pp, _ = compare(s, dev(U), 2)
    assert pp > 0


@pytest.mark.parametrize('wall', ['slip', 'noslip'])
def test_masked_domain(wall):
    nx, ny = 45, 27
    solid = np.zeros((ny, nx), bool)
    solid[9:17, 20:31] = True
    s = hweno.Solver(nx, ny, mu_ref=0.01, bc=('outflow',) * 4)
    s.set_solid(solid, wall)
    compare(s, dev(workloads.random_smooth_2d(nx, ny, seed=77, noise=1e-3)), 3)
