"""Ghost cells formed by the reconstruction as it loads them, on small launches,
against those of the ghost-fill kernel (which runs while its time is recorded):
every rule on every side, corners of two rules, grids no wider than the halo,
inflow states, profiles and stage profiles, and a limited cell at the edge.
Both read the same cells, so every comparison is exact."""

import ctypes
import itertools

import numpy as np
import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import hweno, workloads  # noqa: E402

pytestmark = pytest.mark.gpu

IN = {0: (1.1, 0.6, 0.1, 1.2), 1: (0.9, 0.4, -0.1, 0.9), 2: (1.2, 0.5, 0.2, 1.1),
      3: (0.8, 0.5, -0.2, 0.8)}
KINDS = ('outflow', 'inflow', 'slip', 'noslip')
# every pair of kinds meets at a corner, every kind on every side
BCS = [('periodic',) * 4] + [(a, b, c, d) for (a, b), (c, d) in
                             zip(itertools.product(KINDS, KINDS),
                                 itertools.product(KINDS[1:] + KINDS[:1], KINDS))]
BCS += [('periodic', 'periodic', 'slip', 'inflow'), ('outflow', 'noslip', 'periodic', 'periodic')]


def steps(s, U, timed, staged):
    s.set_timing(timed, classes=['ghost']) if timed else s.set_timing(False)
    R, V, d = s.residual(U)
    s.set_state(U)
    out = [R, V, torch.tensor([d['alpha_star'], d['beta_max'], float(d['pp_cells'])])]
    for _ in range(2):
        q = s.rk_step_inflow(staged) if staged else s.rk_step(0.0)
        out += [s.get_state()[0], torch.tensor([q['dt'], q['min_rho'], q['min_p'],
                                                float(q['pp_cells'])])]
    n = s.timing(reset=True)['ghost'][1] if timed else 0
    return out, n


def compare(s, U, staged=0.0):
    a, n = steps(s, U, True, staged)
    b, _ = steps(s, U, False, staged)
    assert n == 7   # the fill ran as a kernel
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert all(bool(torch.isfinite(x).all()) for x in a)


@pytest.mark.parametrize('bc', BCS)
def test_ghost_variants_same_bits(bc):
    for nx, ny in ((4, 4), (5, 7), (31, 6), (37, 29)):
        print('ghost variants %dx%d %s' % (nx, ny, bc), flush=True)
        U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=nx, noise=1e-3)).cuda()
        # a low-density cell in the corner: the limiter acts there and beside it
        U[:, :, 0, 0] = 0.0
        U[0, 0, 0, 0], U[0, 3, 0, 0] = 1e-3, 2e-3
        s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=bc,
                         inflow={k: IN[k] for k in range(4) if bc[k] == 'inflow'})
        compare(s, U)


@pytest.mark.parametrize('recon', [16, 32])
def test_inflow_profiles(recon):
    nx, ny = 21, 18
    U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=2, noise=1e-3)).cuda()
    s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('inflow', 'outflow', 'slip', 'inflow'),
                     inflow={0: IN[0], 3: IN[3]})
    s.set_tiles(recon=recon, grad=32, flux=0)

    def prof(n, k, t):
        x = np.arange(n)[:, None]
        return np.array(IN[k])[None] * (1.0 + 0.05 * np.sin(x + t))
    s.set_inflow_profile(0, prof(ny, 0, 0.0))
    s.set_inflow_profile(3, prof(nx, 3, 0.3))
    compare(s, U)
    s.set_inflow_stages(0, *[prof(ny, 0, t) for t in (0.1, 0.2, 0.15)])
    s.set_inflow_stages(3, *[prof(nx, 3, t) for t in (0.4, 0.5, 0.45)])
    compare(s, U, staged=1e-4)


@pytest.mark.parametrize('shape', [(504, 248), (504, 250), (504, 251)])
def test_line_between_the_variants(shape):
    """16 x 127 and 16 x 128 = 2048 blocks of the reconstruction, and one row of
    tiles more."""
    nx, ny = shape
    U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=5, noise=1e-3)).cuda()
    s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('noslip', 'outflow', 'slip', 'noslip'))
    compare(s, U)


def test_outputs_in_the_inputs_memory():
    """The reconstruction reads the caller's state itself: R may still be
    written over it, as the state is read before anything is written."""
    nx, ny = 37, 29
    U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=4, noise=1e-3)).cuda()
    s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('noslip', 'outflow', 'slip', 'noslip'))
    R, V, _ = s.residual(U)
    for f in (hweno.lib().hweno_residual, hweno.lib().hweno_residual_noalloc):
        W, V2 = U.clone(), torch.empty_like(V)
        p = [ctypes.c_void_p(q.data_ptr()) for q in (W, W, V2)]
        assert f(s._h, *p, None) == 0
        assert torch.equal(W, R) and torch.equal(V2, V)
