"""The autotuner times the kernels that a step runs: up to the line where the
reconstruction forms the ghost cells in its loads no ghost fill runs while it
measures, so the ghost cells of the state keep whatever they hold; beyond it the
fill runs."""

import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import hweno, workloads  # noqa: E402

pytestmark = pytest.mark.gpu

MARK = -7.0


def ghost_cells(workspace, nx, ny):
    """The workspace starts with the 12 ghosted planes of the (first) state."""
    NX, NY = nx + 8, ny + 8
    S = workspace[:12 * NX * NY * 8].view(torch.float64).view(12, NY, NX)
    m = torch.ones(NY, NX, dtype=torch.bool, device=S.device)
    m[4:4 + ny, 4:4 + nx] = False
    return S, m


# (340 + 8)^2 takes 11 x 173 and 22 x 87 blocks of the two tiles, 504 x 251 more
# than 2048 of either
@pytest.mark.parametrize('shape,formed', [((24, 17), True), ((340, 340), True),
                                          ((504, 251), False)])
@pytest.mark.parametrize('gradients', ['GR', 'DR'])
def test_single_grid(shape, formed, gradients):
    nx, ny = shape
    print('autotune path %dx%d %s' % (nx, ny, gradients), flush=True)
    U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=1)).cuda()
    s = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('noslip', 'outflow', 'slip', 'outflow'),
                     gradients=gradients)
    s.set_state(U)
    S, m = ghost_cells(s.workspace, nx, ny)
    S[:, m] = MARK
    tiles = s.autotune(reps=1)
    assert tiles == s.tiles()
    assert bool((S[:, m] == MARK).all()) == formed
    assert torch.equal(s.get_state()[0], U)
    # a step from there reads nothing that the autotuner left behind
    d = s.rk_step(0.0)
    r = hweno.Solver(nx, ny, mu_ref=1e-3, bc=('noslip', 'outflow', 'slip', 'outflow'),
                     gradients=gradients)
    r.set_state(U)
    assert r.rk_step(0.0) == d and torch.equal(r.get_state()[0], s.get_state()[0])


def test_batch():
    """Two grids, each a group of its own in the run: either alone is below the
    line, both together are not."""
    n = 340
    U = [torch.from_numpy(workloads.random_smooth_2d(n, n, seed=k)).cuda() for k in (1, 2)]
    b = hweno.Batch([dict(nx=n, ny=n, mu_ref=1e-3)] * 2)
    for i in range(2):
        b.set_state(i, U[i])
    S, m = ghost_cells(b.workspace, n, n)
    S[:, m] = MARK
    b.autotune(reps=1)
    assert bool((S[:, m] == MARK).all())
    for i in range(2):
        assert torch.equal(b.get_state(i)[0], U[i])
    b.run(1)
    assert bool((S[:, m] == MARK).all())   # as in the run
