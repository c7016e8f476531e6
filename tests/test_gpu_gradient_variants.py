"""The gradient kernel that forms the weak moments itself, at the edges of its
tiles (8 x 4 cells, 16 x 2 on large launches) and on both sides of the line
between them.  A recorded step runs the separate weak-moment and gradient
kernels of the reverse mode, whose arithmetic is the same, so every comparison
here is exact."""

import numpy as np
import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import hweno, workloads  # noqa: E402

pytestmark = pytest.mark.gpu


# the gradient region is (nx + 2) x (ny + 2): the smallest grid, whole tiles of
# both kinds, one column or row more, and 6144 blocks of 16 x 2 cells and more
@pytest.mark.parametrize('shape', [(4, 4), (6, 6), (14, 14), (15, 15), (30, 5), (31, 6), (7, 61),
                                   (1534, 126), (1534, 127), (1533, 129)])
@pytest.mark.parametrize('mu_exp', [0.0, 0.7])
def test_gradient_variants_same_bits(shape, mu_exp):
    nx, ny = shape
    print('gradient variants %dx%d mu_exp %s' % (nx, ny, mu_exp), flush=True)
    U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=nx + ny, noise=1e-3)).cuda()
    s = hweno.Solver(nx, ny, mu_ref=0.01, mu_exp=mu_exp, T_ref=1.0 / 1.4,
                     bc=('noslip', 'outflow', 'slip', 'outflow'))
    s.set_state(U)
    d = s.rk_step(0.0)
    a = s.get_state()[0]
    assert d['restarts'] == 0 and bool(torch.isfinite(a).all())
    s.set_record(1)
    for grad in (32, 64):
        s.set_tiles(recon=32, grad=grad, flux=0)
        assert torch.equal(s.rk_step_record(0, U, d['dt']), a)
    assert not np.array_equal(a.cpu().numpy(), U.cpu().numpy())
