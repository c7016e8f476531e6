"""HWENO-DR kernel at the edges of its tiles (32 x 2 and 16 x 4 cells of the ghosted
grid) against the oracle, with the bounds of the other HWENO-DR comparisons; and
with the ghost cells formed in its loads against filled ones, which are the same
cells, so that comparison is exact."""

import pytest

torch = pytest.importorskip('torch')

from oracle.common import Options, Physics  # noqa: E402
from oracle.scheme2d import Scheme2D  # noqa: E402
from paper_2608_10569_amd import hweno, workloads  # noqa: E402
from test_gpu_dr import rel_err, to_dev  # noqa: E402
from test_gpu_ghost_variants import IN, compare  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize('mu_exp', [0.0, 0.76])
@pytest.mark.parametrize('recon', [16, 32])
@pytest.mark.parametrize('nx,ny', [(4, 4), (8, 9), (23, 5), (24, 4), (25, 7), (57, 5)])
def test_dr_tile_edges_match_oracle(nx, ny, recon, mu_exp):
    U = workloads.random_smooth_2d(nx, ny, seed=nx, noise=1e-3)
    bc = ('outflow', 'slip', 'noslip', 'outflow')
    kw = dict(mu_ref=0.02, mu_exp=mu_exp, Pr=0.72)
    s = hweno.Solver(nx, ny, bc=bc, gradients='DR', **kw)
    s.set_tiles(recon=recon)
    sc = Scheme2D(nx, ny, 0.0, 1.0, 0.0, 1.0, Physics(**kw), Options(gradients='DR'), bc=bc)
    R, V, d = s.residual(to_dev(U))
    Ro, Vo, do = sc.residual(U)
    eR = rel_err(R.cpu().numpy(), Ro)
    eV = rel_err(V.cpu().numpy(), Vo.reshape(8, ny, nx))
    print('DR %dx%d recon %d: R err %.2e V err %.2e' % (nx, ny, recon, eR, eV))
    assert abs(d['beta_max'] - do['beta_max']) <= 1e-12 * do['beta_max']
    assert eV < 1e-12 and eR < 1e-11


@pytest.mark.parametrize('mu_exp', [0.0, 0.76])
@pytest.mark.parametrize('bc', [('periodic',) * 4, ('outflow', 'inflow', 'slip', 'noslip'),
                                ('inflow', 'noslip', 'outflow', 'inflow')])
def test_dr_ghost_variants_same_bits(bc, mu_exp):
    for nx, ny in ((4, 4), (5, 7), (31, 6), (37, 29)):
        print('DR ghost variants %dx%d %s' % (nx, ny, bc), flush=True)
        U = torch.from_numpy(workloads.random_smooth_2d(nx, ny, seed=nx, noise=1e-3)).cuda()
        s = hweno.Solver(nx, ny, mu_ref=1e-3, mu_exp=mu_exp, bc=bc, gradients='DR',
                         inflow={k: IN[k] for k in range(4) if bc[k] == 'inflow'})
        compare(s, U)
