"""Totals of the event timer over more launches than its pool holds (1024): every
call that waits for its result reads the events, so none is dropped."""

import numpy as np
import pytest

torch = pytest.importorskip('torch')

from paper_2608_10569_amd import hweno, workloads  # noqa: E402

pytestmark = pytest.mark.gpu

CALLS = 1100


def launches(s, cls):
    ms, n = s.timing(reset=True)[cls]
    assert ms > 0.0
    return n


@pytest.mark.parametrize('dim', [1, 2])
def test_every_launch_is_counted(dim):
    if dim == 1:
        s = hweno.Solver(16, extent=(0.0, 2.0 * np.pi), mu_ref=0.01)
        U, cls = workloads.smooth_wave_1d(16), 'fluxup'
    else:
        s = hweno.Solver(8, 8, mu_ref=0.01)
        U, cls = workloads.random_smooth_2d(8, 8, seed=3), 'recon'
    U = torch.from_numpy(U).cuda()
    s.set_timing(True, classes=[cls])
    s.set_state(U)
    for _ in range(CALLS // 3 + 1):      # three stages a step
        assert s.rk_step(1e-6)['restarts'] == 0
    assert launches(s, cls) == 3 * (CALLS // 3 + 1)
    for _ in range(CALLS):
        s.residual(U)
    assert launches(s, cls) == CALLS


def test_every_launch_of_an_adjoint_is_counted():
    s = hweno.Solver(8, 8, mu_ref=0.01)
    U = torch.from_numpy(workloads.random_smooth_2d(8, 8, seed=3)).cuda()
    s.set_timing(True, classes=['recon'])
    for _ in range(CALLS):
        s.residual_vjp(U, U)
    assert launches(s, 'recon') == CALLS
