"""Performance cases of the library: the work its users have it do, through the
public entry points of the Python binding, and a plain float64 torch model of
the same scheme that gives each case's expected outputs.

A case is a dict of plain values.  ``kind`` names the entry points:

* ``steps1d``: a 1D run, ``set_state``, ``steps`` x ``rk_step`` with the
  paper's time-step rule, ``get_state``;
* ``steps2d``: the same on a 2D grid (walls, masked domain, forced inflow with
  ``set_inflow_stages`` / ``rk_step_inflow``, HWENO-GR or the comparison scheme
  HWENO-DR, constant or temperature-dependent viscosity, by ``flow`` and the
  other entries);
* ``residual``: one residual evaluation, ``residual`` or ``residual_noalloc``;
* ``batch``: ``Batch``: every state set, one ``run`` of ``steps`` steps, every
  state fetched;
* ``vjp``: the adjoint of the residual, ``residual_vjp``;
* ``rollout``: ``adjoint.rollout`` forward and backward through
  ``torch.autograd``.

Grids, boundary conditions and physics are those of ``workloads.py``, the
tests and ``bench.py``; the fields carry seeded perturbations.
"""

import math

import numpy as np
import torch

from paper_2608_10569_amd import adjoint, hweno

HALO = 4


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest calls: the smooth-wave accuracy run on 200 cells, where
        # a step is a chain of launches over a few hundred threads
        dict(name='wave1d_200', kind='steps1d', flow='wave', nx=200, steps=10, gradients='GR'),
        # an ordinary 1D run: Sod's Riemann problem on 2000 cells
        dict(name='sod1d_2000', kind='steps1d', flow='riemann', nx=2000, steps=10,
             gradients='GR'),
        # a small 2D run: one periodic grid of the 64^2 class on its own
        dict(name='smooth_64', kind='steps2d', flow='smooth', nx=64, ny=64, steps=10,
             gradients='GR', mu_exp=0.0),
        # one residual of a small odd-sized walled grid for a caller's own time
        # stepper, mu(T), with the library's static buffer (serving loops)
        dict(name='residual_97x61', kind='residual', flow='walls', nx=97, ny=61, mu_exp=0.76,
             noalloc=True),
        # walls inside the grid: the shock diffraction around a step, 104x88
        dict(name='diffraction_104x88', kind='steps2d', flow='diffraction', nx=104, ny=88,
             steps=5, gradients='GR', mu_exp=0.0),
        # inflow data that vary in time: the forced shock-mixing layer, 500x100
        dict(name='layer_500x100', kind='steps2d', flow='layer', nx=500, ny=100, steps=3,
             gradients='GR', mu_exp=0.0),
        # the headline run: the viscous shock tube on 1000x500
        dict(name='tube_1000x500', kind='steps2d', flow='tube', nx=1000, ny=500, steps=3,
             gradients='GR', mu_exp=0.0),
        # the comparison scheme on a mid-size grid of the same flow
        dict(name='tube_dr_500x250', kind='steps2d', flow='tube', nx=500, ny=250, steps=4,
             gradients='DR', mu_exp=0.0),
        # one residual of a large grid
        dict(name='residual_2048x1024', kind='residual', flow='smooth', nx=2048, ny=1024,
             mu_exp=0.0, noalloc=False),
        # many grids of mixed sizes and viscosities in one graph launch
        dict(name='batch_12', kind='batch', count=12, largest=512, steps=6),
        # reverse mode of one residual (an outer solver's adjoint), 256^2
        dict(name='vjp_256', kind='vjp', flow='smooth', nx=256, ny=256, mu_exp=0.0),
        # a differentiable rollout of the shear layer, forward and backward,
        # with the steps of the backward recorded in two banks
        dict(name='rollout_256', kind='rollout', nx=256, ny=256, steps=12, every=6,
             record=True),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges."""
    kind = rng.choice(['steps1d', 'steps1d', 'steps2d', 'steps2d', 'steps2d', 'steps2d',
                       'residual', 'residual', 'batch', 'vjp', 'vjp', 'rollout'])
    if kind == 'steps1d':
        return dict(kind=kind, flow=rng.choice(['wave', 'riemann']), nx=_logint(rng, 40, 20000),
                    steps=rng.randint(4, 12), gradients=rng.choice(['GR', 'GR', 'DR']))
    if kind == 'steps2d':
        flow = rng.choice(['smooth', 'walls', 'tube', 'diffraction', 'layer'])
        if flow == 'diffraction':      # square cells of size 1/m
            m = rng.randint(4, 24)
            nx, ny = 13 * m, 11 * m
        else:
            nx, ny = _logint(rng, 32, 1000), _logint(rng, 32, 500)
        return dict(kind=kind, flow=flow, nx=nx, ny=ny, steps=rng.randint(2, 8),
                    gradients=rng.choice(['GR', 'GR', 'DR']),
                    mu_exp=rng.choice([0.0, 0.0, 0.76]))
    if kind == 'residual':
        noalloc = rng.random() < 0.5
        top = 360 if noalloc else 1400
        return dict(kind=kind, flow=rng.choice(['smooth', 'walls']), nx=_logint(rng, 32, top),
                    ny=_logint(rng, 32, top), mu_exp=rng.choice([0.0, 0.0, 0.76]),
                    noalloc=noalloc)
    if kind == 'batch':
        return dict(kind=kind, count=rng.randint(2, 12), largest=rng.choice([128, 256, 512]),
                    steps=rng.randint(2, 6))
    if kind == 'vjp':
        return dict(kind=kind, flow=rng.choice(['smooth', 'walls']), nx=_logint(rng, 32, 256),
                    ny=_logint(rng, 32, 256), mu_exp=rng.choice([0.0, 0.0, 0.76]))
    every = rng.randint(2, 6)
    return dict(kind=kind, nx=_logint(rng, 48, 256), ny=_logint(rng, 48, 256),
                steps=rng.randint(4, 12), every=every, record=rng.random() < 0.7)


def _setup(case):
    """Problem statement of a case: extent, boundary kinds and physics."""
    kind, flow = case['kind'], case.get('flow')
    p = dict(gamma=1.4, Pr=0.72, mu_ref=1e-2, mu_exp=case.get('mu_exp', 0.0), cfl=0.6)
    extent, bc = (0.0, 1.0, 0.0, 1.0), ('periodic',) * 4
    if kind == 'steps1d':
        if flow == 'wave':
            extent, bc = (0.0, 2.0 * math.pi), ('periodic', 'periodic')
            p.update(cfl=0.3)
        else:
            extent, bc = (0.0, 1.0), ('outflow', 'outflow')
            p.update(mu_ref=1e-3, cfl=0.3)
    elif kind == 'rollout':
        p.update(mu_ref=1e-3)
    elif flow == 'walls':
        bc = ('noslip', 'outflow', 'slip', 'noslip')
    elif flow == 'tube':
        extent, bc = (0.0, 1.0, 0.0, 0.5), ('noslip', 'noslip', 'noslip', 'slip')
        p.update(Pr=0.73, mu_ref=1.0 / 200.0, cfl=0.3)
    elif flow == 'diffraction':
        extent, bc = (0.0, 13.0, 0.0, 11.0), ('inflow', 'outflow', 'outflow', 'outflow')
        p.update(mu_ref=1e-3)
    elif flow == 'layer':
        extent, bc = (0.0, 200.0, -20.0, 20.0), ('inflow', 'outflow', 'slip', 'inflow')
        p.update(mu_ref=1.0 / 500.0)
    return extent, bc, p


LAYER_TOP = (2.1101, 2.9709, -0.1367, 0.4754)


def _post_shock():
    """State behind the Mach-5.09 shock moving into (1.4, 0, 0, 1)."""
    g, m2 = 1.4, 5.09 * 5.09
    r2 = 1.4 * (g + 1.0) * m2 / ((g - 1.0) * m2 + 2.0)
    return (r2, 5.09 * (1.0 - 1.4 / r2), 0.0, (2.0 * g * m2 - (g - 1.0)) / (g + 1.0))


def _solid(nx, ny):
    """Solid cells of the diffraction grid: the step [0,1]x[0,6]."""
    X, Y = np.meshgrid((np.arange(nx) + 0.5) * 13.0 / nx, (np.arange(ny) + 0.5) * 11.0 / ny)
    return (X < 1.0) & (Y < 6.0)


# ---------------------------------------------------------------------------
# Seeded initial data, projected onto averages and first moments
# ---------------------------------------------------------------------------
def _project(prim, nx, ny, extent, gamma, dev):
    """(3, 4, ny, nx) from prim(X, Y) -> (rho, u, v, p), 6-point Gauss rule."""
    gx, gw = np.polynomial.legendre.leggauss(6)
    gx, gw = 0.5 * gx, 0.5 * gw
    x0, x1, y0, y1 = extent
    dx, dy = (x1 - x0) / nx, (y1 - y0) / ny
    xc = x0 + (torch.arange(nx, dtype=torch.float64, device=dev) + 0.5) * dx
    yc = y0 + (torch.arange(ny, dtype=torch.float64, device=dev) + 0.5) * dy
    U = torch.zeros(3, 4, ny, nx, dtype=torch.float64, device=dev)
    for b in range(6):
        for a in range(6):
            X = (xc + gx[a] * dx)[None, :].expand(ny, nx)
            Y = (yc + gx[b] * dy)[:, None].expand(ny, nx)
            r, u, v, p = prim(X, Y)
            Q = torch.stack([r, r * u, r * v, p / (gamma - 1.0) + 0.5 * r * (u * u + v * v)])
            w = gw[a] * gw[b]
            U[0] += w * Q
            U[1] += w * gx[a] * Q
            U[2] += w * gx[b] * Q
    return U


def _modes(rng, n, amp, kmax=3):
    """n random Fourier modes: f(x, y) of about the given amplitude."""
    kx, ky = rng.integers(-kmax, kmax + 1, n), rng.integers(-kmax, kmax + 1, n)
    a, ph = rng.uniform(-1.0, 1.0, n) * amp, rng.uniform(0.0, 2.0 * math.pi, n)

    def f(x, y):
        out = 0.0
        for q in range(n):
            out = out + float(a[q]) * torch.sin(2.0 * math.pi * (int(kx[q]) * x + int(ky[q]) * y)
                                                + float(ph[q]))
        return out
    return f


def _noise(U, seed, amp):
    """Cell-level noise on the first moments (what a developed flow has)."""
    g = torch.Generator(device=U.device)
    g.manual_seed(seed)
    U[1:] += amp * torch.randn(U[1:].shape, dtype=torch.float64, device=U.device, generator=g)
    return U


def _state2d(case, seed, dev):
    extent, _, p = _setup(case)
    nx, ny, flow, gamma = case['nx'], case['ny'], case.get('flow', 'shear'), p['gamma']
    rng = np.random.default_rng([2608, seed])
    x0, x1, y0, y1 = extent

    def unit(X, Y):
        return (X - x0) / (x1 - x0), (Y - y0) / (y1 - y0)
    if flow in ('smooth', 'walls'):
        f = [_modes(rng, 4, a) for a in (0.1, 0.15, 0.15, 0.1)]

        def prim(X, Y):
            x, y = unit(X, Y)
            return 1.0 + f[0](x, y), 0.3 + f[1](x, y), -0.2 + f[2](x, y), 1.0 / gamma + f[3](x, y)
    elif flow == 'tube':
        f = [_modes(rng, 3, 0.02, 5) for _ in range(4)]

        def prim(X, Y):
            x, y = unit(X, Y)
            r = torch.where(X < 0.5, 120.0, 1.2).to(torch.float64)
            return r * (1.0 + f[0](x, y)), f[1](x, y), f[2](x, y), r / gamma * (1.0 + f[3](x, y))
    elif flow == 'diffraction':
        f = [_modes(rng, 3, 0.01) for _ in range(2)]
        post = _post_shock()

        def prim(X, Y):
            x, y = unit(X, Y)
            left = (X < 0.5) & (Y > 6.0)
            q = [torch.where(left, a, b).to(torch.float64) for a, b in
                 zip(post, (1.4, 0.0, 0.0, 1.0))]
            return q[0] * (1.0 + f[0](x, y)), q[1], q[2], q[3] * (1.0 + f[1](x, y))
    elif flow == 'layer':
        f = _modes(rng, 3, 0.02)

        def prim(X, Y):
            x, y = unit(X, Y)
            r = torch.where(Y > 0.0, 1.6374, 0.3626).to(torch.float64)
            return (r, 2.5 + 0.5 * torch.tanh(2.0 * Y), f(x, y) * torch.exp(-Y * Y / 10.0),
                    torch.full_like(Y, 0.3327))
    else:   # the double shear layer
        f = [_modes(rng, 3, 0.02) for _ in range(3)]

        def prim(X, Y):
            u = torch.where(Y <= 0.5, torch.tanh(80.0 * (Y - 0.25)), torch.tanh(80.0 * (0.75 - Y)))
            return (1.0 + f[0](X, Y), u, 0.05 * torch.sin(2.0 * math.pi * X) + f[1](X, Y),
                    1.0 / gamma + f[2](X, Y))
    U = _project(prim, nx, ny, extent, gamma, dev)
    if flow in ('smooth', 'walls'):
        _noise(U, seed, 1e-4)
    elif flow is not None and flow != 'diffraction':
        _noise(U, seed, 1e-6)
    return U.contiguous()


def _state1d(case, seed, dev):
    (x0, x1), _, p = _setup(case)
    nx, gamma = case['nx'], p['gamma']
    rng = np.random.default_rng([2608, 1, seed])
    gx, gw = np.polynomial.legendre.leggauss(6)
    gx, gw = 0.5 * gx, 0.5 * gw
    dx = (x1 - x0) / nx
    X = x0 + (np.arange(nx) + 0.5) * dx + gx[:, None] * dx
    if case['flow'] == 'wave':
        k, ph = np.arange(1, 9), rng.uniform(0.0, 2.0 * math.pi, (3, 8))
        a = rng.standard_normal((3, 8)) * 1e-2 / k
        f = [sum(a[q, m] * np.sin(k[m] * X + ph[q, m]) for m in range(8)) for q in range(3)]
        r, u, pr = 1.0 + 0.2 * np.sin(X) + f[0], 1.0 + f[1], 1.0 + f[2]
    else:
        s = 1.0 + 0.1 * rng.uniform(-1.0, 1.0, 4)
        left = X < 0.5
        r = np.where(left, s[0], 0.125 * s[1])
        u = 0.02 * np.sin(2.0 * math.pi * X + rng.uniform(0.0, 2.0 * math.pi))
        pr = np.where(left, s[2], 0.1 * s[3])
    Q = np.stack([r, r * u, pr / (gamma - 1.0) + 0.5 * r * u * u])
    U = np.stack([np.einsum('g,cgi->ci', gw, Q), np.einsum('g,cgi->ci', gw * gx, Q)])
    return torch.from_numpy(np.ascontiguousarray(U)).to(dev)


def _batch_problems(case):
    """(n, Re) of the instances: sizes 64, 128, 256, 512 in turn up to the
    largest, Reynolds numbers log-uniform in [1e2, 1e4]."""
    sizes = [n for n in (64, 128, 256, 512) if n <= case['largest']]
    res = np.random.default_rng([2608, case['count']]).uniform(2.0, 4.0, case['count'])
    return [(sizes[k % len(sizes)], float(10.0 ** res[k])) for k in range(case['count'])]


def _batch_state(n, k, seed, dev):
    rng = np.random.default_rng([2608, 2, k, seed])
    f = [_modes(rng, 8, 0.1, 4) for _ in range(2)]

    def prim(X, Y):
        return torch.ones_like(X), f[0](X, Y), f[1](X, Y), torch.full_like(X, 1.0 / 1.4)
    return _project(prim, n, n, (0.0, 1.0, 0.0, 1.0), 1.4, dev).contiguous()


def _layer_inflow(case, seed):
    """Left-side profile (ny, 4) of the forced mixing layer as a function of t."""
    rng = np.random.default_rng([2608, 3, seed])
    ph = rng.uniform(0.0, 2.0 * math.pi, 2)
    ny = case['ny']
    y = -20.0 + (np.arange(ny) + 0.5) * (40.0 / ny)

    def at(t):
        v = sum(0.05 * np.cos(2.0 * np.pi * k * t * 2.68 / 30.0 + ph[k - 1]) * np.exp(-y * y / 10.0)
                for k in (1, 2))
        return np.column_stack([np.where(y > 0.0, 1.6374, 0.3626), 2.5 + 0.5 * np.tanh(2.0 * y), v,
                                np.full_like(y, 0.3327)])
    return at


def _layer_dt(case):
    """A fixed step within the paper's rule (wave speeds up to about 4.5)."""
    h = min(200.0 / case['nx'], 40.0 / case['ny'])
    return min(0.1 * h, 0.001 * h * h * 500.0)


def _rollout_dt(case):
    return 0.15 / max(case['nx'], case['ny'])


def _seeds_vjp(case, seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 77)
    nx, ny = case['nx'], case['ny']
    return [torch.randn(s, dtype=torch.float64, device=dev, generator=g)
            for s in ((3, 4, ny, nx), (8, ny, nx))]


# ---------------------------------------------------------------------------
# What a user's program holds, and one pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind, dev = case['kind'], 'cuda'
    st = dict(case=case)
    if kind == 'batch':
        probs = _batch_problems(case)
        st['b'] = hweno.Batch([dict(nx=n, ny=n, mu_ref=1.0 / Re) for n, Re in probs])
        st['U'] = [_batch_state(n, k, seed, dev) for k, (n, _) in enumerate(probs)]
        return st
    extent, bc, p = _setup(case)
    kw = dict(extent=extent, bc=bc, **p)
    if kind == 'steps1d':
        st['U'] = _state1d(case, seed, dev)
        st['s'] = hweno.Solver(case['nx'], gradients=case['gradients'], **kw)
        return st
    nx, ny = case['nx'], case['ny']
    st['U'] = _state2d(case, seed, dev)
    if case.get('flow') == 'layer':
        kw['inflow'] = {0: LAYER_TOP, 3: LAYER_TOP}
        st['at'], st['dt'] = _layer_inflow(case, seed), _layer_dt(case)
    elif case.get('flow') == 'diffraction':
        kw['inflow'] = {0: _post_shock()}
    s = hweno.Solver(nx, ny, gradients=case.get('gradients', 'GR'), **kw)
    if case.get('flow') == 'diffraction':
        s.set_solid(_solid(nx, ny))
    if kind == 'vjp':
        st['R'], st['V'] = _seeds_vjp(case, seed, dev)
    elif kind == 'rollout':
        if case['record']:
            s.set_record(2 * case['every'])
        st['W'], st['dt'] = _seeds_vjp(case, seed, dev)[0], _rollout_dt(case)
        st['mu'] = torch.tensor(p['mu_ref'], dtype=torch.float64, device=dev, requires_grad=True)
        st['U'].requires_grad_(True)
    st['s'] = s
    return st


def run(state):
    case = state['case']
    kind = case['kind']
    if kind == 'batch':
        b = state['b']
        for i, U in enumerate(state['U']):
            b.set_state(i, U)
        b.run(case['steps'])
        return [b.get_state(i) for i in range(b.n)]
    s, U = state['s'], state['U']
    if kind == 'residual':
        R, V, _ = (s.residual_noalloc if case['noalloc'] else s.residual)(U, diag=False)
        return R, V
    if kind == 'vjp':
        return s.residual_vjp(U, state['R'], state['V'])
    if kind == 'rollout':
        Un = adjoint.rollout(s, U, state['mu'], state['dt'], case['steps'], case['every'])
        return (Un.detach(),) + torch.autograd.grad(Un, (U, state['mu']), state['W'])
    s.set_state(U)
    if case['flow'] == 'layer':
        at, dt = state['at'], state['dt']
        for k in range(case['steps']):
            t = k * dt
            s.set_inflow_stages(0, at(t), at(t + dt), at(t + 0.5 * dt))
            s.rk_step_inflow(dt)
    else:
        for _ in range(case['steps']):
            s.rk_step(0.0)
    return s.get_state()


# Floating-point operations per cell-stage of the method (bench.py counts the
# 2D ones kernel by kernel; the 1D ones likewise: 3 + 2 scalar
# reconstructions, the characteristic projection, limiter, fluxes, update).
FLOPS_2D, FLOPS_1D = 12411.0, 900.0


def work(case):
    """Bytes: every call reads its input state and writes its results once;
    flops: the method's operations per cell-stage (a reverse sweep counts
    twice its forward evaluation)."""
    kind = case['kind']
    if kind == 'steps1d':
        n, k = case['nx'], case['steps']
        return dict(bytes=8.0 * 12 * n * (k + 2), flops=3.0 * FLOPS_1D * n * k)
    if kind == 'batch':
        n, k = sum(m * m for m, _ in _batch_problems(case)), case['steps']
        return dict(bytes=8.0 * 24 * n * (k + 2), flops=3.0 * FLOPS_2D * n * k)
    n = case['nx'] * case['ny']
    if kind == 'steps2d':
        k = case['steps']
        return dict(bytes=8.0 * 24 * n * (k + 2), flops=3.0 * FLOPS_2D * n * k)
    if kind == 'residual':
        return dict(bytes=8.0 * 32 * n, flops=FLOPS_2D * n)
    if kind == 'vjp':
        return dict(bytes=8.0 * 44 * n, flops=3.0 * FLOPS_2D * n)
    k = case['steps']
    return dict(bytes=8.0 * 60 * n * k, flops=9.0 * FLOPS_2D * n * k)


# ---------------------------------------------------------------------------
# The scheme in plain float64 torch: ghost cells, characteristic HWENO in two
# bases, positivity limiter, weak-derivative (GR) or differentiated (DR)
# gradients, Lax-Friedrichs and volume fluxes, SSP-RK3 with modified moments
# ---------------------------------------------------------------------------
G3 = np.array([-math.sqrt(15.0) / 10.0, 0.0, math.sqrt(15.0) / 10.0])
W3 = np.array([5.0 / 18.0, 4.0 / 9.0, 5.0 / 18.0])
LGL = np.array([-0.5, -math.sqrt(5.0) / 10.0, math.sqrt(5.0) / 10.0, 0.5])
WLGL = np.array([1.0, 5.0, 5.0, 1.0]) / 12.0
_TABLES = {}


def _int1(n, d, first):
    """int (s + d)^n ds, or with an extra factor s, over the unit cell."""
    x, w = np.polynomial.legendre.leggauss(8)
    x, w = 0.5 * x, 0.5 * w
    return float(np.sum(w * (x + d) ** n * (x if first else 1.0)))


def _tables(dim, dev):
    """Quartic candidate map, smoothness form and point/moment evaluation rows."""
    if (dim, str(dev)) in _TABLES:
        return _TABLES[dim, str(dev)]
    x, w = np.polynomial.legendre.leggauss(6)
    x, w = 0.5 * x, 0.5 * w

    def powers(pts, n, order):
        return np.array([[math.prod(range(k - order + 1, k + 1)) * p ** (k - order)
                          if k >= order else 0.0 for k in range(n)] for p in pts])
    T = {}
    if dim == 1:
        A = np.array([[_int1(k, d, f) for k in range(5)]
                      for d, f in ((-1, 0), (0, 0), (1, 0), (-1, 1), (1, 1))])
        T['Q'] = np.linalg.inv(A)
        T['G'] = sum(E.T @ (w[:, None] * E) for E in (powers(x, 5, o) for o in range(1, 5)))
        T['P'], T['D'] = powers(LGL, 5, 0), powers(LGL, 5, 1)
        T['M'] = np.array([[_int1(k, 0, 1) for k in range(5)]])
    else:
        mono = [(t - b, b) for t in range(5) for b in range(t + 1)]
        off = [(k % 3 - 1, k // 3 - 1) for k in range(9)]

        def row(kind, c):
            return [_int1(a, off[c][0], kind == 1) * _int1(b, off[c][1], kind == 2)
                    for a, b in mono]
        edge = (1, 3, 5, 7)
        slots = [(0, c) for c in range(9)] + [(1, c) for c in edge] + [(2, c) for c in edge]
        lsq = [slots.index(q) for q in ((1, 1), (1, 7), (2, 3), (2, 5))]
        exact_ = [q for q in range(17) if q not in lsq]
        A = np.array([row(*slots[q]) for q in exact_])
        B = np.array([row(*slots[q]) for q in lsq])
        # least squares on B over the affine set A c = a (null-space method)
        _, _, Vt = np.linalg.svd(A)
        Z, Ap = Vt[13:].T, np.linalg.pinv(A)
        H = Z @ np.linalg.pinv(B @ Z)
        Q = np.zeros((15, 17))
        Q[:, exact_] = Ap - H @ B @ Ap
        Q[:, lsq] = H
        T['Q'] = Q
        G = np.zeros((15, 15))
        for oa in range(5):
            for ob in range(5 - oa):
                if oa + ob:
                    Ex, Ey = powers(x, 5, oa), powers(x, 5, ob)
                    E = np.array([[Ex[i, a] * Ey[j, b] for a, b in mono]
                                  for i in range(6) for j in range(6)])
                    G += E.T @ (np.outer(w, w).ravel()[:, None] * E)
        T['G'] = G
        pts = {'x': [(s, g) for s in (-0.5, 0.5) for g in G3],
               'y': [(g, s) for s in (-0.5, 0.5) for g in G3],
               'v': [(a, b) for b in G3 for a in G3]}
        for n, pp in pts.items():
            for o, tag in (((0, 0), ''), ((1, 0), 'dx'), ((0, 1), 'dy')):
                Ex = powers([q[0] for q in pp], 5, o[0])
                Ey = powers([q[1] for q in pp], 5, o[1])
                T[n + tag] = np.array([[Ex[i, a] * Ey[i, b] for a, b in mono]
                                       for i in range(len(pp))])
        T['mx'], T['my'] = np.array([row(1, 4)]), np.array([row(2, 4)])
    _TABLES[dim, str(dev)] = {k: torch.from_numpy(np.ascontiguousarray(v)).to(dev)
                              for k, v in T.items()}
    return _TABLES[dim, str(dev)]


def _apply(M, a):
    return (M @ a.reshape(a.shape[0], -1)).reshape((M.shape[0],) + a.shape[1:])


def _wsum(w, A):
    """sum_q w_q A[q]"""
    return sum(float(wq) * A[q] for q, wq in enumerate(w))


def _combine(a, T, slopes, gam):
    """Coefficients of the nonlinear combination: the quartic candidate and the
    linear ones with the given slope vectors about the own average."""
    c0, eps = _apply(T['Q'], a), 1e-8
    beta = [(_apply(T['G'], c0) * c0).sum(0)] + [sum(s * s for s in sl) for sl in slopes]
    tau = (sum((beta[0] - b).abs() for b in beta[1:]) / len(slopes)) ** 2
    wt = [g * (1.0 + tau / (b + eps)) for g, b in zip(gam, beta)]
    om = [q / sum(wt) for q in wt]
    C = list((om[0] / gam[0]) * c0)
    own = a[1] if a.shape[0] == 5 else a[4]
    for m, sl in enumerate(slopes, 1):
        d = om[m] - om[0] * (gam[m] / gam[0])
        C[0] = C[0] + d * own
        for k, s in enumerate(sl):
            C[1 + k] = C[1 + k] + d * s
    return torch.stack(C)


def _hweno2(a, T):
    l, r, b, t = a[4] - a[3], a[5] - a[4], a[4] - a[1], a[7] - a[4]
    return _combine(a, T, [(l, b), (r, b), (l, t), (r, t)], (0.99,) + (0.0025,) * 4)


def _hweno1(a, T):
    return _combine(a, T, [(a[1] - a[0],), (a[2] - a[1],)], (0.995, 0.0025, 0.0025))


def _pressure(U, gamma):
    return (gamma - 1.0) * (U[-1] - 0.5 * sum(m * m for m in U[1:-1]) / U[0])


def _prims(U):
    vel = [m / U[0] for m in U[1:-1]]
    return vel + [U[-1] / U[0] - 0.5 * sum(v * v for v in vel)]


def _limit(ub, pts, gamma, eps_pp=1e-12):
    """theta1 (density), theta2 (pressure) over the points (component first)."""
    rb, pb = ub[0], _pressure(ub, gamma)
    eps = torch.minimum(torch.minimum(torch.full_like(rb, eps_pp), rb), pb)
    rmin = torch.stack([p[0] for p in pts]).min(0)[0]
    low = rmin < eps
    th1 = torch.where(low, (rb - eps) / torch.where(low, rb - rmin, torch.ones_like(rb)),
                      torch.ones_like(rb))
    th2 = torch.ones_like(rb)
    for p in pts:
        q = _pressure([rb + th1 * (p[0] - rb)] + list(p[1:]), gamma)
        low = q < eps
        th = torch.where(low, (pb - eps) / torch.where(low, pb - q, torch.ones_like(rb)),
                         torch.ones_like(rb))
        th2 = torch.where(th < th2, th, th2)
    return th1, th2


def _limited(ub, p, th1, th2):
    q = torch.stack([ub[0] + th1 * (p[0] - ub[0])] + list(p[1:]))
    return ub + th2 * (q - ub)


class _Model:
    """The scheme on one grid; ``mu`` may be a tensor (for its gradient)."""

    def __init__(self, case, dev, grid=None):
        self.extent, self.bc, p = _setup(case)
        self.dev, self.gamma, self.Pr = dev, p['gamma'], p['Pr']
        self.mu, self.mu_exp, self.cfl = p['mu_ref'], p['mu_exp'], p['cfl']
        self.dr = case.get('gradients', 'GR') == 'DR'
        self.dim = 1 if case['kind'] == 'steps1d' else 2
        self.nx, self.ny = grid or (case['nx'], case.get('ny', 1))
        self.h = [(self.extent[1] - self.extent[0]) / self.nx]
        if self.dim == 2:
            self.h.append((self.extent[3] - self.extent[2]) / self.ny)
        self.T = _tables(self.dim, dev)
        self.inflow = {}          # side -> conservative (4,) or (4, n)
        self.solid = self.mirror = None

    def cons(self, prim):
        q = torch.as_tensor(np.asarray(prim, dtype=np.float64), device=self.dev)
        q = q.T if q.dim() == 2 else q
        r, u, v, p = q
        return torch.stack([r, r * u, r * v, p / (self.gamma - 1.0) + 0.5 * r * (u * u + v * v)])

    def visc(self, U):
        if self.mu_exp == 0.0:
            return self.mu
        return self.mu * (_pressure(U, self.gamma) / U[0]) ** self.mu_exp

    # -- masked domain: mirror images across the nearest wall face -----------
    def set_solid(self, S):
        ny, nx = S.shape
        dst, src, sg = [], [], []
        for j, i in zip(*np.nonzero(S)):
            if S[max(j - HALO, 0):j + HALO + 1, max(i - HALO, 0):i + HALO + 1].all():
                continue
            best = None
            for dj, di in ((0, 1), (0, -1), (1, 0), (-1, 0)):
                k = 1
                while 0 <= j + k * dj < ny and 0 <= i + k * di < nx and S[j + k * dj, i + k * di]:
                    k += 1
                if 0 <= j + k * dj < ny and 0 <= i + k * di < nx and (best is None or k < best[0]):
                    best = (k, dj, di)
            if best is None:
                continue
            k, dj, di = best
            a, b = j + (2 * k - 1) * dj, i + (2 * k - 1) * di
            if not (0 <= a < ny and 0 <= b < nx) or S[a, b]:
                a, b = j + k * dj, i + k * di
            dst.append(j * nx + i)
            src.append(a * nx + b)
            sg.append(self.wall_sign('slip', 0 if di else 1))
        self.solid = torch.from_numpy(S).to(self.dev)
        self.mirror = (torch.tensor(dst, device=self.dev), torch.tensor(src, device=self.dev),
                       torch.tensor(np.stack(sg, -1), device=self.dev))

    def fill_solid(self, U):
        if self.mirror is None:
            return U
        V, (dst, src, sg) = U.reshape(3, 4, -1).clone(), self.mirror
        V[:, :, dst] = sg * V[:, :, src]
        return V.reshape(U.shape)

    def wall_sign(self, kind, axis):
        """Parity per (moment, component) of a wall normal to `axis`."""
        nc = self.dim + 2
        s = np.ones((self.dim + 1, nc))
        s[1 + axis] = -1.0
        for c in range(1, nc - 1):
            if kind == 'noslip' or c - 1 == axis:
                s[:, c] *= -1.0
        return s

    def ghost(self, U):
        for axis in range(self.dim):
            d = U.dim() - 1 - axis
            n = U.shape[d]
            parts = [None, U, None]
            for side in (0, 1):
                kind = self.bc[2 * axis + side]
                if kind == 'periodic':
                    q = U.narrow(d, n - HALO, HALO) if side == 0 else U.narrow(d, 0, HALO)
                elif kind == 'outflow':
                    q = U.narrow(d, 0 if side == 0 else n - 1, 1)
                    q = q.expand(*[HALO if k == d else m for k, m in enumerate(q.shape)])
                elif kind == 'inflow':
                    q = torch.zeros_like(U.narrow(d, 0, HALO))
                    st = self.inflow[2 * axis + side]
                    if st.dim() == 2:
                        if axis == 1:        # ghost columns beyond the corners: end states
                            st = torch.cat([st[:, :1].expand(4, HALO), st,
                                            st[:, -1:].expand(4, HALO)], 1)[:, None, :]
                        else:
                            st = st[:, :, None]
                    else:
                        st = st.reshape((-1,) + (1,) * self.dim)
                    q[0] = st.expand_as(q[0])
                else:
                    sg = torch.tensor(self.wall_sign(kind, axis), device=self.dev)
                    q = U.narrow(d, 0 if side == 0 else n - HALO, HALO).flip(d)
                    q = q * sg.reshape(sg.shape + (1,) * self.dim)
                parts[2 * side] = q
            U = torch.cat(parts, d)
        return U

    # -- characteristic bases ------------------------------------------------
    def eig(self, ub, axis):
        g1 = self.gamma - 1.0
        r, E = ub[0], ub[-1]
        vel = [m / r for m in ub[1:-1]]
        q2 = sum(v * v for v in vel)
        p = _pressure(ub, self.gamma)
        c = (self.gamma * p / r).sqrt()
        H, b1 = (E + p) / r, g1 / (c * c)
        b2 = 0.5 * b1 * q2
        one, zero = torch.ones_like(r), torch.zeros_like(r)
        un = vel[axis]
        if self.dim == 1:
            R = [[one, un - c, H - un * c], [one, un, 0.5 * q2], [one, un + c, H + un * c]]
            L = [[0.5 * (b2 + un / c), -0.5 * (b1 * un + 1 / c), 0.5 * b1],
                 [1 - b2, b1 * un, -b1],
                 [0.5 * (b2 - un / c), 0.5 * (1 / c - b1 * un), 0.5 * b1]]
            return L, R
        ut = vel[1 - axis]
        R = [[one, un - c, ut, H - un * c], [one, un, ut, 0.5 * q2], [zero, zero, one, ut],
             [one, un + c, ut, H + un * c]]
        L = [[0.5 * (b2 + un / c), -0.5 * (b1 * un + 1 / c), -0.5 * b1 * ut, 0.5 * b1],
             [1 - b2, b1 * un, b1 * ut, -b1], [-ut, zero, one, zero],
             [0.5 * (b2 - un / c), 0.5 * (1 / c - b1 * un), -0.5 * b1 * ut, 0.5 * b1]]
        if axis == 1:     # normal momentum in slot 2
            R = [[q[0], q[2], q[1], q[3]] for q in R]
            L = [[q[0], q[2], q[1], q[3]] for q in L]
        return L, R

    # -- physics at points; s = gradients ------------------------------------
    def flux(self, U, s, axis):
        vel, p, mu = [m / U[0] for m in U[1:-1]], _pressure(U, self.gamma), self.visc(U)
        kq = self.gamma * mu / self.Pr
        if self.dim == 1:
            t = [4.0 / 3.0 * mu * s[0]]
            q = kq * s[1]
        else:
            ux, uy, vx, vy, ex, ey = s
            xy = mu * (uy + vx)
            t = ([mu * (4.0 / 3.0 * ux - 2.0 / 3.0 * vy), xy] if axis == 0 else
                 [xy, mu * (4.0 / 3.0 * vy - 2.0 / 3.0 * ux)])
            q = kq * (ex, ey)[axis]
        un = vel[axis]
        f = [U[1 + axis]]
        for c in range(self.dim):
            f.append(U[1 + c] * un + (p if c == axis else 0.0) - t[c])
        f.append((U[-1] + p) * un - (sum(a * b for a, b in zip(t, vel)) + q))
        # the positivity bound of the wave speed, no smaller than |u_n| + c
        r2e = U[0] * p / (self.gamma - 1.0)
        t2 = sum((t[c] - (p if c == axis else 0.0)) ** 2 for c in range(self.dim))
        root = (U[0] * U[0] * q * q + 2.0 * r2e * t2).sqrt()
        bpp = un.abs() + (root + U[0] * q.abs()) / (2.0 * r2e)
        ac = un.abs() + (self.gamma * p / U[0]).sqrt()
        return torch.stack(f), torch.where(ac >= bpp, ac, bpp)

    def prim_grads(self, P, D):
        """Gradients of the velocities and e from conservative derivatives."""
        vel = [m / P[0] for m in P[1:-1]]
        out = [(D[1 + c] - vel[c] * D[0]) / P[0] for c in range(self.dim)]
        e = (D[-1] - P[-1] / P[0] * D[0]) / P[0] - sum(v * o for v, o in zip(vel, out))
        return out + [e]

    def residual(self, U):
        """(F, Vhat, alpha) of the interior state."""
        return self.residual1(U) if self.dim == 1 else self.residual2(U)

    def residual1(self, U):
        Ug, T, dx = self.ghost(U), self.T, self.h[0]
        n = Ug.shape[-1]
        ub = Ug[0][:, 1:n - 1]
        L, R = self.eig(ub, 0)
        st = [Ug[0][:, 0:n - 2], ub, Ug[0][:, 2:n], Ug[1][:, 0:n - 2], Ug[1][:, 2:n]]
        pts, vh, dv = 0.0, 0.0, 0.0
        for k in range(3):
            a = torch.stack([sum(L[k][c] * q[c] for c in range(3)) for q in st])
            C = _hweno1(a, T)
            col = torch.stack(R[k])
            pts = pts + col[None] * _apply(T['P'], C)[:, None]
            vh = vh + col * _apply(T['M'], C)
            dv = dv + col[None] * _apply(T['D'], C)[:, None] / dx
        th1, th2 = _limit(ub, list(pts), self.gamma)
        P = torch.stack([_limited(ub, p, th1, th2) for p in pts])     # (4, 3, n - 2)
        if self.dr:
            s = torch.stack([torch.stack(self.prim_grads(P[q], dv[q])) for q in range(4)])
            s = s[:, :, 2:-2]
        else:
            w = torch.stack([torch.stack(_prims(P[q])) for q in range(4)])
            wb = _wsum(WLGL, w)
            wh = 0.5 * (w[3, :, :-1] + w[0, :, 1:])
            m0 = (wh[:, 1:] - wh[:, :-1]) / dx
            m1 = (0.5 * (wh[:, 1:] + wh[:, :-1]) - wb[:, 1:-1]) / dx
            s = torch.stack([_apply(T['P'], _hweno1(torch.stack(
                [m0[q, :-2], m0[q, 1:-1], m0[q, 2:], m1[q, :-2], m1[q, 2:]]), T))
                for q in range(2)], 1)
        P = P[:, :, 2:-2]
        fs = [self.flux(P[q], s[q], 0) for q in range(4)]
        (fm, bm), (fp, bp) = fs[3], fs[0]
        beta = torch.where(bm[:-1] >= bp[1:], bm[:-1], bp[1:])
        fh = 0.5 * (fm[:, :-1] + fp[:, 1:] - beta * (P[0][:, 1:] - P[3][:, :-1]))
        vol = _wsum(WLGL, [f[0] for f in fs])[:, 1:-1]
        F = torch.stack([-(fh[:, 1:] - fh[:, :-1]) / dx,
                         -(fh[:, 1:] + fh[:, :-1]) / (2.0 * dx) + vol / dx])
        Pi = P[:, :, 1:-1]
        alpha = max(((q[1] / q[0]).abs() + (self.gamma * _pressure(q, self.gamma) / q[0]).sqrt()
                     ).max() for q in (Pi[0], Pi[3]))
        return F, vh[:, 3:-3][None], alpha

    def residual2(self, U):
        Ug, T = self.ghost(U), self.T
        ny, nx = Ug.shape[2:]
        ub = Ug[0][:, 1:-1, 1:-1]

        def nb(m, k):
            return Ug[m][:, k // 3:ny - 2 + k // 3, k % 3:nx - 2 + k % 3]
        st = ([nb(0, k) for k in range(9)] + [nb(1, k) for k in (1, 3, 5, 7)]
              + [nb(2, k) for k in (1, 3, 5, 7)])
        face, vol, vhat, dface, dvol = [], [], [], [], []
        for b, (fn, mn) in enumerate((('x', 'mx'), ('y', 'my'))):
            L, R = self.eig(ub, b)
            acc = [0.0] * 7
            for k in range(4):
                a = torch.stack([sum(L[k][c] * q[c] for c in range(4)) for q in st])
                C = _hweno2(a, T)
                col = torch.stack(R[k])
                names = [fn, 'v', mn] + ([fn + 'dx', fn + 'dy', 'vdx', 'vdy'] if self.dr else [])
                for z, nm in enumerate(names):
                    acc[z] = acc[z] + col[None] * _apply(T[nm], C)[:, None]
            face.append(acc[0])
            vol.append(acc[1])
            vhat.append(acc[2][0])
            if self.dr:
                dface.append((acc[3] / self.h[0], acc[4] / self.h[1]))
                dvol.append((acc[5] / self.h[0], acc[6] / self.h[1]))
        th1, th2 = _limit(ub, [q for A in face + vol for q in A], self.gamma)
        face = [torch.stack([_limited(ub, q, th1, th2) for q in A]) for A in face]
        ring = (Ellipsis, slice(2, -2), slice(2, -2))
        if self.dr:
            def grads(P, D):
                out = []
                for q in range(P.shape[0]):
                    gx, gy = self.prim_grads(P[q], D[0][q]), self.prim_grads(P[q], D[1][q])
                    out.append(torch.stack([gx[0], gy[0], gx[1], gy[1], gx[2], gy[2]]))
                return torch.stack(out)[ring]
            sf = [grads(face[b], dface[b]) for b in range(2)]
            sv = [grads(vol[b], dvol[b]) for b in range(2)]
        else:
            sf, sv = self.weak_gradients(face, vol)
        face = [A[ring] for A in face]
        vol = [A[ring] for A in vol]
        W0, W1 = [], []          # Gauss averages and first moments of the face fluxes
        for b in range(2):
            d = face[b].dim() - 1 - b
            n = face[b].shape[d]
            f = [self.flux(face[b][q], sf[b][q], b) for q in range(6)]

            def lo(A, d=d, n=n, k=face[b].dim()):
                return A.narrow(d - (k - A.dim()), 0, n - 1)

            def hi(A, d=d, n=n, k=face[b].dim()):
                return A.narrow(d - (k - A.dim()), 1, n - 1)
            beta = torch.stack([lo(f[3 + q][1]) for q in range(3)]
                               + [hi(f[q][1]) for q in range(3)]).max(0)[0]
            fh = [0.5 * (lo(f[3 + q][0]) + hi(f[q][0])
                         - beta * (hi(face[b][q]) - lo(face[b][3 + q]))) for q in range(3)]
            cut = (Ellipsis, slice(1, -1), slice(None)) if b == 0 else (Ellipsis, slice(1, -1))
            W0.append(_wsum(W3, fh)[cut])
            W1.append(_wsum(W3 * G3, fh)[cut])
        wv = [W3[q % 3] * W3[q // 3] for q in range(9)]
        fv = [_wsum(wv, [self.flux(vol[b][q], sv[b][q], b)[0] for q in range(9)])
              [..., 1:-1, 1:-1] for b in range(2)]
        (dx, dy), (x0, y0), (x1, y1) = self.h, W0, W1
        R, L_, T_, B = ((slice(None), slice(None), slice(1, None)),
                        (slice(None), slice(None), slice(None, -1)),
                        (slice(None), slice(1, None)), (slice(None), slice(None, -1)))
        F = torch.stack([
            -(x0[R] - x0[L_]) / dx - (y0[T_] - y0[B]) / dy,
            -(x0[R] + x0[L_]) / (2 * dx) - (y1[T_] - y1[B]) / dy + fv[0] / dx,
            -(x1[R] - x1[L_]) / dx - (y0[T_] + y0[B]) / (2 * dy) + fv[1] / dy])
        V = torch.stack([v[:, 3:-3, 3:-3] for v in vhat])
        if self.solid is not None:
            F, V = F.masked_fill(self.solid, 0.0), V.masked_fill(self.solid, 0.0)
        sp = [torch.maximum((q[1] / q[0]).abs(), (q[2] / q[0]).abs())
              + (self.gamma * _pressure(q, self.gamma) / q[0]).sqrt()
              for A in face for q in A[..., 1:-1, 1:-1]]
        return F, V, max(q.max() for q in sp)

    def weak_gradients(self, face, vol):
        """Gradients at the face and volume points (ring 1) from the
        weak-derivative moments of (u, v, e)."""
        wv = [W3[q % 3] * W3[q // 3] for q in range(9)]
        mom = []
        for b in range(2):
            w = [torch.stack(_prims(q)) for q in face[b]]
            wb = _wsum(wv, [torch.stack(_prims(q)) for q in vol[b]])
            d = 2 - b
            n = wb.shape[d]
            h = [0.5 * (w[3 + q].narrow(d, 0, n - 1) + w[q].narrow(d, 1, n - 1)) for q in range(3)]
            A0, A1 = _wsum(W3, h), _wsum(W3 * G3, h)

            def lo(A, d=d, n=n):
                return A.narrow(d, 0, n - 2)

            def hi(A, d=d, n=n):
                return A.narrow(d, 1, n - 2)
            m0, m1 = (hi(A0) - lo(A0)) / self.h[b], (hi(A1) - lo(A1)) / self.h[b]
            mm = (0.5 * (hi(A0) + lo(A0)) - wb.narrow(d, 1, n - 2)) / self.h[b]
            q = [m0, mm, m1] if b == 0 else [m0, m1, mm]
            mom.append([z.narrow(1 + b, 1, z.shape[1 + b] - 2) for z in q])
        J, I = mom[0][0].shape[1:]
        vals = {}
        for w in range(3):
            for b in range(2):
                def nb(m, k):
                    return mom[b][m][w, k // 3:J - 2 + k // 3, k % 3:I - 2 + k % 3]
                a = torch.stack([nb(0, k) for k in range(9)] + [nb(1, k) for k in (1, 3, 5, 7)]
                                + [nb(2, k) for k in (1, 3, 5, 7)])
                C = _hweno2(a, self.T)
                for nm in 'xyv':
                    vals[nm, w, b] = _apply(self.T[nm], C)
        s = {nm: torch.stack([vals[nm, w, b] for w in range(3) for b in range(2)], 1)
             for nm in 'xyv'}
        return [s['x'], s['y']], [s['v'], s['v']]

    # -- time stepping -------------------------------------------------------
    def admissible(self, U):
        ok = torch.isfinite(U).all(0).all(0) & (U[0, 0] > 0.0) & (_pressure(U[0], self.gamma) > 0.0)
        return bool((ok if self.solid is None else ok | self.solid).all())

    def step(self, U, dt=None, stage_inflow=None):
        """(U_new, dt): one SSP-RK3 step; dt None: the paper's rule with
        restarts at half the step."""
        def stage(V, k):
            if stage_inflow is not None:
                self.inflow.update(stage_inflow[k])
            V = self.fill_solid(V)
            F, Vh, al = self.residual(V)
            B = torch.cat([V[:1], Vh.reshape((-1,) + V.shape[1:])])
            return V, B, F, al

        def keep(new, V):
            return new if self.solid is None else torch.where(self.solid, V, new)
        auto, dt0 = dt is None, dt
        V0, B0, F0, al = stage(U, 0)
        if auto:
            h = min(self.h)
            dt0 = min(self.cfl * h / float(al), 0.001 * h * h / float(self.mu))
        for _ in range(64):
            U1 = keep(B0 + dt0 * F0, V0)
            V1, B1, F1, _al = stage(U1, 1)
            U2 = keep(0.75 * B0 + 0.25 * (B1 + dt0 * F1), V1)
            V2, B2, F2, _al = stage(U2, 2)
            U3 = keep(B0 / 3.0 + 2.0 / 3.0 * (B2 + dt0 * F2), V2)
            if not auto or all(self.admissible(q) for q in (U1, U2, U3)):
                return U3, dt0
            dt0 *= 0.5
        raise RuntimeError('no admissible step')


def exact(case, seed):
    """What run() returns, from the float64 torch model (the time of a state
    included)."""
    dev, kind = torch.device('cuda' if torch.cuda.is_available() else 'cpu'), case['kind']
    with torch.no_grad():
        if kind == 'batch':
            out = []
            for k, (n, Re) in enumerate(_batch_problems(case)):
                m = _Model(case, dev, grid=(n, n))
                m.mu = 1.0 / Re
                U, t = _batch_state(n, k, seed, dev), 0.0
                for _ in range(case['steps']):
                    U, dt = m.step(U)
                    t += dt
                out.append((U, t))
            return out
        m = _Model(case, dev)
        if kind == 'steps1d':
            U = _state1d(case, seed, dev)
        else:
            U = _state2d(case, seed, dev)
        if kind in ('steps1d', 'steps2d'):
            t = 0.0
            if case['flow'] == 'layer':
                at, dt = _layer_inflow(case, seed), _layer_dt(case)
                m.inflow = {3: m.cons(LAYER_TOP)}
                for k in range(case['steps']):
                    t = k * dt
                    U, _ = m.step(U, dt, [{0: m.cons(at(q))} for q in (t, t + dt, t + 0.5 * dt)])
                return U, case['steps'] * dt
            if case['flow'] == 'diffraction':
                m.inflow = {0: m.cons(_post_shock())}
                m.set_solid(_solid(case['nx'], case['ny']))
            for _ in range(case['steps']):
                U, dt = m.step(U)
                t += dt
            return U, t
        if kind == 'residual':
            F, V, _ = m.residual(U)
            return F, V.reshape((8,) + V.shape[2:])
    if kind == 'vjp':
        R, V = _seeds_vjp(case, seed, dev)
        U.requires_grad_(True)
        m.mu = torch.tensor(m.mu, dtype=torch.float64, device=dev, requires_grad=True)
        F, Vh, _ = m.residual(U)
        gU, gmu = torch.autograd.grad((F, Vh), (U, m.mu), (R, V.reshape(Vh.shape)))
        return gU, float(gmu)
    W, dt = _seeds_vjp(case, seed, dev)[0], _rollout_dt(case)
    states = [U]
    with torch.no_grad():
        for _ in range(case['steps']):
            states.append(m.step(states[-1], dt)[0])
    g, gmu, mu0 = W, 0.0, m.mu
    for Uk in reversed(states[:-1]):
        x = Uk.clone().requires_grad_(True)
        m.mu = torch.tensor(mu0, dtype=torch.float64, device=dev, requires_grad=True)
        g, q = torch.autograd.grad(m.step(x, dt)[0], (x, m.mu), g)
        gmu = gmu + q
    return states[-1], g, gmu
