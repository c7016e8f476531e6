#!/usr/bin/env python3
"""Throughput benchmark of the HWENO-GR hot path on one MI355X.

Workload: the 2D viscous shock tube on [0,1] x [0,0.5] with 1000 x 500
cells (gamma 1.4, Re 200, Pr 0.73, adiabatic no-slip walls at x = 0, x = 1,
y = 0 and a symmetry line at y = 0.5; rho = 120 | 1.2, p = rho/gamma, at rest),
advanced by SSP-RK3 steps with the paper's time-step rule from t = 0.
A step is three stages; each stage is one full residual evaluation (ghost
fill, characteristic HWENO reconstruction with the positivity limiter, weak
derivative moments, gradient reconstruction, fluxes) plus the stage update.
The state lives in HBM before the timed region starts.

Prints one JSON line.  ``value`` = cell-stage updates per second of that
grid.  Three more measurements ride along in the same line:

* ``developed``: the same grid timed from its t = 0.3 state (shocks, contact
  and wall layers present);
* ``batched``: 64 periodic 2D grids (64^2..512^2, Re log-uniform in
  [1e2, 1e4], random-phase Fourier velocity fields) advanced 100 steps each by
  one graph launch, against the same 64 problems run one after another through
  the single-grid path;
* ``adjoint``: the double shear layer on 256^2 (Re 1000), 200 steps with dt
  frozen, forward plus checkpointed backward (every 20 steps) against the
  plain forward;
* ``dr``: the same grid with the comparison scheme HWENO-DR (gradients by
  differentiating the convective reconstruction), and T_GR / T_DR.
"""

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = '2D cell-stage updates/s FP64 + %HBM roofline; batched & adjoint vs plain'
UNIT = 'cell-stage updates/s'
NX, NY = 1000, 500
EXTENT = (0.0, 1.0, 0.0, 0.5)
BCS = ('noslip', 'noslip', 'noslip', 'slip')
PHYS = dict(gamma=1.4, Pr=0.73, mu_ref=1.0 / 200.0)

# MI355X published peaks
PEAK_FP64_TFLOPS = 78.6        # FP64 vector (FP64 matrix is the same)
PEAK_HBM_GBS = 8000.0

# Algorithmic FP64 operations per cell (per face for 'flux') of each kernel
# class, counted from the operations of the method as the kernels perform
# them once per cell (additions, multiplications, divisions, square roots
# each one flop; a fused multiply-add two):
#   recon: 8 scalar reconstructions (projection 136, quartic candidate 138,
#          smoothness indicator 87, weights 45, combination 35, 15 point values
#          135, moment 5) = 4648; characteristic bases 75; back-transform 1024;
#          limiter on 30 points 420; wbar 240; wave speed 300; convective
#          volume fluxes and their Gauss sums at 18 points 342.
#   grad:  interface averages, face moments and 18 weak moments 414; 6 scalar
#          reconstructions at 21 points (495 each) = 2970; viscous volume fluxes
#          at 18 points and the sums 458.
#   flux:  per face 6 point fluxes and PP speed bounds, 12 LF combinations.
#   update: assembly of 12 residual entries and the stage combination.
#   fluxup: the face fluxes formed inside the update kernel, per cell: the
#          fluxes of two faces and the update (faces on tile edges, formed
#          twice, counted once).
FLOPS = {'recon': 7049, 'grad': 3842, 'flux': 560, 'update': 400,
         'fluxup': 2 * 560 + 400}
# HBM bytes per launch from rocprofv3 FETCH_SIZE and WRITE_SIZE (KiB per
# dispatch) scaled by the factors a 1 GiB device copy gives in the same process
# (FETCH x 2.0, WRITE x 1.0), per kernel class and tile variant, on this grid
# and for the kernels as they are now: e.g. recon with 32-column tiles reads
# 55.8 MB and writes 439.9 MB per launch, with 16-column tiles 63.6 and 439.8.
TRAFFIC_BYTES = {('recon', 16): 503450684, ('recon', 32): 495675392,
                 ('grad', None): 667913216, ('fluxup', None): 617230336}
# Algorithmic HBM bytes per cell-stage of the whole path if every input were
# read once and every output written once (stage average: 256 B residual
# in/out + the RK bases of stages 2 and 3).
ALGO_BYTES_PER_CELL_STAGE = 277.0


def pipeline_hbm(tiles, value):
    """HBM bytes the whole stage pipeline moves per cell-stage (the counter
    table above, for the tiles in use; ghost fill and reductions left out) and
    the rate they imply at the measured throughput."""
    if tiles.get('flux') != 0:   # split face-flux kernels have no entry in the table
        return None
    parts = [('recon', tiles.get('recon')), ('grad', None), ('fluxup', None)]
    if any(p not in TRAFFIC_BYTES for p in parts):
        return None
    per_cell = sum(TRAFFIC_BYTES[p] for p in parts) / (NX * NY)
    rate = per_cell * value
    return {'bytes_per_cell_stage': per_cell, 'GB/s': rate / 1e9,
            'frac': rate / (PEAK_HBM_GBS * 1e9),
            'note': 'rocprofv3 FETCH_SIZE + WRITE_SIZE per launch (calibrated), summed over the '
                    'kernels of one stage, times the measured cell-stage rate'}


def log(msg):
    print('[bench] ' + msg, file=sys.stderr, flush=True)


def units_per_launch(kind):
    if kind == 'recon':
        return (NX + 6) * (NY + 6)
    if kind == 'grad':
        return (NX + 2) * (NY + 2)
    if kind == 'flux':
        return (NX + 1) * NY + NX * (NY + 1)
    return NX * NY


def cpu_model():
    try:
        with open('/proc/cpuinfo') as f:
            for line in f:
                if line.startswith('model name'):
                    return line.split(':', 1)[1].strip()
    except OSError:
        pass
    return 'unknown'


def _c3_window_rate(rows, j0, reps):
    """Oracle cell-stages/s of ``reps`` stage residuals on a 1000 x rows window
    (true neighbours as halo) of the 1000x500 shock tube at t = 0, one thread."""
    from threadpoolctl import threadpool_limits
    from oracle.common import Options, Physics
    from oracle.scheme2d import Scheme2D
    from paper_2608_10569_amd import workloads
    U = workloads.viscous_shock_tube_2d(NX, NY)
    sc = Scheme2D(NX, NY, *EXTENT, Physics(**PHYS), Options(cfl=0.3), bc=BCS)
    W = sc.ghost(U)[:, :, j0:j0 + rows + 8, :]
    with threadpool_limits(1):
        t0 = time.perf_counter()
        for _ in range(reps):
            sc.residual_ghosted(W)
        el = time.perf_counter() - t0
    return reps * rows * NX, el


def _c3_worker(args):
    return _c3_window_rate(*args)


def _cpu_task(task):
    """One single-threaded oracle sample in a worker process: ('c1',) the
    smooth-wave run to t = 1; ('c2', nsteps) Sod at N = 2000; ('c4', n, Re, U)
    one step of a batched instance.  Returns (kind, cell-stages, seconds)."""
    from threadpoolctl import threadpool_limits
    import numpy as np
    from oracle import rk
    from oracle.common import Options, Physics
    from oracle.scheme1d import Scheme1D
    from oracle.scheme2d import Scheme2D
    from paper_2608_10569_amd import workloads
    with threadpool_limits(1):
        t0 = time.perf_counter()
        if task[0] == 'c1':
            sc = Scheme1D(200, 0.0, 2 * np.pi, Physics(gamma=1.4, Pr=0.72, mu_ref=0.01),
                          Options(cfl=0.3, b_visc=0.001, t_final=1.0))
            U, t, steps = workloads.smooth_wave_1d(200), 0.0, 0
            while t < 1.0 - 1e-12:
                U, dt, _ = rk.rk3_step(sc, U, t)
                t += dt
                steps += 1
            return 'c1', 3 * 200 * steps, time.perf_counter() - t0
        if task[0] == 'c2':
            sc = Scheme1D(2000, 0.0, 1.0, Physics(gamma=1.4, Pr=0.72, mu_ref=1e-3),
                          Options(cfl=0.3), bc=('outflow', 'outflow'))
            U, t = workloads.sod_1d(2000), 0.0
            for _ in range(task[1]):
                U, dt, _ = rk.rk3_step(sc, U, t)
                t += dt
            return 'c2', 3 * 2000 * task[1], time.perf_counter() - t0
        _, n, Re, U = task
        sc = Scheme2D(n, n, 0.0, 1.0, 0.0, 1.0, Physics(mu_ref=1.0 / Re), Options())
        rk.rk3_step(sc, U, 0.0)
        return 'c4', 3 * n * n, time.perf_counter() - t0


def cpu_baseline(rows=64, reps=3, c2_steps=1000):
    """The oracle (as it stands) on bounded samples of the benchmark's
    workloads, on this host: the 1000x500 shock tube as 1000 x ``rows``
    windows (three stage residuals = one RK step's spatial work each) on one
    thread (median of five) and on every core the process may use (one
    window per worker process, up to 16); then, over the same worker pool,
    one single-threaded task each: the 1D smooth-wave run to t = 1, Sod at
    N = 2000 for ``c2_steps`` steps, and one step of every batched
    instance."""
    import statistics
    from concurrent.futures import ProcessPoolExecutor
    from paper_2608_10569_amd import workloads
    nproc = os.cpu_count()
    usable = len(os.sched_getaffinity(0)) if hasattr(os, 'sched_getaffinity') else nproc
    workers = max(1, min(usable, 16))
    j0 = (NY - rows) // 2
    one = []
    for _ in range(5):
        n, el = _c3_window_rate(rows, j0, reps)
        one.append(n / el)
    rate1 = statistics.median(one)
    # all cores: the grid's rows split into windows, one per worker process
    starts = [min(k * rows, NY - rows) for k in range(workers)]
    with ProcessPoolExecutor(max_workers=workers) as ex:
        t0 = time.perf_counter()
        res = list(ex.map(_c3_worker, [(rows, j, reps) for j in starts]))
        wall = time.perf_counter() - t0
    rate_all = sum(n for n, _ in res) / wall
    # the other workloads: the two 1D tasks first, then the batched instances
    # largest first (longest-processing-time order)
    inst = sorted(workloads.batched_periodic_2d(), key=lambda x: -x[0])
    tasks = [('c1',), ('c2', c2_steps)] + [('c4', n, Re, U) for n, Re, U in inst]
    with ProcessPoolExecutor(max_workers=workers) as ex:
        t0 = time.perf_counter()
        out = list(ex.map(_cpu_task, tasks))
        wall4 = time.perf_counter() - t0
    by = {k: [(n, el) for kk, n, el in out if kk == k] for k in ('c1', 'c2', 'c4')}
    c4n = sum(n for n, _ in by['c4'])
    c4s = sum(el for _, el in by['c4'])
    extra = {
        'c1_smooth_n200': {'value': by['c1'][0][0] / by['c1'][0][1], 'threads': 1,
                           'sample': 'the whole run to t = 1 (%d cell-stages)' % by['c1'][0][0],
                           's': by['c1'][0][1]},
        'c2_sod_n2000': {'value': by['c2'][0][0] / by['c2'][0][1], 'threads': 1,
                         'sample': '%d steps' % c2_steps, 's': by['c2'][0][1]},
        'c4_batched': {'value_one_thread': c4n / c4s, 'value_all_threads': c4n / wall4,
                       'threads': workers,
                       'sample': 'one step of each of the %d instances (%d cells), one '
                                 'process per instance; all-thread rate over the pool\'s wall '
                                 'time, which also ran the two 1D tasks' % (len(inst), c4n // 3),
                       's_one_thread_sum': c4s, 's_wall': wall4}}
    return {'value': rate_all, 'unit': UNIT, 'cores': workers, 'kind': 'oracle',
            'sample': '%d worker processes, each %d stage residuals on a 1000x%d-cell window of '
                      'the 1000x500 shock tube at t=0 (true neighbours as halo), numpy, one '
                      'thread per process, %.1f s wall' % (workers, reps, rows, wall),
            'one_thread': {'value': rate1, 'unit': UNIT, 'median_of': len(one),
                           'sample': '%d stage residuals on rows %d..%d' % (reps, j0,
                                                                             j0 + rows - 1)},
            'cpu_model': cpu_model(), 'nproc': nproc, 'usable_cpus': usable,
            'other_workloads': extra}


def bench_batched(nsteps, sequential=True):
    """64 instances in one graph launch vs one after another (plain path)."""
    import torch
    from paper_2608_10569_amd import hweno, workloads
    inst = workloads.batched_periodic_2d()
    probs = [dict(nx=n, ny=n, mu_ref=1.0 / Re) for n, Re, _ in inst]
    cells = sum(n * n for n, _, _ in inst)
    states = [torch.from_numpy(U).cuda() for _, _, U in inst]
    b = hweno.Batch(probs)
    for i, U in enumerate(states):
        b.set_state(i, U)
    tiles = b.autotune(reps=3)
    b.run(nsteps)                       # records and instantiates the graph
    runs = []
    for _ in range(3):                  # timed runs from the initial states; the median
        for i, U in enumerate(states):
            b.set_state(i, U)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        b.run(nsteps)
        torch.cuda.synchronize()
        runs.append(time.perf_counter() - t0)
    el = sorted(runs)[1]
    out = {'workload': '64 periodic 2D grids from {64,128,256,512}^2, Re log-uniform [1e2,1e4], '
                       '8 random-phase Fourier modes amplitude 0.3, %d SSP-RK3 steps each, one graph '
                       'launch' % nsteps,
           'instances': len(inst), 'cells': cells, 'steps': nsteps, 'seconds': el,
           'seconds_runs': runs, 'value': cells * 3 * nsteps / el, 'unit': UNIT, 'tiles': tiles,
           'restarts': sum(b.diag(i)['restarts'] for i in range(len(inst)))}
    del b
    torch.cuda.empty_cache()
    if sequential:
        el2 = 0.0
        for (n, Re, _), U in zip(inst, states):
            s = hweno.Solver(n, n, mu_ref=1.0 / Re)
            s.set_state(U)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(nsteps):
                s.rk_step(0.0)
            torch.cuda.synchronize()
            el2 += time.perf_counter() - t0
            s.close()
        out['sequential_seconds'] = el2
        out['sequential_value'] = cells * 3 * nsteps / el2
        out['speedup_vs_sequential'] = el2 / el
    return out


def bench_dr(nsteps, tiles, ms_gr):
    """The comparison scheme HWENO-DR on the same grid, rule and tiles: time
    per step and T_GR / T_DR (the paper's cost ratio of Table 5.3)."""
    import torch
    from paper_2608_10569_amd import hweno, workloads
    s = hweno.Solver(NX, NY, extent=EXTENT, bc=BCS, cfl=0.3, t_final=1.0, gradients='DR',
                     **PHYS)
    s.set_tiles(**tiles)
    s.set_state(torch.from_numpy(workloads.viscous_shock_tube_2d(NX, NY)).cuda())
    for _ in range(5):
        s.rk_step(0.0)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(nsteps):
        s.rk_step(0.0)
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    s.close()
    ms = 1e3 * el / nsteps
    return {'workload': 'the same 1000x500 shock tube and step rule, viscous gradients by '
                        'HWENO-DR (convective reconstruction differentiated, weights reused)',
            'steps': nsteps, 'ms_per_step': ms, 'value': nsteps * 3 * NX * NY / el,
            'unit': UNIT, 't_gr_over_t_dr': ms_gr / ms}


def bench_developed(nsteps, t_dev=0.3):
    """The same grid from a developed state: the shock tube advanced to
    t = 0.3 on the GPU (shock, contact and wall layers present) with the
    viscous step bound off (CFL 0.3, restarts keep the stages admissible),
    then ``nsteps`` timed steps with the paper's rule."""
    import torch
    from paper_2608_10569_amd import hweno, workloads
    kw = dict(extent=EXTENT, bc=BCS, cfl=0.3, **PHYS)
    s = hweno.Solver(NX, NY, b_visc=0.0, t_final=t_dev, **kw)
    s.set_state(torch.from_numpy(workloads.viscous_shock_tube_2d(NX, NY)).cuda())
    t0 = time.perf_counter()
    steps = 0
    while s.rk_step(0.0)['dt'] > 0.0:
        steps += 1
    t_prep = time.perf_counter() - t0
    U, t = s.get_state()
    s.close()
    s = hweno.Solver(NX, NY, t_final=1.0, **kw)
    s.set_state(U, t)
    for _ in range(5):
        s.rk_step(0.0)
    restarts = pp = 0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(nsteps):
        d = s.rk_step(0.0)
        restarts += d['restarts']
        pp += d['pp_cells']
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    s.close()
    return {'workload': 'the same 1000x500 shock tube from its t=%.1f state (%d preparation steps '
                        'with the viscous bound off, %.1f s), paper dt rule' % (t_dev, steps, t_prep),
            'steps': nsteps, 'ms_per_step': 1e3 * el / nsteps,
            'value': nsteps * 3 * NX * NY / el, 'unit': UNIT, 'restarts': restarts,
            'pp_cell_stages': pp}


def bench_adjoint(nsteps=200, every=20):
    """Double shear layer: forward + checkpointed backward vs plain forward.
    The backward recomputes each segment once, recording every step's stage
    intermediates (two banks of ``every`` recording slots in HBM, the next
    segment recorded on a second stream while the current one's adjoints
    run), and runs the step adjoints from the recordings; the same gradient
    from recomputing every
    stage residual inside each step adjoint (stage intermediates of stages 2
    and 3 kept) is timed too."""
    import numpy as np
    import torch
    from paper_2608_10569_amd import adjoint, hweno
    n, mu, gamma = 256, 1e-3, 1.4
    f = adjoint.shear_layer_fields(n)
    rho, u, v = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in f[:3]]
    s = hweno.Solver(n, n, mu_ref=mu, keep_stages=1)
    U0 = adjoint.project_fields(rho, u, v, f[3], gamma)
    s.set_state(U0)
    dt = s.rk_step(0.0)['dt']
    # plain forward: the same fixed-step steps through rk_step (median of three)
    fwd = []
    for _ in range(3):
        s.set_state(U0)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(nsteps):
            s.rk_step(dt)
        torch.cuda.synchronize()
        fwd.append(time.perf_counter() - t0)
    t_fwd = sorted(fwd)[1]
    def run(n_steps):
        r = rho.clone().requires_grad_(True)
        m = torch.tensor(mu, dtype=torch.float64, device=rho.device, requires_grad=True)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        J = adjoint.kinetic_energy(adjoint.rollout(s, adjoint.project_fields(r, u, v, f[3], gamma),
                                                   m, dt, n_steps, every), s.dx, s.dy)
        J.backward()
        torch.cuda.synchronize()
        return time.perf_counter() - t0, J.item(), m.grad.item(), r.grad
    # untimed warm-up: one checkpoint segment forward and backward (first
    # launches of the reverse-mode kernels, autograd set-up), without and
    # with recordings
    run(every)
    s.set_record(2 * every)
    run(2 * every)
    recs = [run(nsteps) for _ in range(3)]          # the median of three
    t_runs = [r[0] for r in recs]
    t_rec, J_rec, g_rec, r_rec = sorted(recs, key=lambda r: r[0])[1]
    rec_bytes = s._rec.numel()
    s.set_record(0)
    t_all, J, gmu, r_all = run(nsteps)
    # the recorded steps run the full-layout kernels, whose residuals differ
    # from the forward's by a unit in the last place in a few entries
    diff = {'rho_grad': ((r_rec - r_all).abs().max() / r_all.abs().max()).item(),
            'mu_grad': abs(g_rec - gmu) / abs(gmu), 'J': abs(J_rec - J) / abs(J)}
    cs = n * n * 3 * nsteps
    return {'workload': 'double shear layer 256^2, Re 1000, %d steps with dt frozen, checkpoints '
                        'every %d; d KE / d (rho, u, v node fields, mu)' % (nsteps, every),
            'forward_seconds': t_fwd, 'forward_seconds_runs': fwd,
            'forward_backward_seconds': t_rec,
            'forward_backward_seconds_runs': t_runs,
            'ratio_to_forward': t_rec / t_fwd, 'forward_value': cs / t_fwd,
            'value': cs / t_rec, 'unit': UNIT + ' (forward-equivalent, with gradient)',
            'recording_bytes': rec_bytes,
            'recompute_in_step_adjoints': {'forward_backward_seconds': t_all,
                                           'ratio_to_forward': t_all / t_fwd},
            'recorded_vs_recomputed_rel_diff': diff, 'J': J, 'dJ_dmu': gmu}


def main():
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument('--gpus', type=int, default=1)
    ap.add_argument('--steps', type=int, default=100)
    ap.add_argument('--warmup', type=int, default=10)
    ap.add_argument('--no-cpu-baseline', action='store_true')
    ap.add_argument('--cpu-rows', type=int, default=64)
    ap.add_argument('--batch-steps', type=int, default=100)
    ap.add_argument('--no-batched', action='store_true')
    ap.add_argument('--no-sequential', action='store_true')
    ap.add_argument('--no-adjoint', action='store_true')
    ap.add_argument('--no-developed', action='store_true')
    ap.add_argument('--no-dr', action='store_true')
    ap.add_argument('--no-autotune', action='store_true')
    ap.add_argument('--calib-copy-mib', type=int, default=0,
                    help='first run one device-to-device copy of this many MiB (a plain copy '
                         'kernel of known size, for calibrating HBM byte counters)')
    args = ap.parse_args()
    if args.gpus != 1:
        print('bench.py measures one GPU only: the library has no multi-GPU path (a grid '
              'would be split into y-slabs with a 4-row halo exchange per RK stage).',
              file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2608_10569_amd import hweno, workloads

    dev = torch.device('cuda:0')
    torch.cuda.set_device(dev)
    if args.calib_copy_mib > 0:
        n = args.calib_copy_mib * (1 << 20) // 8
        src = torch.ones(n, dtype=torch.float64, device=dev)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()
        log('calibration copy: %d bytes read, %d bytes written' % (8 * n, 8 * n))
        del src, dst
    U0 = torch.from_numpy(workloads.viscous_shock_tube_2d(NX, NY)).to(dev)
    s = hweno.Solver(NX, NY, extent=EXTENT, bc=BCS, device=dev, cfl=0.3, t_final=1.0, **PHYS)
    s.set_state(U0)
    tiles = s.tiles() if args.no_autotune else s.autotune(reps=3)
    for _ in range(args.warmup):
        s.rk_step(0.0)
    # every kernel class timed over a few untimed steps: the breakdown and the
    # dominant kernel (two events per launch slow the steps down)
    s.set_timing(True)
    s.timing(reset=True)
    for _ in range(5):
        s.rk_step(0.0)
    tm = s.timing(reset=True)
    dom = max(tm, key=lambda k: tm[k][0])
    # the timed region: only the dominant kernel's launches carry events
    s.set_timing(True, classes=[dom])
    restarts = 0
    pp = 0
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        d = s.rk_step(0.0)
        restarts += d['restarts']
        pp += d['pp_cells']
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    ms, n = s.timing()[dom]
    s.set_timing(False)
    _, t_end = s.get_state()
    # four more runs of the same length, untimed by events, for the spread
    reps = [1e3 * el / args.steps]
    for _ in range(4):
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        for _ in range(args.steps):
            s.rk_step(0.0)
        torch.cuda.synchronize()
        reps.append(1e3 * (time.perf_counter() - t1) / args.steps)

    cell_stages = args.steps * 3 * NX * NY
    value = cell_stages / el
    avg_s = ms / n / 1e3
    achieved = FLOPS[dom] * units_per_launch(dom) / avg_s / 1e12
    traffic = TRAFFIC_BYTES.get((dom, tiles.get(dom)), TRAFFIC_BYTES.get((dom, None)))
    kern = {k: {'ms_total': round(v[0], 3), 'launches': v[1],
                'us_avg': round(1e3 * v[0] / v[1], 2) if v[1] else None}
            for k, v in tm.items()}
    # the roof the kernel is nearer to: its FP64 work or the bytes it moves
    mem = bool(traffic) and traffic / avg_s / (PEAK_HBM_GBS * 1e9) > achieved / PEAK_FP64_TFLOPS
    path_flops = FLOPS['recon'] + FLOPS['grad'] + FLOPS['update'] + 2 * FLOPS['flux']
    out = {
        'metric': METRIC, 'value': value, 'unit': UNIT, 'n_gpus': 1,
        'steps': args.steps, 'warmup': args.warmup, 'ms_per_step': 1e3 * el / args.steps,
        'higher_is_better': True, 'scaling': 'weak', 'vs_baseline': None, 'dtype': 'f64',
        'data': 'synthetic',
        'config': {'workload': '2D viscous shock tube 1000x500, Re=200, Pr=0.73, no-slip walls + '
                               'symmetry top, SSP-RK3 CFL 0.3 from t=0, paper dt rule',
                   'cells': NX * NY, 'stages_per_step': 3, 't_end': t_end,
                   'restarts': restarts, 'pp_cell_stages': pp, 'tiles': tiles},
        'roofline': {'bound': 'hbm' if mem else 'alu', 'kernel': dom,
                     'achieved': traffic / avg_s / 1e9 if mem else achieved,
                     'peak': PEAK_HBM_GBS if mem else PEAK_FP64_TFLOPS,
                     'unit': 'GB/s' if mem else 'TFLOP/s',
                     'frac': traffic / avg_s / (PEAK_HBM_GBS * 1e9) if mem
                     else achieved / PEAK_FP64_TFLOPS,
                     'fp64_tflops': achieved,
                     'traffic': traffic,
                     'traffic_unit': 'HBM bytes per launch (rocprofv3 counters, calibrated)',
                     'traffic_gbs': traffic / avg_s / 1e9 if traffic else None,
                     'flops_per_unit': FLOPS[dom], 'units_per_launch': units_per_launch(dom),
                     'us_per_launch': avg_s * 1e6, 'launches_timed': n},
        # the whole residual pipeline (every kernel of a stage) against both
        # roofs: its algorithmic FP64 work and HBM bytes at the measured rate,
        # and the HBM bytes the counters measured for its kernels
        'path': {'fp64_tflops_algorithmic': value * path_flops / 1e12,
                 'fp64_frac': value * path_flops / 1e12 / PEAK_FP64_TFLOPS,
                 'flops_per_cell_stage': path_flops,
                 'hbm_bytes_per_cell_stage_algorithmic': ALGO_BYTES_PER_CELL_STAGE,
                 'hbm_frac_algorithmic':
                     value * ALGO_BYTES_PER_CELL_STAGE / (PEAK_HBM_GBS * 1e9),
                 'hbm_measured': pipeline_hbm(tiles, value)},
        'kernels': kern,
        'kernels_note': 'every class timed over 5 untimed steps before the timed region',
        'kernel_only_ms_per_step': sum(v[0] for v in tm.values()) / 5.0,
        'repeats_ms_per_step': reps,
        'median_ms_per_step': sorted(reps)[len(reps) // 2],
        'repeats_note': 'the timed run first, then four more runs of the same number of steps '
                        'continuing from its state',

    }
    s.close()
    del s
    torch.cuda.empty_cache()
    log('single grid: %.3e %s, %.3f ms/step' % (value, UNIT, 1e3 * el / args.steps))
    if not args.no_dr:
        out['dr'] = bench_dr(args.steps, tiles, 1e3 * el / args.steps)
        log('HWENO-DR: %.3f ms/step, T_GR/T_DR = %.2f' % (out['dr']['ms_per_step'],
                                                           out['dr']['t_gr_over_t_dr']))
    if not args.no_developed:
        out['developed'] = bench_developed(args.steps)
        log('developed state: %.3e %s' % (out['developed']['value'], UNIT))
    if not args.no_batched:
        out['batched'] = bench_batched(args.batch_steps, sequential=not args.no_sequential)
        log('batched: %.3e %s' % (out['batched']['value'], UNIT))
    if not args.no_adjoint:
        out['adjoint'] = bench_adjoint()
        log('adjoint: forward+backward / forward = %.2f' % out['adjoint']['ratio_to_forward'])
    if not args.no_cpu_baseline:
        out['cpu_baseline'] = cpu_baseline(args.cpu_rows)
        log('cpu baseline: %.3e %s' % (out['cpu_baseline']['value'], UNIT))
    print(json.dumps(out), flush=True)


if __name__ == '__main__':
    main()
