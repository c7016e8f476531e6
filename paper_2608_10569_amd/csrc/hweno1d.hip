// 1D HWENO residual and SSP-RK3 stage update (Sec. 2 of arXiv 2608.10569).
//
//   stage   a whole stage in one kernel: ghost cells, characteristic
//           reconstruction (eq. (2.4)) and PP limiter on the four LGL values,
//           weak-derivative moments (eqs. (2.6)-(2.8)) and their
//           reconstruction (eq. (2.9)) or the comparison scheme's gradients
//           (eq. (2.5)), fluxes (eq. (2.3)), assembly and the stage
//           combination (eqs. (2.2), (2.12))
//   ghost, recon, rbar, grad   the residual's HWENO-GR intermediates in memory
//           that the reverse mode reads

#include "hweno_kernels.h"

namespace hw {

namespace {

constexpr int HALO = 4;

__device__ __forceinline__ double wmax(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wmin(double v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

__global__ void k_ghost1(Grid1 g, double* S) {
    const int t = threadIdx.x;
    if (t >= 2 * HALO) return;
    const int right = t >= HALO;
    const int d = (t % HALO) + 1;
    const Side& sd = g.side[right];
    const long long N = g.NX;
    int di, si;
    if (!right) {
        di = HALO - d;
        si = sd.kind == 0 ? HALO + g.nx - d : (sd.kind == 1 ? HALO : HALO + d - 1);
    } else {
        di = HALO + g.nx - 1 + d;
        si = sd.kind == 0 ? HALO + d - 1 : (sd.kind == 1 ? HALO + g.nx - 1 : HALO + g.nx - d);
    }
    if (sd.kind == 2) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            S[c * N + di] = sd.inflow[c];
            S[(3 + c) * N + di] = 0.0;
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) S[q * N + di] = sd.sign[q] * S[q * N + si];
}

// Characteristic reconstruction + PP limiter on cells 1 .. NX-2.
__global__ void k_recon1(Grid1 g, const double* __restrict__ S) {
    const Consts& K = g.K;
    const long long N = g.NX;
    const int i = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    if (i > g.NX - 2) return;
    double ub[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) ub[c] = S[c * N + i];
    Eig1 e;
    eig1(K, ub, e);
    double P[4][3] = {{0.0}};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double l = e.L[k][c];
            a[0] += l * S[c * N + i - 1];
            a[1] += l * S[c * N + i];
            a[2] += l * S[c * N + i + 1];
            a[3] += l * S[(3 + c) * N + i - 1];
            a[4] += l * S[(3 + c) * N + i + 1];
        }
        double C[5], v[4];
        hweno1d(a, K, C);
        eval1d(C, v);
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int p = 0; p < 4; ++p) P[p][c] += e.R[c][k] * v[p];
    }
    // positivity limiter on the four LGL values (all four are rescaled)
    const double rbar = ub[0];
    const double pbar = pressure1(K, ub[0], ub[1], ub[2]);
    const double eps = fmin(fmin(K.eps_pp, rbar), pbar);
    double rmin = P[0][0];
#pragma unroll
    for (int p = 1; p < 4; ++p) rmin = fmin(rmin, P[p][0]);
    const double th1 = rmin < eps ? (rbar - eps) / (rbar - rmin) : 1.0;
    double th2 = 1.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        P[p][0] = rbar + th1 * (P[p][0] - rbar);
        const double pt = pressure1(K, P[p][0], P[p][1], P[p][2]);
        if (pt < eps) th2 = fmin(th2, (pbar - eps) / (pbar - pt));
    }
    double su = 0.0, se = 0.0;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            P[p][c] = ub[c] + th2 * (P[p][c] - ub[c]);
            g.pts[(p * 3 + c) * N + i] = P[p][c];
        }
        const double wq = (p == 0 || p == 3) ? LGL_W0 : LGL_W1;
        const double u = P[p][1] / P[p][0];
        su += wq * u;
        se += wq * (P[p][2] / P[p][0] - 0.5 * u * u);
    }
    g.wb[0 * N + i] = su;
    g.wb[1 * N + i] = se;
}

__device__ __forceinline__ void prim_ue(const Grid1& g, long long i, int p, double* w) {
    const long long N = g.NX;
    const double r = g.pts[(p * 3 + 0) * N + i];
    const double u = g.pts[(p * 3 + 1) * N + i] / r;
    w[0] = u;
    w[1] = g.pts[(p * 3 + 2) * N + i] / r - 0.5 * u * u;
}

// Weak-derivative moments on cells 2 .. NX-3.
__global__ void k_rbar1(Grid1 g) {
    const int i = 2 + blockIdx.x * blockDim.x + threadIdx.x;
    if (i > g.NX - 3) return;
    const long long N = g.NX;
    double a[2], b[2], c[2], d[2];
    prim_ue(g, i - 1, 3, a);
    prim_ue(g, i, 0, b);
    prim_ue(g, i, 3, c);
    prim_ue(g, i + 1, 0, d);
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const double hm = 0.5 * (a[w] + b[w]);
        const double hp = 0.5 * (c[w] + d[w]);
        g.rb[(w * 2 + 0) * N + i] = (hp - hm) * g.K.idx;
        g.rb[(w * 2 + 1) * N + i] = (0.5 * (hp + hm) - g.wb[w * N + i]) * g.K.idx;
    }
}

// Gradient reconstruction on cells 3 .. NX-4.
__global__ void k_grad1(Grid1 g) {
    const int i = 3 + blockIdx.x * blockDim.x + threadIdx.x;
    if (i > g.NX - 4) return;
    const long long N = g.NX;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const double* r0 = g.rb + (w * 2 + 0) * N;
        const double* r1 = g.rb + (w * 2 + 1) * N;
        const double a[5] = {r0[i - 1], r0[i], r0[i + 1], r1[i - 1], r1[i + 1]};
        double C[5], v[4];
        hweno1d(a, grad_consts(g.K), C);
        eval1d(C, v);
#pragma unroll
        for (int p = 0; p < 4; ++p) g.gr[(p * 2 + w) * N + i] = v[p];
    }
}

// ---------------------------------------------------------------------------
// A whole stage.  One wavefront takes ST_CELLS cells and the HALO cells on
// each side of them; lane l holds ghosted cell i = i0 + l and every
// intermediate of it in registers, neighbours are read by lane moves, so a
// stage has no exchange through memory and no barrier.  The cells at a
// wavefront's ends lose one valid lane per step of the stencil chain
// (reconstruction, weak moments, gradients, faces), which is the halo.
// A step is latency: as six launches per stage, each a chain of divisions on
// a few wavefronts, a step took 123 us on 200 and 126 us on 2000 cells (74 us
// of them in kernels); as three launches it takes 49 us on both.
// ---------------------------------------------------------------------------
constexpr int ST_CELLS = 64 - 2 * HALO;

__device__ __forceinline__ void atomic_max_key(HW_GLOBAL unsigned long long* slot, double v) {
    if (v > -INFINITY) atomicMax((unsigned long long*)slot, dkey(v));
}
__device__ __forceinline__ void atomic_min_key(HW_GLOBAL unsigned long long* slot, double v) {
    if (v < INFINITY) atomicMin((unsigned long long*)slot, dkey(v));
}

// rho > 0, p > 0 and every value finite
__device__ __forceinline__ bool admissible1(const Consts& K, const double* q, double& p) {
    p = pressure1(K, q[0], q[1], q[2]);
    bool ok = q[0] > 0.0 && p > 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) ok = ok && isfinite(q[k]);
    return ok;
}

template <bool DR>
__global__ __launch_bounds__(64) void k_stage1(Grid1 g, Stage1 A) {
    const Consts& K = g.K;
    const long long N = g.NX;
    const int lane = threadIdx.x;
    const int i = (int)blockIdx.x * ST_CELLS + lane;
    const bool own = lane >= HALO && lane < HALO + ST_CELLS && i < HALO + g.nx;
    // step size of stages 2 and 3: stage 2 forms it from the wave speed of
    // stage 1 (every wavefront the same), stage 3 reads it
    double dt = 0.0;
    if (A.stage == 2) {
        const double al = dkey_inv(g.red->alpha_key);
        dt = A.auto_dt ? fmin(fmin(A.cfl_h / al, A.visc_dt), A.t_left) : A.dt;
        if (blockIdx.x == 0 && lane == 0) {
            g.red->alpha1_key = g.red->alpha_key;
            g.red->dt = dt;
        }
    } else if (A.stage == 3) {
        dt = g.red->dt;
        if (A.clear && blockIdx.x == 0 && lane == 0) {
            Reduce* r = A.clear;
            r->alpha_key = r->beta_key = dkey(-INFINITY);
            r->pp_cells = 0;
            r->min_rho_key = r->min_p_key = dkey(INFINITY);
            r->bad[0] = r->bad[1] = r->bad[2] = r->bad[3] = 0;
        }
    }
    // stage input of this cell, ghost cells by the rule of their side
    const int right = i >= HALO + g.nx;
    const bool ghost = i < HALO || right;
    const int kind = g.side[right].kind;
    int si = min(i, g.NX - 1);
    if (ghost) {
        const int d = right ? si - (HALO + g.nx - 1) : HALO - si;   // distance from the side
        const int n = g.nx;
        if (!right) si = kind == 0 ? HALO + n - d : (kind == 1 ? HALO : HALO + d - 1);
        else si = kind == 0 ? HALO + d - 1 : (kind == 1 ? HALO + n - 1 : HALO + n - d);
    }
    double u[6];
    if (A.stage == 2) {   // U1 = B(U^n) + dt F(U^n)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            u[c] = fma(dt, g.fr[c * N + si], A.S0[c * N + si]);
            u[3 + c] = fma(dt, g.fr[(3 + c) * N + si], g.vn[c * N + si]);
        }
    } else {
        const double* in = A.in + (si - HALO) + A.first;
#pragma unroll
        for (int q = 0; q < 6; ++q) u[q] = in[q * A.plane];
    }
    if (ghost) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
            u[q] = kind == 2 ? (q < 3 ? g.side[right].inflow[q] : 0.0) : g.side[right].sign[q] * u[q];
    }
    double rmin = INFINITY, pmin = INFINITY;
    unsigned bad_in = 0;
    if (A.stage == 2) {
        double p;
        const bool ok = admissible1(K, u, p);
        if (own) {
            rmin = u[0];
            pmin = p;
        }
        bad_in = (unsigned)__popcll(__ballot(own && !ok));
        if (A.u1 && own) {
#pragma unroll
            for (int q = 0; q < 6; ++q) A.u1[q * N + i] = u[q];
        }
    } else if (A.stage == 1 && A.check) {
        double p;
        bad_in = (unsigned)__popcll(__ballot(own && !admissible1(K, u, p)));
    }
    // characteristic reconstruction (eq. (2.4)) in the basis of the cell average
    double P[4][3] = {{0.0}}, vh[3] = {0.0, 0.0, 0.0};
    double dP[4][3] = {{0.0}};
    {
        double l[6], r[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            l[q] = from_left(u[q]);
            r[q] = from_right(u[q]);
        }
        Eig1 e;
        eig1(K, u, e);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const double L = e.L[k][c];
                a[0] += L * l[c];
                a[1] += L * u[c];
                a[2] += L * r[c];
                a[3] += L * l[3 + c];
                a[4] += L * r[3 + c];
            }
            double C[5], v[4];
            hweno1d(a, K, C);
            eval1d(C, v);
            const double mo = moment1d(C);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
#pragma unroll
                for (int p = 0; p < 4; ++p) P[p][c] += e.R[c][k] * v[p];
                vh[c] += e.R[c][k] * mo;
            }
            if constexpr (DR) {   // the combination differentiated, its weights kept
                double dv[4];
                deval1d(C, dv);
#pragma unroll
                for (int c = 0; c < 3; ++c)
#pragma unroll
                    for (int p = 0; p < 4; ++p) dP[p][c] += e.R[c][k] * (dv[p] * K.idx);
            }
        }
    }
    // positivity limiter on the four LGL values (all four are rescaled)
    bool acted;
    {
        const double rbar = u[0];
        const double pbar = pressure1(K, u[0], u[1], u[2]);
        const double eps = fmin(fmin(K.eps_pp, rbar), pbar);
        const double rm = fmin(fmin(P[0][0], P[1][0]), fmin(P[2][0], P[3][0]));
        const double th1 = rm < eps ? (rbar - eps) / (rbar - rm) : 1.0;
        double th2 = 1.0;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            P[p][0] = rbar + th1 * (P[p][0] - rbar);
            const double pt = pressure1(K, P[p][0], P[p][1], P[p][2]);
            if (pt < eps) th2 = fmin(th2, (pbar - eps) / (pbar - pt));
        }
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int c = 0; c < 3; ++c) P[p][c] = u[c] + th2 * (P[p][c] - u[c]);
        acted = th1 < 1.0 || th2 < 1.0;
    }
    // gradients (u_x, e_x) at the LGL points
    double gr[4][2];
    if constexpr (DR) {
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double r = P[p][0], v = P[p][1] / r;
            const double ux = (dP[p][1] - v * dP[p][0]) / r;
            gr[p][0] = ux;
            gr[p][1] = (dP[p][2] - (P[p][2] / r) * dP[p][0]) / r - v * ux;
        }
    } else {
        double w[4][2], wb[2] = {0.0, 0.0};
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const double wq = (p == 0 || p == 3) ? LGL_W0 : LGL_W1;
            w[p][0] = P[p][1] / P[p][0];
            w[p][1] = P[p][2] / P[p][0] - 0.5 * w[p][0] * w[p][0];
            wb[0] += wq * w[p][0];
            wb[1] += wq * w[p][1];
        }
#pragma unroll
        for (int z = 0; z < 2; ++z) {
            const double hm = 0.5 * (from_left(w[3][z]) + w[0][z]);
            const double hp = 0.5 * (w[3][z] + from_right(w[0][z]));
            const double m0 = (hp - hm) * K.idx;
            const double m1 = (0.5 * (hp + hm) - wb[z]) * K.idx;
            const double a[5] = {from_left(m0), m0, from_right(m0), from_left(m1), from_right(m1)};
            double C[5], v[4];
            hweno1d(a, grad_consts(K), C);
            eval1d(C, v);
#pragma unroll
            for (int p = 0; p < 4; ++p) gr[p][z] = v[p];
        }
    }
    // fluxes at the LGL points: the volume quadrature, and the two sides of
    // the cell's faces
    double f[4][3], vf[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        flux1(K, P[p], gr[p][0], gr[p][1], f[p]);
        const double wq = (p == 0 || p == 3) ? LGL_W0 : LGL_W1;
#pragma unroll
        for (int c = 0; c < 3; ++c) vf[c] += wq * f[p][c];
    }
    const double bl = speed1(K, P[0], gr[0][0], gr[0][1]);
    const double br = speed1(K, P[3], gr[3][0], gr[3][1]);
    // face i + 1/2: this cell's upper side and the right neighbour's lower side
    const double beta = fmax(br, from_right(bl));
    double fh[3], F1[3], F2[3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
        fh[c] = 0.5 * (f[3][c] + from_right(f[0][c]) - beta * (from_right(P[0][c]) - P[3][c]));
    const double blo = from_left(beta);   // the face i - 1/2 (an own cell's lower face)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double fl = from_left(fh[c]);
        F1[c] = -(fh[c] - fl) * K.idx;
        F2[c] = -(fl + fh[c]) * (0.5 * K.idx) + vf[c] * K.idx;
    }
    const int t = i - HALO;
    if (own && A.src) {   // prescribed source moments (layout of R)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            F1[c] += A.src[c * g.nx + t];
            F2[c] += A.src[(3 + c) * g.nx + t];
        }
    }
    bool bad = false;
    if (own) {
        if (A.stage == 0) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                A.R[c * g.nx + t] = F1[c];
                A.R[(3 + c) * g.nx + t] = F2[c];
                A.V[c * g.nx + t] = vh[c];
            }
        } else if (A.stage == 1) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                g.fr[c * N + i] = F1[c];
                g.fr[(3 + c) * N + i] = F2[c];
                g.vn[c * N + i] = vh[c];
            }
        } else {
            const double a = A.stage == 2 ? 0.75 : 1.0 / 3.0;
            const double bb = A.stage == 2 ? 0.25 : 2.0 / 3.0;
            double nw[6], p;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                nw[c] = a * A.S0[c * N + i] + bb * (u[c] + dt * F1[c]);
                nw[3 + c] = a * g.vn[c * N + i] + bb * (vh[c] + dt * F2[c]);
            }
#pragma unroll
            for (int q = 0; q < 6; ++q) A.out[q * N + i] = nw[q];
            bad = !admissible1(K, nw, p);
            rmin = fmin(rmin, nw[0]);
            pmin = fmin(pmin, p);
        }
    }
    // reductions
    const double bm = wmax(own ? fmax(beta, blo) : -INFINITY);
    double am = -INFINITY;
    if (A.stage < 2) {
        if (own) {
#pragma unroll
            for (int p = 0; p < 4; p += 3) {
                const double pr = pressure1(K, P[p][0], P[p][1], P[p][2]);
                am = fmax(am, fabs(P[p][1] / P[p][0]) + sqrt(K.gamma * pr / P[p][0]));
            }
        }
        am = wmax(am);
    }
    rmin = wmin(rmin);
    pmin = wmin(pmin);
    const unsigned long long npp = __popcll(__ballot(own && acted));
    const unsigned nbad = (unsigned)__popcll(__ballot(bad));
    if (lane == 0) {
        atomic_max_key(&g.red->beta_key, bm);
        atomic_max_key(&g.red->alpha_key, am);
        atomic_min_key(&g.red->min_rho_key, rmin);
        atomic_min_key(&g.red->min_p_key, pmin);
        if (npp) atomicAdd((unsigned long long*)&g.red->pp_cells, npp);
        // stage 1 checks the input (slot 0), stage 2 U1 (slot 1) and U2
        if (bad_in) atomicAdd((unsigned int*)&g.red->bad[A.stage - 1], bad_in);
        if (nbad) atomicAdd((unsigned int*)&g.red->bad[A.stage], nbad);
    }
}

__global__ void k_copy_in1(Grid1 g, const double* __restrict__ U, double* __restrict__ S) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= g.nx * 6) return;
    const int q = t / g.nx, i = t % g.nx;
    S[(long long)q * g.NX + i + HALO] = U[t];
}

__global__ void k_copy_out1(Grid1 g, const double* __restrict__ S, double* __restrict__ U) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= g.nx * 6) return;
    const int q = t / g.nx, i = t % g.nx;
    U[t] = S[(long long)q * g.NX + i + HALO];
}

inline unsigned nb(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_copy_in1(const Grid1& g, const double* U, double* S, hipStream_t st) {
    k_copy_in1<<<nb((long long)g.nx * 6, 256), 256, 0, st>>>(g, U, S);
    return hipGetLastError();
}

hipError_t launch_copy_out1(const Grid1& g, const double* S, double* U, hipStream_t st) {
    k_copy_out1<<<nb((long long)g.nx * 6, 256), 256, 0, st>>>(g, S, U);
    return hipGetLastError();
}

hipError_t launch_ghost1(const Grid1& g, double* S, hipStream_t st, Timer* tm) {
    tbeg(tm, KC_GHOST, st);
    k_ghost1<<<1, 64, 0, st>>>(g, S);
    tend(tm, st);
    return hipGetLastError();
}

hipError_t launch_residual1(const Grid1& g, const double* S, hipStream_t st, Timer* tm) {
    tbeg(tm, KC_RECON, st);
    k_recon1<<<nb(g.NX - 2, 128), 128, 0, st>>>(g, S);
    tend(tm, st);
    tbeg(tm, KC_RBAR, st);
    k_rbar1<<<nb(g.NX - 4, 128), 128, 0, st>>>(g);
    tend(tm, st);
    tbeg(tm, KC_GRAD, st);
    k_grad1<<<nb(g.NX - 6, 128), 128, 0, st>>>(g);
    tend(tm, st);
    return hipGetLastError();
}

hipError_t launch_stage1(const Grid1& g, const Stage1& a, hipStream_t st, Timer* tm) {
    tbeg(tm, KC_FLUXUP, st);
    const unsigned n = nb(g.nx, ST_CELLS);
    if (g.K.dr) k_stage1<true><<<n, 64, 0, st>>>(g, a);
    else k_stage1<false><<<n, 64, 0, st>>>(g, a);
    tend(tm, st);
    return hipGetLastError();
}

}  // namespace hw
