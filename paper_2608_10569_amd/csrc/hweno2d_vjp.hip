// Reverse mode (vector-Jacobian product) of the 2D HWENO-GR residual of
// arXiv 2608.10569 (eq. (3.2) with eqs. (3.3)-(3.9)): given the adjoints of
// the residual R and of the modified moments, the adjoint of the input state
// and of the viscosity mu_ref.
//
// The forward pipeline is recomputed first (its intermediates stay in the
// workspace); the adjoint kernels then run in reverse order.  Every adjoint
// slot has exactly one writer and cross-cell sums are gathers in a fixed
// order, so the result is deterministic.
// Branches (limiter thetas, LF-speed maximum, |.| in the weights) follow the
// forward point; ties go to the lowest index in the order of the oracle.
//
//   k_adj_flux     face-flux adjoint (eq. (3.3)) -> trace / face-gradient adjoints
//   k_adj_grad     volume-flux + gradient-reconstruction adjoint (eq. (3.9))
//   k_adj_rgather  gather of the weak-moment adjoints from the 3x3 stencils
//   k_adj_recon    weak-moment adjoint (eqs. (3.6)-(3.8)), limiter, back-transform,
//                  scalar HWENO, eigen-system and projection adjoints; stencil sums
//   k_adj_out      sums of the tiles' stencil shares and the adjoint of the ghost
//                  fill (Remark 4.1), written to the output
//   k_mu_sum       fixed-order sum of the mu-adjoint block partials

#include "hweno_adj.h"
#include "hweno_basis2.h"
#include "hweno_vjp.h"

namespace hw {

namespace {

constexpr int HALO = 4;

__device__ __forceinline__ double gw(int g) { return g == 1 ? GW1 : GW0; }
__device__ __forceinline__ double gx(int g) { return g == 0 ? -GS : (g == 1 ? 0.0 : GS); }

__device__ __forceinline__ bool interior(const Grid2& g, int j, int i) {
    return j >= HALO && j < HALO + g.ny && i >= HALO && i < HALO + g.nx;
}

// Whether face f (0 left, 1 right, 2 bottom, 3 top) of cell (j, i) is one of
// the faces k_adj_flux visits (the faces of the interior cells): its trace
// and gradient adjoints are then assigned there, and later kernels add to
// them; the other slots the later kernels assign (or read as zero), so the
// adjoint workspace needs no clearing.
__device__ __forceinline__ bool flux_face(const Grid2& g, int j, int i, int f) {
    if (f < 2) {
        if (j < HALO || j >= HALO + g.ny) return false;
        return f == 0 ? (i >= HALO && i <= HALO + g.nx) : (i >= HALO - 1 && i <= HALO + g.nx - 1);
    }
    if (i < HALO || i >= HALO + g.nx) return false;
    return f == 2 ? (j >= HALO && j <= HALO + g.ny) : (j >= HALO - 1 && j <= HALO + g.ny - 1);
}

// Solid cell of a masked grid (interior index t)
__device__ __forceinline__ bool solid_cell(const Grid2& g, long long t) {
    return g.solid && g.solid[t];
}

// residual adjoint of interior cell (j, i): F1, F2, F3 component c (on a
// masked grid the seeds come with the solid cells' zeroed, k_mask_seeds)
__device__ __forceinline__ double rbar(const AdjIn& A, const Grid2& g, int m, int c, int j, int i) {
    const long long nint = (long long)g.nx * g.ny;
    return A.rs * A.Rb[(m * 4 + c) * nint + (long long)(j - HALO) * g.nx + (i - HALO)];
}

// Logical index of this block: XCD-aware (each XCD takes a contiguous range
// of the launch, so neighbouring rows of a stencil share an L2), last first
// where bit k of W.rev is set (k: 0 face fluxes; 2 gradients; 3
// weak-moment gather; 5 reconstruction).
// The mu partials are stored by it, so their fixed summation order is
// unchanged.
__device__ __forceinline__ int lblock(const AdjWs& W, int k) {
    return xcd_block((int)blockIdx.x, (int)gridDim.x, (W.rev >> k) & 1u);
}

// fixed-order block sum of the mu adjoint: one partial per (logical) block;
// a butterfly within each wavefront, then the wavefronts' sums in order
template <int NT>
__device__ __forceinline__ void mu_partial(double v, double* part, int lb) {
    static_assert(NT % 64 == 0, "whole wavefronts");
    __shared__ double sh[NT / 64];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) s += sh[w];
        part[lb] = s;
    }
}

// ---------------------------------------------------------------------------
// Face fluxes: fhat = 1/2 (f(u-,s-) + f(u+,s+) - beta (u+ - u-)), beta the
// max over the face's 3 Gauss points x 2 sides of max(|u_n| + c, beta_PP).
// Block: 64 faces, a wavefront per side and Gauss point; the x-faces' blocks
// (W.mu_off1 of them), then the y-faces', in one launch.  With both sides in a
// thread (204 registers, two wavefronts per SIMD) and a launch per direction the
// two took 54 us on 256 x 256; now 48.
// ---------------------------------------------------------------------------
constexpr int AF = 64;

template <int d, bool VarMu>
__device__ __forceinline__ void adj_flux_body(const Grid2& g, const AdjIn& A, const AdjWs& W, int lb,
                                              double (*shs)[AF], double (*shu)[4][AF],
                                              double (*shb)[AF]) {
    const Consts& K = g.K;
    const int nfi = d == 0 ? g.nx + 1 : g.nx;
    const int nfj = d == 0 ? g.ny : g.ny + 1;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / AF);
    const int side = wv / 3, G = wv % 3;         // side 0: minus, 1: plus
    const int fl = threadIdx.x % AF;
    const long long t = (long long)lb * AF + fl;
    const bool valid = t < (long long)nfi * nfj;
    const long long N = g.ncell;
    int j = HALO, i = HALO;
    if (valid) {
        const int fj = (int)(t / nfi), fi = (int)(t % nfi);
        j = d == 0 ? HALO + fj : HALO - 1 + fj;
        i = d == 0 ? HALO - 1 + fi : HALO + fi;
    }
    const long long cm = (long long)j * g.NX + i;
    const int jp = d == 0 ? j : j + 1, ip = d == 0 ? i + 1 : i;
    const long long co = side ? (d == 0 ? cm + 1 : cm + g.NX) : cm;   // this side's cell
    const int po = side ? G : 3 + G;                                  // its face point
    const double* F = d == 0 ? g.xf : g.yf;
    const int pg = d == 0 ? 0 : 6;
    double U[4], s[6];
#pragma unroll
    for (int c = 0; c < 4; ++c) U[c] = F[(po * 4 + c) * N + co];
#pragma unroll
    for (int z = 0; z < 6; ++z) s[z] = g.gf[((pg + po) * 6 + z) * N + co];
    // adjoint of fhat at this Gauss point from the two adjacent residuals
    double fb[4] = {0.0, 0.0, 0.0, 0.0};
    if (valid) {
        const double w = gw(G), x = gx(G);
        const bool im = interior(g, j, i), ipn = interior(g, jp, ip);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double v = 0.0;
            if (d == 0) {
                if (im) v += -w * K.idx * rbar(A, g, 0, c, j, i) - 0.5 * w * K.idx * rbar(A, g, 1, c, j, i)
                             - w * x * K.idx * rbar(A, g, 2, c, j, i);
                if (ipn) v += w * K.idx * rbar(A, g, 0, c, jp, ip) - 0.5 * w * K.idx * rbar(A, g, 1, c, jp, ip)
                              + w * x * K.idx * rbar(A, g, 2, c, jp, ip);
            } else {
                if (im) v += -w * K.idy * rbar(A, g, 0, c, j, i) - w * x * K.idy * rbar(A, g, 1, c, j, i)
                             - 0.5 * w * K.idy * rbar(A, g, 2, c, j, i);
                if (ipn) v += w * K.idy * rbar(A, g, 0, c, jp, ip) + w * x * K.idy * rbar(A, g, 1, c, jp, ip)
                              - 0.5 * w * K.idy * rbar(A, g, 2, c, jp, ip);
            }
            fb[c] = v;
        }
    }
    const double sp = speed2<d>(K, U, s);
    shs[wv][fl] = valid ? sp : -INFINITY;
    if (side) {
#pragma unroll
        for (int c = 0; c < 4; ++c) shu[G][c][fl] = U[c];
    }
    __syncthreads();
    // beta and its argmax in the order (minus side G = 0,1,2, plus side G = 0,1,2)
    double beta = -INFINITY;
    int arg = 0;
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const double v = shs[q][fl];
        if (v > beta) {
            beta = v;
            arg = q;
        }
    }
    if (side == 0) {
        double betab = 0.0;
#pragma unroll
        for (int c = 0; c < 4; ++c) betab -= 0.5 * fb[c] * (shu[G][c][fl] - U[c]);
        shb[G][fl] = betab;
    }
    __syncthreads();
    double Ub[4], sb[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, hf[4];
    // the viscosity at the point: mu_ref, or mu(T) of the state, whose adjoint
    // is chained through T below
    const double mu = VarMu ? point_mu(K, U) : K.mu_ref;
    double mub = 0.0;
    const double hb = side ? -0.5 * beta : 0.5 * beta;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        hf[c] = 0.5 * fb[c];
        Ub[c] = hb * fb[c];
    }
    if (valid) {
        flux2_vjp<d>(K, U, s, mu, hf, Ub, sb, mub);
        if (arg == wv)
            speed2_vjp<d>(K, U, s, mu, shb[0][fl] + shb[1][fl] + shb[2][fl], Ub, sb, mub);
        if constexpr (VarMu) mub *= mu_T_vjp(K, U, mub, Ub);
        double* XB = d == 0 ? W.xfb : W.yfb;
#pragma unroll
        for (int c = 0; c < 4; ++c) XB[(po * 4 + c) * N + co] = Ub[c];
#pragma unroll
        for (int z = 0; z < 6; ++z) W.gfb[((pg + po) * 6 + z) * N + co] = sb[z];
    }
    mu_partial<6 * AF>(valid ? mub : 0.0, W.mupart + (d == 0 ? 0 : W.mu_off1), lb);
}

template <bool VarMu>
__global__ __launch_bounds__(6 * AF) void k_adj_flux(Grid2 g, AdjIn A, AdjWs W) {
    __shared__ double shs[6][AF];         // speeds
    __shared__ double shu[3][4][AF];      // states of the plus side
    __shared__ double shb[3][AF];         // beta-bar partial sums
    const int lb = lblock(W, 0);
    if (lb < W.mu_off1) adj_flux_body<0, VarMu>(g, A, W, lb, shs, shu, shb);
    else adj_flux_body<1, VarMu>(g, A, W, lb - W.mu_off1, shs, shu, shb);
}

// ---------------------------------------------------------------------------
// Gradient reconstruction (and, on interior cells, the volume fluxes).
// Block: 32 cells x 6 gradient components s = 2 w + l.
// ---------------------------------------------------------------------------
constexpr int AG = 32;

template <bool VarMu>
__global__ __launch_bounds__(6 * AG) void k_adj_grad(Grid2 g, AdjIn A, AdjWs W) {
    __shared__ double shv[6 * 9 * AG];       // forward volume gradients
    __shared__ double shvb[2][6 * 9 * AG];   // their adjoints from f and from g
    const Consts& K = g.K;
    const int tid = threadIdx.x;
    const int cl = tid % AG;
    const int s = tid / AG;
    const int w = s >> 1, l = s & 1;
    const int wc = g.NX - 6;
    const long long nreg = (long long)wc * (g.NY - 6);
    const int lb = lblock(W, 2);
    const long long cid = (long long)lb * AG + cl;
    const bool valid = cid < nreg;
    int j = 3, i = 3;
    if (valid) {
        j = 3 + (int)(cid / wc);
        i = 3 + (int)(cid % wc);
    }
    const long long N = g.ncell;
    const long long cell = (long long)j * g.NX + i;
    const double* R0 = g.rb + ((l * 3 + w) * 3 + 0) * N;
    const double* R1 = g.rb + ((l * 3 + w) * 3 + 1) * N;
    const double* R2 = g.rb + ((l * 3 + w) * 3 + 2) * N;
    double a[17];
#pragma unroll
    for (int q = 0; q < 9; ++q) a[q] = R0[cell + (long long)(q / 3 - 1) * g.NX + (q % 3 - 1)];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = 2 * e + 1;
        const long long nb = cell + (long long)(q / 3 - 1) * g.NX + (q % 3 - 1);
        a[9 + e] = R1[nb];
        a[13 + e] = R2[nb];
    }
    double C[15], vo[9];
    hweno2d(a, grad_consts(K), C);
    eval_vol(C, vo);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        shv[(s * 9 + q) * AG + cl] = vo[q];
        shvb[0][(s * 9 + q) * AG + cl] = 0.0;
        shvb[1][(s * 9 + q) * AG + cl] = 0.0;
    }
    __syncthreads();
    const bool inter = valid && interior(g, j, i);
    double mub = 0.0;
    if (inter) {
        // volume flux: vf = sum_q w_q f(U_q, s_q); vf-bar = F2-bar/dx (f), F3-bar/dy (g).
        // The 18 point adjoints over the cell's 6 threads: direction dv = s / 3,
        // points 3 (s % 3) .. 3 (s % 3) + 2
        const int dv = s / 3, q0 = 3 * (s % 3);
        double fb[4];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            fb[c] = dv == 0 ? rbar(A, g, 1, c, j, i) * K.idx : rbar(A, g, 2, c, j, i) * K.idy;
        const double* V = dv == 0 ? g.xv : g.yv;
        double* VB = dv == 0 ? W.xvb : W.yvb;
        for (int q = q0; q < q0 + 3; ++q) {
            const double wq = gw(q / 3) * gw(q % 3);
            double Uq[4], sq[6], Uqb[4] = {0.0, 0.0, 0.0, 0.0}, sqb[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            double f[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                Uq[c] = V[(q * 4 + c) * N + cell];
                f[c] = wq * fb[c];
            }
#pragma unroll
            for (int z = 0; z < 6; ++z) sq[z] = shv[(z * 9 + q) * AG + cl];
            const double muq = VarMu ? point_mu(K, Uq) : K.mu_ref;
            double mubq = 0.0;
            double& mb = VarMu ? mubq : mub;
            if (dv == 0) flux2_vjp<0>(K, Uq, sq, muq, f, Uqb, sqb, mb);
            else flux2_vjp<1>(K, Uq, sq, muq, f, Uqb, sqb, mb);
            if constexpr (VarMu) mub += mubq * mu_T_vjp(K, Uq, mubq, Uqb);
#pragma unroll
            for (int c = 0; c < 4; ++c) VB[(q * 4 + c) * N + cell] = Uqb[c];
#pragma unroll
            for (int z = 0; z < 6; ++z) shvb[dv][(z * 9 + q) * AG + cl] = sqb[z];
        }
    }
    __syncthreads();
    // adjoint of this component's 21 point values
    double yb[21];
#pragma unroll
    for (int p = 0; p < 12; ++p)
        yb[p] = flux_face(g, j, i, p / 3) ? g_ld(W.gfb, (p * 6 + s) * N + cell) : 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q)
        yb[12 + q] = shvb[0][(s * 9 + q) * AG + cl] + shvb[1][(s * 9 + q) * AG + cl];
    double Cb[15];
#pragma unroll
    for (int k = 0; k < 15; ++k) Cb[k] = 0.0;
    adj::xface_T(yb, Cb);
    adj::yface_T(yb + 6, Cb);
    adj::vol_T(yb + 12, Cb);
    double ab[17];
    hweno2d_vjp(a, grad_consts(K), Cb, ab);
    if (valid) {
#pragma unroll
        for (int k = 0; k < 17; ++k) W.rbc[(s * 17 + k) * N + cell] = ab[k];
    }
    mu_partial<6 * AG>(mub, W.mupart + W.mu_off2, lb);
}

// ---------------------------------------------------------------------------
// Gather of the weak-moment adjoints: cell X is slot k of the 3x3 stencil of
// cell X - off(k).  Cells of halo ring 2.
// ---------------------------------------------------------------------------
// One gradient component s = 2 w + l per thread (the grid's second index); the 17
// loads are unconditional (at the cell itself where the stencil's cell is not in
// ring 1) and issued together: with a branch per slot and all components in one
// thread the kernel took 25 us on 256 x 256.
__global__ void k_adj_rgather(Grid2 g, AdjWs W) {
    const int wc = g.NX - 4;
    const int nreg = wc * (g.NY - 4);
    const int cid = lblock(W, 3) * (int)blockDim.x + (int)threadIdx.x;
    if (cid >= nreg) return;
    const int j = 2 + cid / wc, i = 2 + cid % wc;
    const long long N = g.ncell;
    const int cell = j * g.NX + i;
    const int s = (int)blockIdx.y, w = s >> 1, l = s & 1;
    const double* P = W.rbc + (long long)s * 17 * N;
    double m0 = 0.0, m1 = 0.0, m2 = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const int ox = k % 3 - 1, oy = k / 3 - 1;
        const int yj = j - oy, yi = i - ox;
        const bool in = yj >= 3 && yj <= g.NY - 4 && yi >= 3 && yi <= g.NX - 4;   // ring 1
        const int Y = in ? yj * g.NX + yi : cell;
        const double x0 = P[k * N + Y];
        m0 += in ? x0 : 0.0;
        if (k & 1) {
            const int e = k >> 1;     // k = 1, 3, 5, 7 -> edge slot 0..3
            const double x1 = P[(9 + e) * N + Y], x2 = P[(13 + e) * N + Y];
            m1 += in ? x1 : 0.0;
            m2 += in ? x2 : 0.0;
        }
    }
    W.rbb[((l * 3 + w) * 3 + 0) * N + cell] = m0;
    W.rbb[((l * 3 + w) * 3 + 1) * N + cell] = m1;
    W.rbb[((l * 3 + w) * 3 + 2) * N + cell] = m2;
}

// Ring 2: the cells with weak moments.
__device__ __forceinline__ bool in_ring2(const Grid2& g, int j, int i) {
    return j >= 2 && j <= g.NY - 3 && i >= 2 && i <= g.NX - 3;
}

// ---------------------------------------------------------------------------
// Reconstruction adjoint: weak-moment shares of the point values (eqs.
// (3.6)-(3.8)), limiter, back-transform, scalar HWENO, eigen-system and
// projection adjoints of a tile of cells in one kernel.
// Block: AT_X x AT_Y cells, four wavefronts, one thread per cell in each, split
// as the forward kernel: wavefront (b, h) works in basis b on the fields
// {0, 3} (h = 0) or {1, 2} and owns the face points (h = 0) or the volume points
// of its basis, in the basis's (normal, tangential) coordinates.  It recomputes the
// point values, forms the cotangents of all four fields at its own points,
// hands the partner's two over in LDS and takes its own two back through
// the scalar reconstruction.  The stencil shares of the tile's cells are summed
// in LDS: in each of four phases a wavefront adds its share of one conserved
// component, so every sum has a fixed order, and the tile with its ring of one
// cell (20 doubles per cell) goes to the workspace for k_adj_out.
// Bound: the latency of two wavefronts per SIMD (256 registers, about 6000
// instructions each).  A thread per field in two kernels, which exchanged the
// point values through LDS and 160 cotangents per cell through memory, a
// weak-moment kernel that read and wrote all point cotangents (360 doubles per
// cell) and a gather of 136 stencil shares per cell took 77 + 92 + 48 + 18 us on
// 256 x 256; this kernel takes 100.  Tiles of 32 x 2 cells (a twelfth of their cells
// outside the grid there, 5 % more blocks) take 108, 8 x 8 112; 240 x 200: 71, 75
// and 81 us, 64 x 64: 27.8, 29.1 and 30.9.
// ---------------------------------------------------------------------------
constexpr int AT_X = 16, AT_Y = 4, AT_W = AT_X + 2, AT_H = AT_Y + 2, AT_P = AT_W * AT_H;

inline __host__ __device__ int at_tiles_x(const Grid2& g) { return (g.NX - 1 + AT_X - 1) / AT_X; }
inline __host__ __device__ int at_tiles_y(const Grid2& g) { return (g.NY - 2 + AT_Y - 1) / AT_Y; }

// Basis b's normal direction is x (b = 0) or y (b = 1): offset of stencil slot
// s in the tile and plane of the normal and tangential moment fields.
template <int b>
struct TileBasis {
    static constexpr int sn = b ? AT_W : 1, st = b ? 1 : AT_W;
    static constexpr int mn = b ? 8 : 4, mt = b ? 4 : 8;
    static constexpr int off(int s) { return (s % 3 - 1) * sn + (s / 3 - 1) * st; }
};

// Adjoint of row L = (left eigenvector of field f) of project2: Lb[c] = sum_s ab[s] *
// stencil datum (s, c).
template <int b>
__device__ __forceinline__ void project2_rowbar(const double* T0, const double* ab, double* Lb) {
    constexpr int cm[4] = {0, b ? 2 : 1, b ? 1 : 2, 3};
    using TB = TileBasis<b>;
#pragma unroll
    for (int c = 0; c < 4; ++c) Lb[c] = 0.0;
#pragma unroll
    for (int s = 0; s < 9; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) Lb[c] += ab[s] * T0[TB::off(s) + cm[c] * AT_P];
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            Lb[c] += ab[9 + e] * T0[TB::off(2 * e + 1) + (TB::mn + cm[c]) * AT_P] +
                     ab[13 + e] * T0[TB::off(2 * e + 1) + (TB::mt + cm[c]) * AT_P];
}

// Add v to an LDS word: no other wavefront touches it in this phase and the lanes
// of one call have words of their own, so the sums have the program's order.
__device__ __forceinline__ void lds_add(double* p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Share of a field (entry l of its row of L, input adjoints ab) in component G
// (global number) of the cell's stencil.
template <int b>
__device__ __forceinline__ void scatter2(double* A0, int G, double l, const double* ab) {
    using TB = TileBasis<b>;
#pragma unroll
    for (int s = 0; s < 9; ++s) lds_add(A0 + TB::off(s) + G * AT_P, l * ab[s]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        lds_add(A0 + TB::off(2 * e + 1) + (TB::mn + G) * AT_P, l * ab[9 + e]);
        lds_add(A0 + TB::off(2 * e + 1) + (TB::mt + G) * AT_P, l * ab[13 + e]);
    }
}

__global__ __launch_bounds__(256, 2) void k_adj_recon(Grid2 g, AdjIn A, AdjWs W,
                                                      const double* __restrict__ S) {
    constexpr int PL = AT_P;
    constexpr int NP = (PL + 63) / 64;
    constexpr int XB = 2 * (9 + 7) * 64;   // values at the partner's points: one field of each wavefront
    __shared__ double sh[2 * XB];
    __shared__ double tile[12 * PL];
    __shared__ double sums[12 * PL];       // the stencil sums
    __shared__ double shm[2][4][64];       // least [density, pressure] of a wavefront's points
    __shared__ int shi[2][4][64];          // and where (index in the oracle's point order)
    __shared__ double shl[4][64];          // rare: theta adjoints; conserved values at a point
    const Consts& K = g.K;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = wv >> 1, hh = wv & 1;
    const long long N = g.ncell;
    const int lb = lblock(W, 5);
    const int tiles_x = at_tiles_x(g);
    const int i0 = (lb % tiles_x) * AT_X, j0 = 1 + (lb / tiles_x) * AT_Y;
    const int lx = lane % AT_X, ly = lane / AT_X;
    const int i = i0 + lx, j = j0 + ly;
    const bool valid = i >= 1 && i <= g.NX - 2 && j <= g.NY - 2;
    const long long cell = valid ? (long long)j * g.NX + i : (long long)g.NX + 1;
    {
        double v[3][NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int t = lane + 64 * q, r = t / AT_W, c = t - r * AT_W;
            const int gj = min(j0 - 1 + r, g.NY - 1), gi = min(max(i0 - 1 + c, 0), g.NX - 1);
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if (t < PL) v[f][q] = S[(3 * wv + f) * N + (long long)gj * g.NX + gi];
        }
#pragma unroll
        for (int q = 0; q < NP; ++q)
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if (lane + 64 * q < PL) tile[(3 * wv + f) * PL + lane + 64 * q] = v[f][q];
    }
    for (int t = threadIdx.x; t < 12 * PL; t += 256) sums[t] = 0.0;
    __syncthreads();
    const int tc = (ly + 1) * AT_W + lx + 1;
    const double* T0 = tile + tc;
    const double rbar_ = T0[0];
    const double pbar = pressure2(K, rbar_, T0[PL], T0[2 * PL], T0[3 * PL]);
    const double mn = T0[(1 + b) * PL], mt = T0[(2 - b) * PL], Et = T0[3 * PL];
    const Basis2 e = basis2(K, rbar_, mn, mt, Et);
    // ---- forward: this wavefront's fields at its own points (last slot of
    // h = 0: 6 face values, then the moment), the rest to the partner ----
    double va[9], vb[9];
#pragma unroll 1
    for (int kk = 0; kk < 2; ++kk) {
        const int k = hh == 0 ? 3 * kk : 1 + kk;
        double C[15];
        {
            double L[4], R[4], a[17];
            field_rows(e, k, L, R);
            if (b == 0) project2<0, AT_W, PL>(T0, L, a);
            else project2<1, AT_W, PL>(T0, L, a);
            hweno2d(a, K, C);
        }
        double* X = sh + kk * XB + b * (XB / 2) + lane;
        double f[7], w[9];
        eval_xface(C, f);
        f[6] = moment_xi(C);
        eval_vol(C, w);
        if (hh == 0) {
#pragma unroll
            for (int q = 0; q < 9; ++q) X[q * 64] = w[q];
#pragma unroll
            for (int q = 0; q < 7; ++q) {
                va[q] = vb[q];
                vb[q] = f[q];
            }
        } else {
#pragma unroll
            for (int q = 0; q < 7; ++q) X[(9 + q) * 64] = f[q];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                va[q] = vb[q];
                vb[q] = w[q];
            }
        }
    }
    __syncthreads();
    double* XP = sh + b * (XB / 2) + lane;   // partner's values at own points: + kk * XB
    // the fields' values x and the conserved components u (basis order) at own
    // point o (h = 0: face points, then the moment; h = 1: volume points)
    auto point = [&](auto H, int o, double* x, double* u) {
#pragma clang fp contract(off)   // the same bits wherever it is formed
        if constexpr (H.value == 0) {
            x[0] = va[o];
            x[1] = XP[(9 + o) * 64];
            x[2] = XP[XB + (9 + o) * 64];
            x[3] = vb[o];
        } else {
            x[0] = XP[o * 64];
            x[1] = va[o];
            x[2] = vb[o];
            x[3] = XP[XB + o * 64];
        }
        const double sm = x[0] + x[3], df = x[3] - x[0];
        u[0] = sm + x[1];
        u[1] = fma(e.un, u[0], e.c * df);
        u[2] = fma(e.ut, u[0], x[2]);
        u[3] = fma(e.H, sm, fma(e.un * e.c, df, fma(0.5 * e.q2, x[1], e.ut * x[2])));
    };
    const int gc[4] = {0, 1 + b, 2 - b, 3};   // global number of a basis component
    auto gq = [&](int q) { return b ? 3 * (q % 3) + q / 3 : q; };
    // own point o in the order of the oracle's minima (ties go to the first)
    auto pidx = [&](auto H, int o) { return H.value == 0 ? b * 6 + o : 12 + b * 9 + gq(o); };
    const Part<0> face{};
    const Part<1> vol{};
    // ---- limiter forward: least density and pressure ----
    double th1 = 1.0, th2 = 1.0;
    double rmin = INFINITY, pmin = INFINITY;
    auto minima = [&](auto H) {
#pragma unroll
        for (int o = 0; o < H.points; ++o) {
            double x[4], u[4];
            point(H, o, x, u);
            rmin = fmin(rmin, u[0]);
            pmin = fmin(pmin, pressure2(K, u[0], u[1], u[2], u[3]));
        }
    };
    if (hh == 0) minima(face);
    else minima(vol);
    auto least = [&](int q) {
        return fmin(fmin(shm[q][0][lane], shm[q][1][lane]), fmin(shm[q][2][lane], shm[q][3][lane]));
    };
    shm[0][wv][lane] = rmin;
    shm[1][wv][lane] = pmin;
    __syncthreads();
    rmin = least(0);
    pmin = least(1);
    const double e1 = K.eps_pp <= rbar_ ? K.eps_pp : rbar_;
    const int esrc1 = K.eps_pp <= rbar_ ? 0 : 1;
    const double eps = e1 <= pbar ? e1 : pbar;
    const int esrc = e1 <= pbar ? esrc1 : 2;
    const bool low1 = rmin < eps;
    // ---- cotangents of the point values.  Loads are unconditional (a lane
    // outside the region reads cell (1, 1)) and what does not count is dropped ----
    const bool inter = valid && interior(g, j, i);
    const bool ring2 = valid && in_ring2(g, j, i);
    const double ih = b == 0 ? K.idx : K.idy;
    // weak-moment adjoint of variable w, moment mom of the cell or a neighbour
    auto RB = [&](int w, int mom, int off, bool in) {
        const double x = W.rbb[((b * 3 + w) * 3 + mom) * N + cell + off];
        return in ? x : 0.0;
    };
    // cotangents of (u_n, u_t, e): h = 0: of the lower (0) and upper face's
    // average and first moment; h = 1: of the cell average wbar
    double wa0[2][3], wa1[2][3];
#pragma unroll
    for (int z = 0; z < 3; ++z) {
        const int w = z == 2 ? 2 : (z == 0 ? b : 1 - b);
        const double ownm = RB(w, 1 + b, 0, ring2);   // the (W0+ + W0-) / 2 moment
        if (hh == 0) {
            const double own0 = RB(w, 0, 0, ring2);
            const double own1 = RB(w, 2 - b, 0, ring2);   // the transverse moment
#pragma unroll
            for (int hi = 0; hi < 2; ++hi) {
                const int s = 2 * hi - 1;
                const int off = b ? s * g.NX : s;
                const bool in = valid && in_ring2(g, b ? j + s : j, b ? i : i + s);
                const double nb0 = RB(w, 0, off, in), nbm = RB(w, 1 + b, off, in);
                const double nb1 = RB(w, 2 - b, off, in);
                wa0[hi][z] = 0.5 * ((s * (own0 - nb0) + 0.5 * (ownm + nbm)) * ih);
                wa1[hi][z] = 0.5 * (s * (own1 - nb1) * ih);
            }
        } else {
            wa0[0][z] = -ownm * ih;
        }
    }
    const double* PB = hh == 0 ? (b == 0 ? W.xfb : W.yfb) : (b == 0 ? W.xvb : W.yvb);
    const bool facelo = valid && flux_face(g, j, i, 2 * b), facehi = valid && flux_face(g, j, i, 2 * b + 1);
    // cotangent of the (limited) value ul at own point o
    auto cot = [&](auto H, int o, const double* ul, double* yb) {
        double wb[3];
        if constexpr (H.value == 0) {
            const int hi = o / 3, G = o % 3;
            const bool add = hi ? facehi : facelo;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double x = PB[(o * 4 + gc[c]) * N + cell];
                yb[c] = add ? x : 0.0;
            }
#pragma unroll
            for (int z = 0; z < 3; ++z) wb[z] = gw(G) * (wa0[hi][z] + gx(G) * wa1[hi][z]);
            adj::prim2_vjp(ul, wb, yb);
        } else {
            double z4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int z = 0; z < 3; ++z) wb[z] = gw(o / 3) * gw(o % 3) * wa0[0][z];
            adj::prim2_vjp(ul, wb, z4);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double x = PB[(gq(o) * 4 + gc[c]) * N + cell];
                yb[c] = (ring2 ? z4[c] : 0.0) + (inter ? x : 0.0);
            }
        }
    };
    // limited face value ul (u1: at the limited density) from the unlimited u
    const double ub[4] = {rbar_, mn, mt, Et};
    bool acted = false;
    auto limit = [&](const double* u, double* u1, double* ul) {
        u1[0] = acted ? rbar_ + th1 * (u[0] - rbar_) : u[0];
#pragma unroll
        for (int c = 1; c < 4; ++c) u1[c] = u[c];
#pragma unroll
        for (int c = 0; c < 4; ++c) ul[c] = acted ? ub[c] + th2 * (u1[c] - ub[c]) : u[c];
    };
    // where the limiter acts, the adjoints of its thetas go to the cell average
    // and to the points that set them (id1: density, id2: pressure); every
    // wavefront holds the same cells and minima, so the whole block takes the
    // branch or none of it
    double P1b = 0.0, P2b[4] = {0.0, 0.0, 0.0, 0.0};
    int id1 = -1, id2 = -1;
    double ctr[4] = {0.0, 0.0, 0.0, 0.0};     // cell-average adjoint (basis order)
    const bool rare = __ballot(valid && (low1 || pmin < eps)) != 0;
    if (rare) {
        if (low1) th1 = (rbar_ - eps) / (rbar_ - rmin);
        auto lower = [](double v, int id, double& m, int& im) {
            if (v < m || (v == m && id < im)) {
                m = v;
                im = id;
            }
        };
        double m1 = INFINITY, m2 = INFINITY;   // density; pressure at the limited densities
        int n1 = 1 << 30, n2 = 1 << 30;
        auto where = [&](auto H) {
#pragma unroll
            for (int o = 0; o < H.points; ++o) {
                double x[4], u[4];
                point(H, o, x, u);
                lower(u[0], pidx(H, o), m1, n1);
                lower(pressure2(K, low1 ? rbar_ + th1 * (u[0] - rbar_) : u[0], u[1], u[2], u[3]),
                      pidx(H, o), m2, n2);
            }
        };
        if (hh == 0) where(face);
        else where(vol);
        __syncthreads();                       // the minima have been read
        shm[0][wv][lane] = m1;
        shm[1][wv][lane] = m2;
        shi[0][wv][lane] = n1;
        shi[1][wv][lane] = n2;
        __syncthreads();
        int irmin = 1 << 30, ipmin = 1 << 30;
        rmin = pmin = INFINITY;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            lower(shm[0][w][lane], shi[0][w][lane], rmin, irmin);
            lower(shm[1][w][lane], shi[1][w][lane], pmin, ipmin);
        }
        const bool low2 = pmin < eps && (pbar - eps) / (pbar - pmin) < 1.0;
        if (low2) th2 = (pbar - eps) / (pbar - pmin);
        acted = low1 || low2;
        double t1 = 0.0, t2 = 0.0;
        auto thetas = [&](auto H) {
#pragma unroll
            for (int o = 0; o < H.points; ++o) {
                double x[4], u[4];
                point(H, o, x, u);
                if constexpr (H.value == 0) {
                    double u1[4], ul[4], yb[4];
                    limit(u, u1, ul);
                    cot(H, o, ul, yb);
                    t1 += th2 * yb[0] * (u[0] - rbar_);
#pragma unroll
                    for (int c = 0; c < 4; ++c) t2 += yb[c] * (u1[c] - ub[c]);
                }
                if (low2 && pidx(H, o) == ipmin) {   // in global order
#pragma unroll
                    for (int c = 0; c < 4; ++c) shl[gc[c]][lane] = u[c];
                }
            }
        };
        if (hh == 0) thetas(face);
        else thetas(vol);
        __syncthreads();
        if (hh == 0) {
            shm[0][b][lane] = t1;
            shm[0][2 + b][lane] = t2;
        }
        __syncthreads();
        double T1b = shm[0][0][lane] + shm[0][1][lane];
        const double T2b = shm[0][2][lane] + shm[0][3][lane];
        double rb_ = 0.0, pb_ = 0.0, epsb = 0.0;
        if (low2) {
            const double rho = shl[0][lane];
            const double Ut[4] = {rbar_ + th1 * (rho - rbar_), shl[1][lane], shl[2][lane],
                                  shl[3][lane]};
            const double den = pbar - pmin;
            pb_ += T2b * (eps - pmin) / (den * den);
            epsb += -T2b / den;
            double Utb[4] = {0.0, 0.0, 0.0, 0.0};
            adj::pres2_vjp(K, Ut, T2b * (pbar - eps) / (den * den), Utb);
            rb_ += Utb[0] * (1.0 - th1);
            P2b[0] = Utb[0] * th1;
            P2b[1] = b ? Utb[2] : Utb[1];
            P2b[2] = b ? Utb[1] : Utb[2];
            P2b[3] = Utb[3];
            T1b += Utb[0] * (rho - rbar_);
            id2 = ipmin;
        }
        if (low1) {
            const double den = rbar_ - rmin;
            rb_ += T1b * (eps - rmin) / (den * den);
            epsb += -T1b / den;
            P1b = T1b * (rbar_ - eps) / (den * den);
            id1 = irmin;
        }
        if (esrc == 1) rb_ += epsb;
        if (esrc == 2) pb_ += epsb;
        if (wv == 0) {
            ctr[0] = rb_;
            if (pb_ != 0.0) adj::pres2_vjp(K, ub, pb_, ctr);
        }
    }
    // ---- point cotangents to field cotangents: own two kept, the partner's two
    // in place of its values; sums for the eigenvectors' adjoint ----
    PointSums2 pts;
    auto back = [&](auto H, auto Rare) {
#pragma unroll
        for (int o = 0; o < H.slots; ++o) {
            double x[4], u[4], y[4];
            point(H, o, x, u);
            if (o == H.points) {     // the own-cell moment
                const long long nint = (long long)g.nx * g.ny;
                const long long t = inter ? (long long)(j - HALO) * g.nx + (i - HALO) : 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double s = A.Vb ? A.vs * A.Vb[(b * 4 + gc[c]) * nint + t] : 0.0;
                    y[c] = inter ? s : 0.0;
                }
            } else if constexpr (Rare.value == 0) {
                cot(H, o, u, y);
            } else {
                double u1[4], ul[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) ul[c] = u[c];
                if constexpr (H.value == 0) limit(u, u1, ul);
                cot(H, o, ul, y);
                if constexpr (H.value == 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const double th = c == 0 ? th2 * th1 : th2;
                        ctr[c] += acted ? y[c] * (1.0 - th) : 0.0;
                        y[c] = acted ? y[c] * th : y[c];
                    }
                }
                if (pidx(H, o) == id1) y[0] += P1b;
                if (pidx(H, o) == id2)
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] += P2b[c];
            }
            double z[4];
            cons2_vjp(e, x, y, pts, z);
            if constexpr (H.value == 0) {
                va[o] = z[0];
                vb[o] = z[3];
                XP[(9 + o) * 64] = z[1];
                XP[XB + (9 + o) * 64] = z[2];
            } else {
                va[o] = z[1];
                vb[o] = z[2];
                XP[o * 64] = z[0];
                XP[XB + o * 64] = z[3];
            }
        }
    };
    if (rare) {
        if (hh == 0) back(face, Part<1>{});
        else back(vol, Part<1>{});
    } else {
        if (hh == 0) back(face, Part<0>{});
        else back(vol, Part<0>{});
    }
    __syncthreads();
    // ---- scalar reconstruction, projection row and eigenvector adjoints ----
    Basis2Bar eb(e, pts);
    double* A0 = sums + tc;
    auto component = [&](int G) { return b == 1 && (G == 1 || G == 2) ? 3 - G : G; };
    auto sel = [](int c, const double* v) {
        return c == 0 ? v[0] : (c == 1 ? v[1] : (c == 2 ? v[2] : v[3]));
    };
#pragma unroll 1
    for (int kk = 0; kk < 2; ++kk) {
        const int k = hh == 0 ? 3 * kk : 1 + kk;
        double Cb[15];
#pragma unroll
        for (int q = 0; q < 15; ++q) Cb[q] = 0.0;
        {
            const double* X = XP + kk * XB;
            double y[16];
            if (hh == 0) {
#pragma unroll
                for (int q = 0; q < 7; ++q) y[q < 6 ? q : 15] = kk ? vb[q] : va[q];
#pragma unroll
                for (int q = 0; q < 9; ++q) y[6 + q] = X[q * 64];
            } else {
#pragma unroll
                for (int q = 0; q < 7; ++q) y[q < 6 ? q : 15] = X[(9 + q) * 64];
#pragma unroll
                for (int q = 0; q < 9; ++q) y[6 + q] = kk ? vb[q] : va[q];
            }
            adj::xface_T(y, Cb);
            adj::vol_T(y + 6, Cb);
            moment_xi_T(y[15], Cb);
        }
        double L[4], R[4], a[17], ab[17], Lb[4];
        field_rows(e, k, L, R);
        if (b == 0) project2<0, AT_W, PL>(T0, L, a);
        else project2<1, AT_W, PL>(T0, L, a);
        hweno2d_vjp(a, K, Cb, ab);
        if (b == 0) project2_rowbar<0>(T0, ab, Lb);
        else project2_rowbar<1>(T0, ab, Lb);
        row2_vjp(e, k, Lb, eb);
#pragma unroll 1
        for (int ph = 0; ph < 4; ++ph) {
            const int G = (wv + ph) & 3;
            const double l = sel(component(G), L);
            if (valid) {
                if (b == 0) scatter2<0>(A0, G, l, ab);
                else scatter2<1>(A0, G, l, ab);
            }
            __syncthreads();
        }
    }
    basis2_vjp(K, e, rbar_, mn, mt, Et, pts.a5, eb, ctr);
#pragma unroll 1
    for (int ph = 0; ph < 4; ++ph) {
        const int G = (wv + ph) & 3;
        if (valid) lds_add(A0 + G * PL, sel(component(G), ctr));
        __syncthreads();
    }
    double* out = W.uc + (long long)lb * (12 * PL);
    for (int t = threadIdx.x; t < 12 * PL; t += 256) out[t] = sums[t];
}

// State adjoint of ghosted cell (j, i), component q: the sums of the tiles that
// hold the cell (each tile its ring of one cell too), in a fixed order.
__device__ __forceinline__ double state_bar(const Grid2& g, const AdjWs& W, int q, int j, int i) {
    const int ntx = at_tiles_x(g), nty = at_tiles_y(g);
    const int t1 = j / AT_Y, x1 = i / AT_X, xr = i % AT_X;
    double v = 0.0;
#pragma unroll
    for (int d = 1; d >= 0; --d) {
        const int ty = t1 - d;
        if (ty < 0 || ty >= nty || (d && j % AT_Y >= 2)) continue;
        const double* R = W.uc + ((long long)ty * ntx * 12 + q) * AT_P + (j % AT_Y + AT_Y * d) * AT_W;
        auto T = [&](int tx) { return R[(long long)tx * (12 * AT_P) + i - tx * AT_X + 1]; };
        if (xr == 0 && x1 > 0) v += T(x1 - 1);
        if (x1 < ntx) v += T(x1);
        if (xr == AT_X - 1 && x1 + 1 < ntx) v += T(x1 + 1);
    }
    return v;
}
static_assert(AT_Y >= 2, "state_bar: a row lies in at most two tiles");

// ---------------------------------------------------------------------------
// Adjoint of the ghost fill: the y sweep is undone first (its sources include
// the x-ghost columns), then the x sweep.  Each source cell gathers the
// ghost cells copied from it, in a fixed order.
// ---------------------------------------------------------------------------
// The ghost rows (columns) of one side that copy interior row r of n: first one
// and count (outflow copies the boundary row to all of them, the other kinds map
// one to one as n >= HALO).
__device__ __forceinline__ int ghosts_of(int kind, int side, int r, int n, int* count) {
    const int first = side ? HALO + n : 0;          // the side's ghost rows: HALO from here
    if (kind == 1) {
        *count = r == (side ? HALO + n - 1 : HALO) ? HALO : 0;
        return first;
    }
    const int gj = kind == 0 ? (side ? r + n : r - n)
                             : (side ? 2 * (HALO + n) - 1 - r : 2 * HALO - 1 - r);
    *count = kind != 2 && gj >= first && gj < first + HALO ? 1 : 0;   // inflow: constant
    return gj;
}

// Component q of the adjoint at cell (r, i) of an interior row once the y
// sweep is undone: its own value plus the ghost rows copied from it.
__device__ __forceinline__ double ghost_y_gather(const Grid2& g, const AdjWs& W, int q, int r,
                                                 int i) {
    double v = state_bar(g, W, q, r, i);
    if (r >= 2 * HALO && r < g.ny) return v;
    for (int side = 0; side < 2; ++side) {
        const Side& sd = g.side[2 + side];
        int n;
        const int gj = ghosts_of(sd.kind, side, r, g.ny, &n);
        for (int d = 0; d < n; ++d) v += sd.sign[q] * state_bar(g, W, q, gj + d, i);
    }
    return v;
}

// Both sweeps undone for interior cell (j, c0), component q, written to the
// caller's interior array: the y sweep's gather at the cell, then the x
// ghost columns copied from it, each with its own y sweep's gather (the
// corner ghost cells reach the interior through the x-ghost columns).
// Component q is the grid's second index.
__global__ void k_adj_out(Grid2 g, AdjWs W, double* __restrict__ Ubar,
                          const double* __restrict__ add, double add_a,
                          const double* __restrict__ pass) {
    const unsigned nint = (unsigned)g.nx * (unsigned)g.ny;
    const unsigned r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nint) return;
    const int q = (int)blockIdx.y;
    const long long t = (long long)q * nint + r;
    const int j = HALO + (int)(r / (unsigned)g.nx), c0 = HALO + (int)(r % (unsigned)g.nx);
    // a stage's direct term: fluid cells (averages) or, on a masked grid,
    // solid cells (every component: a stage leaves them at its filled input)
    const bool sol = solid_cell(g, r);
    double v = ghost_y_gather(g, W, q, j, c0);
    // every ghost cell copies one of the HALO cells next to a side
    if (c0 < 2 * HALO || c0 >= g.nx) {
        for (int side = 0; side < 2; ++side) {
            const Side& sd = g.side[side];
            int n;
            const int gi = ghosts_of(sd.kind, side, c0, g.nx, &n);
            for (int d = 0; d < n; ++d) v += sd.sign[q] * ghost_y_gather(g, W, q, j, gi + d);
        }
    }
    if (sol) {
        if (pass) v += pass[t];
    } else if (add && q < 4) {
        v += add_a * add[t];
    }
    Ubar[t] = v;
}

// Seeds of a masked grid with the solid cells' entries zeroed (solid cells
// carry no residual and no modified moments): the residual seed into rbm (12
// per cell), the modified-moment seed (if any) into vbm (8 per cell).
__global__ void k_mask_seeds(Grid2 g, AdjWs W, const double* __restrict__ Rb,
                             const double* __restrict__ Vb) {
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nint * 20) return;
    const int q = (int)(t / nint);
    const long long r = t % nint;
    const bool sol = g.solid[r] != 0;
    if (q < 12) W.rbm[t] = sol ? 0.0 : Rb[t];
    else if (Vb) W.vbm[t - 12 * nint] = sol ? 0.0 : Vb[t - 12 * nint];
}

// Adjoint of the mirror fill of a masked grid's solid cells (k_solid2):
// each mirror source gathers sign * adjoint of the solid cells copied from it
// (in the list's order), then every listed solid cell's adjoint is zero (its
// value was overwritten).  Ubar in the interior layout.
__global__ void k_adj_solid_gather(Grid2 g, AdjWs W, double* __restrict__ Ubar) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)W.nsrc * 12) return;
    const int u = (int)(t / 12), q = (int)(t % 12);
    const int m = q / 4, c = q % 4;
    const long long nint = (long long)g.nx * g.ny;
    auto interior = [&](int gi) -> long long {
        return (long long)(gi / g.NX - HALO) * g.nx + (gi % g.NX - HALO);
    };
    const long long s = interior(W.ssrcu[u]);
    double acc = Ubar[q * nint + s];
    for (int k = W.sstart[u]; k < W.sstart[u + 1]; ++k) {
        const int e = W.sord[k];
        const int dir = g.sdir[e];
        const bool vel = g.solid_wall == 4 ? (c == 1 || c == 2) : (c == 1 + dir);
        const bool mom = m == 1 + dir;
        const double sg = (vel != mom) ? -1.0 : 1.0;
        acc += sg * Ubar[q * nint + interior(g.sdst[e])];
    }
    Ubar[q * nint + s] = acc;
}

__global__ void k_adj_solid_zero(Grid2 g, double* __restrict__ Ubar) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long long)g.nsolid * 12) return;
    const int e = (int)(t / 12), q = (int)(t % 12);
    const int gi = g.sdst[e];
    const long long nint = (long long)g.nx * g.ny;
    Ubar[q * nint + (long long)(gi / g.NX - HALO) * g.nx + (gi % g.NX - HALO)] = 0.0;
}

// mu-bar = fixed-order sum of the block partials (added to *out if acc)
__global__ __launch_bounds__(256) void k_mu_sum(const double* part, int n, double* out, int acc) {
    __shared__ double sh[256];
    const int t = threadIdx.x;
    // each thread sums its partials q = t, t + 256, ... in order; the loads
    // of eight of them are issued together
    double s = 0.0;
    int q = t;
    for (; q + 7 * 256 < n; q += 8 * 256) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = part[q + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    for (; q < n; q += 256) s += part[q];
    sh[t] = s;
    __syncthreads();
    // pairwise tree in a fixed order
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) sh[t] += sh[t + w];
        __syncthreads();
    }
    if (t == 0) *out = acc ? *out + sh[0] : sh[0];
}

__global__ void k_axpy(double* __restrict__ y, const double* __restrict__ x, double a, long long n) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] += a * x[t];
}

__global__ void k_lin3(double* __restrict__ y, const double* __restrict__ u, double a, double b,
                       const double* __restrict__ x, long long n) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) y[t] = a * u[t] + b * y[t] + x[t];
}

inline unsigned nb2(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

size_t adj_tile_doubles2(const Grid2& g) {
    return (size_t)at_tiles_x(g) * at_tiles_y(g) * (12 * AT_P);
}

long long adj_mu_partials2(const Grid2& g) {
    return (long long)nb2((long long)(g.nx + 1) * g.ny, AF) + nb2((long long)g.nx * (g.ny + 1), AF) +
           nb2((long long)(g.NX - 6) * (g.NY - 6), AG);
}

hipError_t launch_vjp2(const Grid2& g, const AdjIn& A0, AdjWs W, const double* S, double* Ubar,
                       double* mu_out, int mu_acc, hipStream_t st, const double* add,
                       double add_a, const double* pass) {
    const unsigned bx = nb2((long long)(g.nx + 1) * g.ny, AF);
    const unsigned by = nb2((long long)g.nx * (g.ny + 1), AF);
    const unsigned bg = nb2((long long)(g.NX - 6) * (g.NY - 6), AG);
    W.mu_off1 = bx;
    W.mu_off2 = bx + by;
    // the reconstruction adjoint walks its blocks last first, opposite to the
    // kernels before it (1.5 % of a step adjoint on 256^2; the other kernels
    // showed no gain)
    W.rev = 1u << 5;
    AdjIn A = A0;
    if (g.solid) {   // masked grid: the solid cells' seeds zeroed once, for every kernel
        k_mask_seeds<<<nb2((long long)g.nx * g.ny * 20, 256), 256, 0, st>>>(g, W, A0.Rb, A0.Vb);
        A.Rb = W.rbm;
        A.Vb = A0.Vb ? W.vbm : nullptr;
    }
    if (g.K.mu_exp != 0.0) {   // mu(T): the viscosity's dependence on the state too
        k_adj_flux<true><<<bx + by, 6 * AF, 0, st>>>(g, A, W);
        k_adj_grad<true><<<bg, 6 * AG, 0, st>>>(g, A, W);
    } else {
        k_adj_flux<false><<<bx + by, 6 * AF, 0, st>>>(g, A, W);
        k_adj_grad<false><<<bg, 6 * AG, 0, st>>>(g, A, W);
    }
    const dim3 br(nb2((long long)(g.NX - 4) * (g.NY - 4), 256), 6);
    k_adj_rgather<<<br, 256, 0, st>>>(g, W);
    k_adj_recon<<<(unsigned)(at_tiles_x(g) * at_tiles_y(g)), 256, 0, st>>>(g, A, W, S);
    const dim3 bo(nb2((long long)g.nx * g.ny, 256), 12);
    k_adj_out<<<bo, 256, 0, st>>>(g, W, Ubar, add, add_a, pass);
    if (g.nsolid > 0) {   // masked grid: the mirror fill, undone
        if (W.nsrc > 0)
            k_adj_solid_gather<<<nb2((long long)W.nsrc * 12, 256), 256, 0, st>>>(g, W, Ubar);
        k_adj_solid_zero<<<nb2((long long)g.nsolid * 12, 256), 256, 0, st>>>(g, Ubar);
    }
    k_mu_sum<<<1, 256, 0, st>>>(W.mupart, (int)(bx + by + bg), mu_out, mu_acc);
    return hipGetLastError();
}

hipError_t launch_axpy(double* y, const double* x, double a, long long n, hipStream_t st) {
    if (n > 0) k_axpy<<<nb2(n, 256), 256, 0, st>>>(y, x, a, n);
    return hipGetLastError();
}

hipError_t launch_lin3(double* y, const double* u, double a, double b, const double* x, long long n,
                       hipStream_t st) {
    if (n > 0) k_lin3<<<nb2(n, 256), 256, 0, st>>>(y, u, a, b, x, n);
    return hipGetLastError();
}

}  // namespace hw
