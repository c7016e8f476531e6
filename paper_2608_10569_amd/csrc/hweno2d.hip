// 2D HWENO-GR residual and SSP-RK3 stage update (Sec. 3 of arXiv 2608.10569)
// as a pipeline of HIP kernels over a ghosted structure-of-arrays grid.
//
//   ghost            : halo of width 4 (Remark 4.1; small launches form these
//                      cells in the reconstruction's loads instead)
//   recon            : characteristic HWENO in the x- and y-bases (eq. (3.4)),
//                      positivity limiter on the face values, wbar, hat-v/w,
//                      CFL wave speed                 [cells of halo ring 3]
//   rgrad            : interface averages, face moments, weak-derivative
//                      moments (eqs. (3.6)-(3.8)) of a tile of cells and the
//                      ring around it in LDS, then gradient HWENO (eq. (3.9)) at
//                      12 face + 9 volume points and the volume-flux
//                      quadratures                     [halo ring 1]
//   rbar, grad       : the same as two kernels for the reverse mode, which reads
//                      the weak moments from memory    [halo rings 2, 1]
//   recon_dr         : HWENO-DR's recon, with the gradients and volume fluxes
//   flux_x, flux_y   : PP Lax-Friedrichs fluxes at face Gauss points (eq. (3.3))
//   update           : assembly of eq. (3.2) and the stage combination of the
//                      SSP-RK3 scheme with modified moments (eq. (2.12))
//   fluxup           : flux_x + flux_y + update in one kernel per tile of
//                      cells, the face fluxes kept in LDS (the default; the
//                      three kernels apart are a tile choice)
//
// Every other intermediate lives in HBM, laid out component-major over the
// ghosted grid so that consecutive lanes touch consecutive cells.

#include <hip/hip_ext.h>

#include <mutex>

#include "hweno_basis2.h"
#include "hweno_kernels.h"

namespace hw {

namespace {

constexpr int HALO = 4;

// Wavefront maximum / minimum by data-parallel-primitive moves (row shifts by
// 1, 2, 4, 8, then the row broadcasts; lanes without a source keep their own
// value), read from lane 63.  Every lane of the wavefront takes part.  The
// cross-lane moves cost a few cycles where a shuffle through LDS takes over a
// hundred, six times in a row at the end of a block.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = (int)b, hi = (int)(b >> 32);
    const int l = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
    const int h = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)h << 32) | (unsigned)l);
}
__device__ __forceinline__ double lane63(double v) {
    const long long b = __double_as_longlong(v);
    const int l = __builtin_amdgcn_readlane((int)b, 63);
    const int h = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)h << 32) | (unsigned)l);
}
__device__ __forceinline__ double wave_max(double v) {
    v = fmax(v, dpp_move<0x111, 0xf>(v));
    v = fmax(v, dpp_move<0x112, 0xf>(v));
    v = fmax(v, dpp_move<0x114, 0xf>(v));
    v = fmax(v, dpp_move<0x118, 0xf>(v));
    v = fmax(v, dpp_move<0x142, 0xa>(v));
    v = fmax(v, dpp_move<0x143, 0xc>(v));
    return lane63(v);
}
__device__ __forceinline__ double wave_min(double v) {
    v = fmin(v, dpp_move<0x111, 0xf>(v));
    v = fmin(v, dpp_move<0x112, 0xf>(v));
    v = fmin(v, dpp_move<0x114, 0xf>(v));
    v = fmin(v, dpp_move<0x118, 0xf>(v));
    v = fmin(v, dpp_move<0x142, 0xa>(v));
    v = fmin(v, dpp_move<0x143, 0xc>(v));
    return lane63(v);
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Block-level reductions: wave shuffles, then LDS across the block's waves;
// thread 0 issues at most one atomic, and only when it can change the slot.
template <int NT>
__device__ __forceinline__ void red_max(unsigned long long* slot, double v) {
    __shared__ double sh[NT / 64];
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) v = fmax(v, sh[w]);
        const unsigned long long k = dkey(v);
        if (v > -INFINITY && k > *(volatile HW_GLOBAL unsigned long long*)slot) atomicMax(slot, k);
    }
}
// The reductions of an update kernel in one pass: the largest LF coefficient,
// and with `stage` (a stage update) the least density and pressure and the
// inadmissible cells.  Threads 0..2 each look at their slot and issue an
// atomic only if it would change it (the three looks overlap; looking at the
// kernel's start instead finds stale values and costs far more atomics than
// it hides).
template <int NT>
__device__ __forceinline__ void reduce_update(Reduce HW_GLOBAL* red, int stage, double bmax,
                                              double rmin, double pmin, bool bad) {
    constexpr int NW = NT / 64;
    __shared__ double sh[3][NW];
    __shared__ unsigned int shn[NW];
    const int w = threadIdx.x >> 6;
    const double b = wave_max(bmax), r = wave_min(rmin), p = wave_min(pmin);
    const unsigned int n = (unsigned int)__popcll(__ballot(bad));
    if ((threadIdx.x & 63) == 0) {
        sh[0][w] = b;
        sh[1][w] = r;
        sh[2][w] = p;
        shn[w] = n;
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 3) {
        double v = sh[t][0];
#pragma unroll
        for (int q = 1; q < NW; ++q) v = t == 0 ? fmax(v, sh[t][q]) : fmin(v, sh[t][q]);
        const unsigned long long k = dkey(v);
        HW_GLOBAL unsigned long long* s =
            t == 0 ? &red->beta_key : (t == 1 ? &red->min_rho_key : &red->min_p_key);
        const unsigned long long slot = *(volatile HW_GLOBAL unsigned long long*)s;
        if (t == 0) {
            if (v > -INFINITY && k > slot) atomicMax((unsigned long long*)s, k);
        } else if (stage > 0 && v < INFINITY && k < slot) {
            atomicMin((unsigned long long*)s, k);
        }
    } else if (t == 3 && stage > 0) {
        unsigned int v = 0;
#pragma unroll
        for (int q = 0; q < NW; ++q) v += shn[q];
        if (v) atomicAdd((unsigned int*)&red->bad[stage], v);
    }
}
template <int NT>
__device__ __forceinline__ void red_add32(unsigned int* slot, unsigned int v) {
    __shared__ unsigned long long sh[NT / 64];
    unsigned long long s = wave_sum((unsigned long long)v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) s += sh[w];
        if (s) atomicAdd(slot, (unsigned int)s);
    }
}

// Slot of the instance that owns this block and the block's index within it
// (uniform per block: binary search of the launch's block prefix table).
struct Loc {
    int p, b;
};
__device__ __forceinline__ Loc locate(const Batch& B) {
    const int nb = (int)gridDim.x;
    const int bid = B.xcd ? xcd_block((int)blockIdx.x, nb, B.rev)
                          : (B.rev ? nb - 1 - (int)blockIdx.x : (int)blockIdx.x);
    int lo = 0, hi = B.n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (B.start[mid] <= bid) lo = mid;
        else hi = mid;
    }
    return Loc{lo, bid - B.start[lo]};
}

// ---------------------------------------------------------------------------
// Ghost cells (Remark 4.1).  The x rule fills the ghost columns of interior
// rows and the y rule every column of the ghost rows; a corner cell takes the
// y rule applied to the value the x rule gives the ghost cell of its source
// row (what an x sweep followed by a y sweep would leave), so one launch
// fills the whole halo.
// ---------------------------------------------------------------------------
// Source of ghost index gi (0..HALO-1 below the interior, HALO+n.. above)
// along a direction with n interior cells: the periodic image, the boundary
// cell (outflow) or the mirror cell (walls).
__device__ __forceinline__ int ghost_src(int kind, int gi, int n) {
    if (gi < HALO) {
        const int d = HALO - gi;   // distance from the boundary
        return kind == 0 ? HALO + n - d : (kind == 1 ? HALO : HALO + d - 1);
    }
    const int d = gi - (HALO + n - 1);
    return kind == 0 ? HALO + d - 1 : (kind == 1 ? HALO + n - 1 : HALO + n - d);
}

// Inflow: the prescribed average of boundary cell k (of n along the side;
// the stage's profile when the fill names a stage), zero moments.
__device__ __forceinline__ void inflow_values(const Side& sd, int k, int n, int stage, double* v) {
    const double* st = (stage >= 0 && sd.prof_stage) ? sd.prof_stage + 4 * (stage * n + k)
                       : sd.prof                      ? sd.prof + 4 * k
                                                      : sd.inflow;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        v[c] = st[c];
        v[4 + c] = 0.0;
        v[8 + c] = 0.0;
    }
}

// Value the x rule of side sd gives ghost column i of interior row j.
__device__ __forceinline__ void x_ghost(const Grid2& g, const Side& sd, const double* S, int j,
                                        int i, int stage, double* v) {
    if (sd.kind == 2) {
        inflow_values(sd, j - HALO, g.ny, stage, v);
        return;
    }
    const long long src = (long long)j * g.NX + ghost_src(sd.kind, i, g.nx);
#pragma unroll
    for (int q = 0; q < 12; ++q) v[q] = sd.sign[q] * S[q * g.ncell + src];
}

__device__ __forceinline__ double flip_sign(double v, unsigned neg) {
    return __hiloint2double(__double2hiint(v) ^ (int)(neg << 31), __double2loint(v));
}

// Prescribed average of ghost cell (j, i) whose rules lead to an inflow side
// (its first moments are zero); gs: the descriptor in memory.
__device__ __forceinline__ void inflow_at(const Grid2& gs, int j, int i, int stage, double* st) {
    const bool yg = j < HALO || j >= HALO + gs.ny;
    const Side& sy = gs.side[j < HALO ? 2 : 3];
    const Side& sx = gs.side[i < HALO ? 0 : 1];
    const bool y = yg && sy.kind == 2;
    // on a y side the ghost columns take the profile's end states; on an x side
    // the ghost rows take their source row's, with the y side's signs
    const int k = y ? min(max(i - HALO, 0), gs.nx - 1)
                    : (yg ? ghost_src(sy.kind, j, gs.ny) : j) - HALO;
    double v[12];
    inflow_values(y ? sy : sx, k, y ? gs.nx : gs.ny, stage, v);
#pragma unroll
    for (int c = 0; c < 4; ++c) st[c] = yg && !y ? sy.sign[c] * v[c] : v[c];
}

// Walls inside the grid (masked domains): solid cell = mirror image of a fluid
// cell across the nearest wall face, with the box walls' parities (Remark 4.1);
// a cell listed with source -1 holds the prescribed state with zero first
// moments instead, as the ghost cells of an inflow side do.
__global__ void k_solid2(const Grid2* gp, int sidx) {
    const Grid2& g = *gp;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= g.nsolid) return;
    double* S = g.S[sidx];
    const long long N = g.ncell;
    const long long d = g.sdst[t], s = g.ssrc[t];
    if (s < 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            S[c * N + d] = g.fixed_state[c];
            S[(4 + c) * N + d] = 0.0;
            S[(8 + c) * N + d] = 0.0;
        }
        return;
    }
    const int dir = g.sdir[t];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool vel = g.solid_wall == 4 ? (c == 1 || c == 2) : (c == 1 + dir);
            const bool mom = m == 1 + dir;
            const double sg = (vel != mom) ? -1.0 : 1.0;
            S[(m * 4 + c) * N + d] = sg * S[(m * 4 + c) * N + s];
        }
    }
}

// Threads 0 .. 2 HALO ny - 1: ghost columns of the interior rows; then the
// 2 HALO ghost rows, every column.
__global__ void k_ghost2(Batch bt, int sidx, int stage) {
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    double* S = gsrc.S[sidx];
    const int t = lc.b * blockDim.x + threadIdx.x;
    const int nxg = g.ny * 2 * HALO;
    if (t >= nxg + g.NX * 2 * HALO) return;
    double v[12];
    long long dst;
    if (t < nxg) {
        const int j = HALO + t / (2 * HALO);
        const int gi = t % (2 * HALO);
        const int i = gi < HALO ? gi : g.nx + gi;
        x_ghost(g, gsrc.side[gi >= HALO], S, j, i, stage, v);
        dst = (long long)j * g.NX + i;
    } else {
        const int u = t - nxg;
        const int i = u % g.NX;
        const int gj = u / g.NX;
        const int j = gj < HALO ? gj : g.ny + gj;
        const Side& sd = gsrc.side[2 + (gj >= HALO)];
        if (sd.kind == 2) {
            // ghost columns take the profile's end states
            inflow_values(sd, min(max(i - HALO, 0), g.nx - 1), g.nx, stage, v);
        } else {
            const int sj = ghost_src(sd.kind, j, g.ny);
            if (i < HALO || i >= HALO + g.nx) {
                x_ghost(g, gsrc.side[i >= HALO], S, sj, i, stage, v);
            } else {
#pragma unroll
                for (int q = 0; q < 12; ++q) v[q] = S[q * g.ncell + (long long)sj * g.NX + i];
            }
#pragma unroll
            for (int q = 0; q < 12; ++q) v[q] = sd.sign[q] * v[q];
        }
        dst = (long long)j * g.NX + i;
    }
#pragma unroll
    for (int q = 0; q < 12; ++q) S[q * g.ncell + dst] = v[q];
}

// Element i (cell offset in bytes) of a plane; base uniform per wavefront.
__device__ __forceinline__ gdouble& at(gdouble* base, unsigned off) {
    return *(gdouble*)((HW_GLOBAL char*)base + off);
}

// The 12 fields of a tile of TX x (64 / TX) cells at (i0, j0) and the ring around
// it into LDS (planes of the tile with ring, clamped to the grid): wavefront wv
// of four loads fields 3 wv .. 3 wv + 2, every load issued before the first LDS
// write.  GH: no fill has written the ghost cells (inflow profiles of stage gst),
// and the input may be the caller's interior array U.
template <int TX, bool GH>
__device__ __forceinline__ void load_tile(const Grid2& g, const Grid2& gsrc, int si, int gst,
                                          const double* U, int i0, int j0, int lane, int wv,
                                          double* tile) {
    constexpr int TY = 64 / TX, TW = TX + 2, TH = TY + 2, PL = TW * TH;
    constexpr int NP = (PL + 63) / 64;
    // plane and row sizes pl and nr; U has interior cell (0, 0) first
    const double* __restrict__ S = GH && U ? U : gsrc.S[si];
    const long long N = g.ncell;
    const long long pl = GH && U ? (long long)g.nx * g.ny : N;
    const int nr = GH && U ? g.nx : g.NX, n0 = GH && U ? HALO * (g.nx + 1) : 0;
    double v[3][NP];
    if constexpr (!GH) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int t = lane + 64 * q, r = t / TW, c = t - r * TW;
            const int gj = min(j0 - 1 + r, g.NY - 1), gi = min(max(i0 - 1 + c, 0), g.NX - 1);
            const unsigned src = 8u * (unsigned)(gj * g.NX + gi);
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if (t < PL) v[f][q] = at((gdouble*)S + (3 * wv + f) * N, src);
        }
    } else {
        // no fill has written the ghost cells: they are read from their
        // source cells, sources and signs without branches (index gi of a
        // ghost cell has source ga * gi + gb); prescribed states (inflow)
        // replace theirs afterwards
        int ga[4], gb[4];
#pragma unroll
        for (int sd = 0; sd < 4; ++sd) {
            const int kind = g.rule[sd] & 15, n = sd < 2 ? g.nx : g.ny;
            ga[sd] = kind == 0 ? 1 : (kind == 1 ? 0 : -1);
            if (sd & 1) gb[sd] = kind == 0 ? -n : (kind == 1 ? HALO + n - 1 : 2 * (HALO + n) - 1);
            else gb[sd] = kind == 0 ? n : (kind == 1 ? HALO : 2 * HALO - 1);
        }
        unsigned in = 0;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int t = lane + 64 * q, r = t / TW, c = t - r * TW;
            const int gj = min(j0 - 1 + r, g.NY - 1), gi = min(max(i0 - 1 + c, 0), g.NX - 1);
            const bool yl = gj < HALO, yh = gj >= HALO + g.ny;
            const bool xl = gi < HALO, xh = gi >= HALO + g.nx;
            const int sj = (yl ? ga[2] : (yh ? ga[3] : 1)) * gj + (yl ? gb[2] : (yh ? gb[3] : 0));
            const int sx = (xl ? ga[0] : (xh ? ga[1] : 1)) * gi + (xl ? gb[0] : (xh ? gb[1] : 0));
            const unsigned ry = yl ? g.rule[2] : (yh ? g.rule[3] : 0u);
            const unsigned rx = xl ? g.rule[0] : (xh ? g.rule[1] : 0u);
            in |= ((ry | rx) >> 31) << q;
            const unsigned src = 8u * (unsigned)(sj * nr + sx - n0);
            const unsigned neg = (ry ^ rx) >> (4 + 3 * wv);
#pragma unroll
            for (int f = 0; f < 3; ++f)
                if (t < PL)
                    v[f][q] = flip_sign(at((gdouble*)S + (3 * wv + f) * pl, src), neg >> f & 1u);
        }
        if (__ballot(in != 0)) {
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const int t = lane + 64 * q, r = t / TW, c = t - r * TW;
                const int gj = min(j0 - 1 + r, g.NY - 1);
                const int gi = min(max(i0 - 1 + c, 0), g.NX - 1);
                double st[4];
                if (t < PL && (in >> q & 1)) {
                    inflow_at(gsrc, gj, gi, gst, st);
#pragma unroll
                    for (int f = 0; f < 3; ++f)   // wavefront 0: fields 0-2, 1: 3-5, ...
                        v[f][q] = wv == 0 ? st[f] : (wv == 1 && f == 0 ? st[3] : 0.0);
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NP; ++q)
#pragma unroll
        for (int f = 0; f < 3; ++f)
            if (lane + 64 * q < PL) tile[(3 * wv + f) * PL + lane + 64 * q] = v[f][q];
}

// ---------------------------------------------------------------------------
// Characteristic reconstruction + positivity limiter (HWENO-GR).
// Block: a TX x (64 / TX) tile of cells, four wavefronts, one thread per cell
// in each: wavefront (b, h) works in basis b (0: x-Jacobian, 1: y-Jacobian) on
// two of its four characteristic fields (h = 0: the acoustic ones 0 and 3,
// h = 1: fields 1 and 2) and then owns the basis's face points (h = 0) or
// volume points (h = 1).  Threads work in their basis's own coordinates
// (normal, tangential), so every wavefront runs the same reconstruction code
// on a stencil tile that basis 1 reads transposed.  A wavefront evaluates its
// two fields at all points and hands the values at its partner's points over
// through LDS; each then forms the four conserved components at its own
// points in registers.
// Bound: the 848 bytes per cell it writes (98 us at the 4.9 TB/s a kernel
// without arithmetic reaches on these planes at 1000x500).  A thread per field
// and component, which exchanged every value twice through LDS behind ten
// barriers and formed the basis eight times per cell, took 190 us there,
// 28 us on 500x100 and 10.5 us on 64^2; this split takes 136, 22.0 and 9.6.  A
// thread per basis (all four fields, no exchange) needs 256 registers: 136
// us, but 12.1 us on 64^2.  Four wavefronts per SIMD instead of three spill
// (193 us).
// ---------------------------------------------------------------------------
// FULL: 0, or the reverse mode's 1 (the full volume values as well) and 2 (these
// alone, where no residual is formed from them).
template <int TX, bool VarMu, int FULL, bool GH>
__global__ __launch_bounds__(256, 3) void k_recon2(Batch bt, int si, int want_alpha, int gst,
                                                 const double* U) {
    constexpr int TY = 64 / TX, TW = TX + 2, TH = TY + 2, PL = TW * TH;
    // handed-over values: per basis and field of a wavefront, 9 volume values
    // (h = 0) or 6 face values and the moment (h = 1) per cell; the second
    // fields' share reuses the stencil tile's memory
    constexpr int XB = 2 * (9 + 7) * 64;   // one field of each of the four wavefronts
    __shared__ double sh[XB + (XB > 12 * PL ? XB : 12 * PL)];
    __shared__ double shm[2][4][64];       // [density, pressure][wavefront][cell]
    __shared__ double shu[4][64];          // GH: cell averages, for the limiter
    double* const tile = sh + XB;
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const double* __restrict__ S = gsrc.S[si];
    const Consts& K = g.K;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = wv >> 1, hh = wv & 1;
    const long long N = g.ncell;
    // region: rows 1..NY-2, columns 1..NX-2; tiles start at multiples of TX
    // columns of the ghosted grid
    const int tiles_x = (g.NX - 1 + TX - 1) / TX;
    const int i0 = (lc.b % tiles_x) * TX, j0 = 1 + (lc.b / tiles_x) * TY;
    const int lx = lane % TX, ly = lane / TX;
    const int i = i0 + lx, j = j0 + ly;
    const bool valid = i >= 1 && i <= g.NX - 2 && j <= g.NY - 2;
    load_tile<TX, GH>(g, gsrc, si, gst, U, i0, j0, lane, wv, tile);
    __syncthreads();
    const double* T0 = tile + (ly + 1) * TW + lx + 1;
    if constexpr (GH) shu[wv][lane] = T0[wv * PL];
    // cell average: in the global order (pbar: the same bits in every
    // wavefront) and in the basis's
    const double rbar = T0[0];
    const double pbar = pressure2(K, rbar, T0[PL], T0[2 * PL], T0[3 * PL]);
    const Basis2 e = basis2(K, rbar, T0[(1 + b) * PL], T0[(2 - b) * PL], T0[3 * PL]);
    // this wavefront's values of its fields at its own points (the last slot
    // of h = 0: 6 face values, then the moment)
    double va[9], vb[9];
#pragma unroll 1
    for (int kk = 0; kk < 2; ++kk) {
        const int k = hh == 0 ? 3 * kk : 1 + kk;
        double C[15];
        {
            double L[4], R[4], a[17];
            field_rows(e, k, L, R);
            if (b == 0) project2<0, TW, PL>(T0, L, a);
            else project2<1, TW, PL>(T0, L, a);
            hweno2d(a, K, C);
        }
        if (kk == 1) __syncthreads();   // every wavefront has read the tile
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
    // the four conserved components (basis order) at own point o, from the
    // fields' values x0, x3 (acoustic), x1, x2 there; contraction fixed in the
    // source here and below, for the same bits in every variant of the kernel
    auto cons = [&](double x0, double x1, double x2, double x3, double* u) {
#pragma clang fp contract(off)
        const double sm = x0 + x3, df = x3 - x0;
        u[0] = sm + x1;
        u[1] = fma(e.un, u[0], e.c * df);
        u[2] = fma(e.ut, u[0], x2);
        u[3] = fma(e.H, sm, fma(e.un * e.c, df, fma(0.5 * e.q2, x1, e.ut * x2)));
    };
    const double* XP = sh + b * (XB / 2) + lane;   // partner's values: + kk * XB
    // planes of the components and of the volume points in global ordering
    const int gc[4] = {0, 1 + b, 2 - b, 3};
    auto gq = [&](int q) { return b ? 3 * (q % 3) + q / 3 : q; };
    const unsigned off = 8u * (unsigned)(j * g.NX + i);
    const bool inter = valid && j >= HALO && j < HALO + g.ny && i >= HALO && i < HALO + g.nx;
    double rmin = INFINITY, pmin = INFINITY;
    double v[4][6];      // h = 0: the components at the face points
    if (hh == 0) {
#pragma unroll
        for (int o = 0; o < 7; ++o) {
            double u[4];
            cons(va[o], XP[(9 + o) * 64], XP[XB + (9 + o) * 64], vb[o], u);
            if (o < 6) {
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c][o] = u[c];
                rmin = fmin(rmin, u[0]);
                pmin = fmin(pmin, pressure2(K, u[0], u[1], u[2], u[3]));
            } else if (inter) {
#pragma unroll
                for (int c = 0; c < 4; ++c) at(g.vk + (b * 4 + gc[c]) * N, off) = u[c];
            }
        }
    } else if (valid) {
        // volume points (unlimited): wbar of (u, v, e), and the compact data of
        // the gradient kernel's volume flux (Gauss sum of the convective flux,
        // velocities and, with mu(T), T / T_ref at the points: the power law's
        // registers would cost this kernel spills)
#pragma clang fp contract(off)
        double sn = 0.0, st = 0.0, se = 0.0, fs[4] = {0.0, 0.0, 0.0, 0.0};
        gdouble* VC = g.vc + (long long)b * VC_B * N;
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            double u[4];
            cons(XP[q * 64], va[q], vb[q], XP[XB + q * 64], u);
            const double w = (q / 3 == 1 ? GW1 : GW0) * (q % 3 == 1 ? GW1 : GW0);
            const double ir = rcp(u[0]);
            const double un = u[1] * ir, ut = u[2] * ir;
            sn = fma(w, un, sn);
            st = fma(w, ut, st);
            se = fma(w, fma(-0.5, fma(un, un, ut * ut), u[3] * ir), se);
            const double p = K.gm1 * fma(-0.5, fma(u[1], un, u[2] * ut), u[3]);
            rmin = fmin(rmin, u[0]);
            pmin = fmin(pmin, p);
            if constexpr (FULL != 2) {
                fs[0] = fma(w, u[1], fs[0]);
                fs[1] = fma(w, fma(u[1], un, p), fs[1]);
                fs[2] = fma(w, u[2] * un, fs[2]);
                fs[3] = fma(w, (u[3] + p) * un, fs[3]);
                at(VC + ((b ? 13 : 4) + gq(q)) * N, off) = un;
                at(VC + ((b ? 4 : 13) + gq(q)) * N, off) = ut;
                if constexpr (VarMu) at(VC + (22 + gq(q)) * N, off) = (p / u[0]) / K.T_ref;
            }
            if constexpr (FULL) {   // the reverse mode reads the full volume values
                gdouble* V = b ? g.yv : g.xv;
#pragma unroll
                for (int c = 0; c < 4; ++c) at(V + (gq(q) * 4 + gc[c]) * N, off) = u[c];
            }
        }
        gdouble* WB = g.wb + (long long)b * 3 * N;
        at(WB + b * N, off) = sn;
        at(WB + (1 - b) * N, off) = st;
        at(WB + 2 * N, off) = se;
        if constexpr (FULL != 2) {
#pragma unroll
            for (int c = 0; c < 4; ++c) at(VC + gc[c] * N, off) = fs[c];
        }
    }
    // positivity limiter: theta1 from the least density, theta2 from the least
    // pressure over the points of both bases ((pbar - eps) / (pbar - p) falls
    // with p, so its minimum is taken at the least pressure)
    shm[0][wv][lane] = rmin;
    shm[1][wv][lane] = pmin;
    __syncthreads();
    auto least = [&](int q) {
        return fmin(fmin(shm[q][0][lane], shm[q][1][lane]), fmin(shm[q][2][lane], shm[q][3][lane]));
    };
    rmin = least(0);
    pmin = least(1);
    const double eps = fmin(fmin(K.eps_pp, rbar), pbar);
    double th1 = 1.0;
    // every wavefront holds the same cells and minima: the branch is taken by
    // the whole block or not at all
    if (__ballot(valid && rmin < eps)) {
        th1 = rmin < eps ? (rbar - eps) / (rbar - rmin) : 1.0;
        // pressures at the limited densities
        pmin = INFINITY;
        if (hh == 0) {
#pragma unroll
            for (int o = 0; o < 6; ++o) {
                v[0][o] = rbar + th1 * (v[0][o] - rbar);
                pmin = fmin(pmin, pressure2(K, v[0][o], v[1][o], v[2][o], v[3][o]));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                double u[4];
                cons(XP[q * 64], va[q], vb[q], XP[XB + q * 64], u);
                pmin = fmin(pmin, pressure2(K, rbar + th1 * (u[0] - rbar), u[1], u[2], u[3]));
            }
        }
        __syncthreads();   // the unlimited minima have been read
        shm[1][wv][lane] = pmin;
        __syncthreads();
        pmin = least(1);
    }
    if (hh != 0) return;
    const bool acted = valid && (th1 < 1.0 || pmin < eps);
    if (__ballot(acted)) {
        if (acted) {
            const double th2 = pmin < eps ? fmin((pbar - eps) / (pbar - pmin), 1.0) : 1.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double ub =
                    GH ? shu[gc[c]][lane] : at((gdouble*)S + gc[c] * N, off);
#pragma unroll
                for (int o = 0; o < 6; ++o) v[c][o] = ub + th2 * (v[c][o] - ub);
            }
        }
        const unsigned long long n = __ballot(inter && acted);
        if (b == 0 && lane == 0 && n)
            atomicAdd((unsigned long long*)&gsrc.red->pp_cells, (unsigned long long)__popcll(n));
    }
    if (valid) {
        gdouble* F = b ? g.yf : g.xf;
#pragma unroll
        for (int o = 0; o < 6; ++o)
#pragma unroll
            for (int c = 0; c < 4; ++c) at(F + (o * 4 + gc[c]) * N, off) = v[c][o];
    }
    // CFL wave speed over the limited face traces of interior cells
    if (want_alpha) {
        double amax = -INFINITY;
#pragma unroll
        for (int o = 0; o < 6; ++o) {
            const double ir = rcp(v[0][o]);
            const double un = v[1][o] * ir, ut = v[2][o] * ir;
            const double p = K.gm1 * fma(-0.5, fma(v[1][o], un, v[2][o] * ut), v[3][o]);
            amax = fmax(amax, fmax(fabs(un), fabs(ut)) + sqrt(K.gamma * p * ir));
        }
        amax = wave_max(inter ? amax : -INFINITY);
        if (lane == 0) {
            const unsigned long long k = dkey(amax);
            HW_GLOBAL unsigned long long* slot = &gsrc.red->alpha_key;
            if (amax > -INFINITY && k > *(volatile HW_GLOBAL unsigned long long*)slot)
                atomicMax((unsigned long long*)slot, k);
        }
    }
}

// ---------------------------------------------------------------------------
// Characteristic reconstruction + positivity limiter, HWENO-DR (eq. (3.5)).
// The block, the split over its wavefronts and the handing over are those of
// k_recon2.  A wavefront keeps the coefficients of its two fields and, after
// the limiter, differentiates them (weights kept) along the normal, then along the
// tangent of its basis; the derivatives take the same way as the values: the
// partner's points through LDS, four conserved components at its own points in
// registers.  There they give the gradients of (u_n, u_t, e) with the point values
// that enter the flux (limited face traces; unlimited volume values), so the
// kernel writes the face gradients and the volume-flux quadratures itself, in
// place of the weak-moment and gradient kernels.
// Bound: arithmetic at two wavefronts per SIMD (two fields' coefficients are live
// throughout).  A thread per field, which exchanged every value and derivative
// twice through LDS behind 19 barriers, took 97 us per stage on 500x250 and 111
// with mu(T); this one takes 77 and 97 (13.5 and 15.4 on 64x64, where the ghost
// cells formed in its loads save a launch of 5).
// ---------------------------------------------------------------------------
template <int TX, bool VarMu, bool GH>
__global__ __launch_bounds__(256, 2) void k_recon2_dr(Batch bt, int si, int want_alpha, int gst,
                                                      const double* U) {
    constexpr int TY = 64 / TX, TW = TX + 2, TH = TY + 2, PL = TW * TH;
    // handed over per basis, one field of each wavefront: 9 volume values (h = 0),
    // 6 face values and the moment (h = 1); the derivatives likewise
    constexpr int XV = 2 * (9 + 7) * 64, XD = 2 * (9 + 6) * 64;
    __shared__ double shv[2 * XV];
    __shared__ double shd[2 * XD];         // the stencil tile first
    __shared__ double shm[2][4][64];       // [density, pressure][wavefront][cell]
    __shared__ double shk[VarMu ? 2 * 9 * 64 : 1];   // mu(T) at the volume points
    static_assert(2 * XD >= 12 * PL, "the derivatives reuse the tile");
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const Consts& K = g.K;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = wv >> 1, hh = wv & 1;
    const long long N = g.ncell;
    // region: rows 1..NY-2, columns 1..NX-2; tiles start at multiples of TX
    // columns of the ghosted grid
    const int tiles_x = (g.NX - 1 + TX - 1) / TX;
    const int i0 = (lc.b % tiles_x) * TX, j0 = 1 + (lc.b / tiles_x) * TY;
    const int lx = lane % TX, ly = lane / TX;
    const int i = i0 + lx, j = j0 + ly;
    const bool valid = i >= 1 && i <= g.NX - 2 && j <= g.NY - 2;
    const unsigned off = 8u * (unsigned)(j * g.NX + i);
    load_tile<TX, GH>(g, gsrc, si, gst, U, i0, j0, lane, wv, shd);
    __syncthreads();
    const double* T0 = shd + (ly + 1) * TW + lx + 1;
    // cell average in basis order (pbar: the same bits in every wavefront)
    const double ub[4] = {T0[0], T0[(1 + b) * PL], T0[(2 - b) * PL], T0[3 * PL]};
    const double rbar = ub[0];
    const double pbar = pressure2(K, rbar, T0[PL], T0[2 * PL], T0[3 * PL]);
    const Basis2 e = basis2(K, rbar, ub[1], ub[2], ub[3]);
    const Part<0> face{};
    const Part<1> vol{};
    // this wavefront's fields: coefficients, and values at its own points (the
    // last slot of h = 0: 6 face values, then the moment)
    double Ca[15], Cb[15], va[9], vb[9];
#pragma unroll 1
    for (int kk = 0; kk < 2; ++kk) {
        const int k = hh == 0 ? 3 * kk : 1 + kk;
#pragma unroll
        for (int q = 0; q < 15; ++q) Ca[q] = Cb[q];
        {
            double L[4], R[4], a[17];
            field_rows(e, k, L, R);
            if (b == 0) project2<0, TW, PL>(T0, L, a);
            else project2<1, TW, PL>(T0, L, a);
            hweno2d(a, K, Cb);
        }
        double* X = shv + kk * XV + b * (XV / 2) + lane;
        double f[7], w[9];
        eval_xface(Cb, f);
        f[6] = moment_xi(Cb);
        eval_vol(Cb, w);
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
    __syncthreads();   // the values are handed over and the tile is dead
    auto cons = [&](double x0, double x1, double x2, double x3, double* u) {
#pragma clang fp contract(off)
        const double sm = x0 + x3, df = x3 - x0;
        u[0] = sm + x1;
        u[1] = fma(e.un, u[0], e.c * df);
        u[2] = fma(e.ut, u[0], x2);
        u[3] = fma(e.H, sm, fma(e.un * e.c, df, fma(0.5 * e.q2, x1, e.ut * x2)));
    };
    // conserved components at own point o from the wavefront's fields xa, xb and
    // the partner's at X and X + step
    auto point = [&](auto H, int o, const double* xa, const double* xb, const double* X, int step,
                     double* u) {
        if constexpr (H.value == 0) cons(xa[o], X[(9 + o) * 64], X[step + (9 + o) * 64], xb[o], u);
        else cons(X[o * 64], xa[o], xb[o], X[step + o * 64], u);
    };
    const double* XP = shv + b * (XV / 2) + lane;
    const int gc[4] = {0, 1 + b, 2 - b, 3};   // global number of a basis component
    const bool inter = valid && j >= HALO && j < HALO + g.ny && i >= HALO && i < HALO + g.nx;
    // positivity limiter, as in k_recon2
    double rmin = INFINITY, pmin = INFINITY, th1 = 1.0, th2 = 1.0;
    bool acted = false;
    auto minima = [&](auto H, bool limited) {
#pragma unroll
        for (int o = 0; o < H.points; ++o) {
            double u[4];
            point(H, o, va, vb, XP, XV, u);
            if (!limited) rmin = fmin(rmin, u[0]);
            const double r = limited ? rbar + th1 * (u[0] - rbar) : u[0];
            pmin = fmin(pmin, pressure2(K, r, u[1], u[2], u[3]));
        }
    };
    if (hh == 0) minima(face, false);
    else minima(vol, false);
    shm[0][wv][lane] = rmin;
    shm[1][wv][lane] = pmin;
    __syncthreads();
    auto least = [&](int q) {
        return fmin(fmin(shm[q][0][lane], shm[q][1][lane]), fmin(shm[q][2][lane], shm[q][3][lane]));
    };
    rmin = least(0);
    pmin = least(1);
    const double eps = fmin(fmin(K.eps_pp, rbar), pbar);
    // every wavefront holds the same cells and minima: the branch is taken by
    // the whole block or not at all
    if (__ballot(valid && rmin < eps)) {
        th1 = rmin < eps ? (rbar - eps) / (rbar - rmin) : 1.0;
        pmin = INFINITY;
        if (hh == 0) minima(face, true);
        else minima(vol, true);
        __syncthreads();   // the unlimited minima have been read
        shm[1][wv][lane] = pmin;
        __syncthreads();
        pmin = least(1);
    }
    acted = th1 < 1.0 || pmin < eps;
    if (pmin < eps) th2 = fmin((pbar - eps) / (pbar - pmin), 1.0);
    // value that enters the flux at own point o
    auto value = [&](auto H, int o, double* u) {
        point(H, o, va, vb, XP, XV, u);
        if constexpr (H.value == 0) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double x = c == 0 ? rbar + th1 * (u[0] - rbar) : u[c];
                u[c] = acted ? ub[c] + th2 * (x - ub[c]) : u[c];
            }
        }
    };
    if (hh == 0) {
        double amax = -INFINITY;
        gdouble* F = b ? g.yf : g.xf;
#pragma unroll
        for (int o = 0; o < 7; ++o) {
            double u[4];
            if (o == 6) {
                point(face, o, va, vb, XP, XV, u);
                if (inter) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) at(g.vk + (b * 4 + gc[c]) * N, off) = u[c];
                }
                continue;
            }
            value(face, o, u);
            if (valid) {
#pragma unroll
                for (int c = 0; c < 4; ++c) at(F + (o * 4 + gc[c]) * N, off) = u[c];
            }
            // CFL wave speed over the limited face traces of interior cells
            const double ir = rcp(u[0]);
            const double un = u[1] * ir, ut = u[2] * ir;
            const double p = K.gm1 * fma(-0.5, fma(u[1], un, u[2] * ut), u[3]);
            amax = fmax(amax, fmax(fabs(un), fabs(ut)) + sqrt(K.gamma * p * ir));
        }
        if (want_alpha) {
            amax = wave_max(inter ? amax : -INFINITY);
            if (lane == 0) {
                const unsigned long long k = dkey(amax);
                HW_GLOBAL unsigned long long* slot = &gsrc.red->alpha_key;
                if (amax > -INFINITY && k > *(volatile HW_GLOBAL unsigned long long*)slot)
                    atomicMax((unsigned long long*)slot, k);
            }
        }
        const unsigned long long n = __ballot(inter && acted);
        if (b == 0 && lane == 0 && n)
            atomicAdd((unsigned long long*)&gsrc.red->pp_cells, (unsigned long long)__popcll(n));
    }
    // mu(T) at the volume points ahead of the gradients, whose registers it would
    // spill (the wavefront reads its own back)
    double* M = shk + (VarMu ? b * (9 * 64) + lane : 0);
    if constexpr (VarMu) {
        if (hh == 1) {
#pragma unroll
            for (int o = 0; o < 9; ++o) {
                double u[4];
                value(vol, o, u);
                M[o * 64] = viscosity<true>(K, u[0], pressure2(K, u[0], u[1], u[2], u[3]));
            }
        }
    }
    // derivatives along the normal (dir 0) and the tangent (dir 1), and from them
    // the gradients; faces of interior cells read those of the cells on both
    // sides, volume fluxes are needed in interior cells only
    const bool ring = valid && j >= HALO - 1 && j <= HALO + g.ny && i >= HALO - 1 &&
                      i <= HALO + g.nx;
    double sn[9][3];                      // normal derivatives of (u_n, u_t, e)
    double vfs[4] = {0.0, 0.0, 0.0, 0.0};
    auto gradients = [&](auto H, int dir, const double* da, const double* db) {
        const double* X = shd + b * (XD / 2) + lane;
        const double h = (b == 0) == (dir == 0) ? K.idx : K.idy;
#pragma unroll
        for (int o = 0; o < H.points; ++o) {
            double P[4], D[4];
            value(H, o, P);
            point(H, o, da, db, X, XD, D);
#pragma unroll
            for (int c = 0; c < 4; ++c) D[c] *= h;
            const double ir = rcp(P[0]);
            const double un = P[1] * ir, ut = P[2] * ir;
            const double dn = (D[1] - un * D[0]) * ir, dt = (D[2] - ut * D[0]) * ir;
            const double de = (D[3] - P[3] * ir * D[0]) * ir - un * dn - ut * dt;
            if (dir == 0) {
                sn[o][0] = dn;
                sn[o][1] = dt;
                sn[o][2] = de;
                continue;
            }
            // (u_n)_n, (u_n)_t, (u_t)_n, (u_t)_t, e_n, e_t: direction 0 of the
            // basis's own coordinates
            const double sg[6] = {sn[o][0], dn, sn[o][1], dt, sn[o][2], de};
            if constexpr (H.value == 0) {
                double dc[3];
                stress_combos<0>(sg, dc);
                if (ring) {
#pragma unroll
                    for (int z = 0; z < 3; ++z) at(g.gf + ((b * 6 + o) * 3 + z) * N, off) = dc[z];
                }
            } else {
                const double w = (o / 3 == 1 ? GW1 : GW0) * (o % 3 == 1 ? GW1 : GW0);
                const double mu = VarMu ? M[o * 64] : K.mu_ref;
                const double p = K.gm1 * fma(-0.5, fma(P[1], un, P[2] * ut), P[3]);
                const Stress tau = stresses(mu, sg);
                double f[4];
                f[0] = P[1];
                f[1] = fma(P[1], un, p) - tau.xx;
                f[2] = fma(P[2], un, -tau.xy);
                f[3] = fma(P[3] + p, un, -fma(tau.xx, un, fma(tau.xy, ut, K.gPr * mu * sg[4])));
#pragma unroll
                for (int c = 0; c < 4; ++c) vfs[c] = fma(w, f[c], vfs[c]);
            }
        }
    };
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
        double da[9], db[9];
        if (dir == 1) __syncthreads();   // the normal derivatives have been read
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const double* C = kk == 0 ? Ca : Cb;
            double* X = shd + kk * XD + b * (XD / 2) + lane;
            double* d = kk == 0 ? da : db;
            double D[15], w[9];
            if (dir == 0) dxi_coeffs(C, D);
            else deta_coeffs(C, D);
            if (hh == 0) {
                eval_xface(D, d);
                eval_vol(D, w);
#pragma unroll
                for (int q = 0; q < 9; ++q) X[q * 64] = w[q];
            } else {
                eval_xface(D, w);
                eval_vol(D, d);
#pragma unroll
                for (int q = 0; q < 6; ++q) X[(9 + q) * 64] = w[q];
            }
        }
        __syncthreads();
        if (hh == 0) gradients(face, dir, da, db);
        else gradients(vol, dir, da, db);
    }
    if (hh == 1 && inter) {
#pragma unroll
        for (int c = 0; c < 4; ++c) at(g.vf + (b * 4 + gc[c]) * N, off) = vfs[c];
    }
}

// ---------------------------------------------------------------------------
// Weak-derivative moments (eqs. (3.6)-(3.8)) on cells of halo ring 2.
// ---------------------------------------------------------------------------
// Primitives (u, v, e) of face point p of `cell` (one reciprocal of rho).
__device__ __forceinline__ void prim3(const double* F, long long N, long long cell, int p,
                                      double* w) {
#pragma clang fp contract(off)
    const double r = F[(p * 4 + 0) * N + cell];
    const double ir = rcp(r);
    const double u = F[(p * 4 + 1) * N + cell] * ir;
    const double v = F[(p * 4 + 2) * N + cell] * ir;
    w[0] = u;
    w[1] = v;
    w[2] = F[(p * 4 + 3) * N + cell] * ir - 0.5 * (u * u + v * v);
}

// Gauss average W0 = sum_G w_G h_G and first moment W1 = sum_G w_G x_G h_G of
// the interface average h = (w- + w+)/2 of (u, v, e) over the face between
// cell `lo` (its upper points 3..5) and cell `hi` (its lower points 0..2).
// Mirror-symmetric forms: exchanging the outer points gives the same W0 and
// the negated W1.  Contraction is fixed in the source, so every kernel that
// forms the weak moments gets the same bits.
__device__ __forceinline__ void face_wavg(const double* F, long long N, long long lo, long long hi,
                                          double* W0, double* W1) {
#pragma clang fp contract(off)
    double h[3][3];   // [G][w]
#pragma unroll
    for (int G = 0; G < 3; ++G) {
        double a[3], c[3];
        prim3(F, N, lo, 3 + G, a);
        prim3(F, N, hi, G, c);
#pragma unroll
        for (int w = 0; w < 3; ++w) h[G][w] = 0.5 * (a[w] + c[w]);
    }
#pragma unroll
    for (int w = 0; w < 3; ++w) {
        W0[w] = fma(GW0, h[0][w] + h[2][w], GW1 * h[1][w]);
        W1[w] = (GW0 * GS) * (h[2][w] - h[0][w]);
    }
}

// The three weak moments (eqs. (3.6)-(3.8)) of d w / d x_l of a cell from the
// face data of its lower and upper l-faces and its w-bar; ih = 1/dx_l.
// m[0] = moment 0, m[1] = xi moment, m[2] = eta moment.
__device__ __forceinline__ void cell_wmom(double W0lo, double W0hi, double W1lo, double W1hi,
                                          double wbl, double ih, int l, double* m) {
#pragma clang fp contract(off)
    const double d0 = (W0hi - W0lo) * ih;                    // moment 0
    const double dm = (0.5 * (W0hi + W0lo) - wbl) * ih;      // moment along l
    const double d1 = (W1hi - W1lo) * ih;                    // transverse moment
    m[0] = d0;
    m[1] = l ? d1 : dm;
    m[2] = l ? dm : d1;
}

// Block = RB_TX x RB_TY cells of the region (rows and columns 2 .. N-3).
// First every face of the tile gets its interface averages w^ = (w- + w+)/2
// at the three Gauss points, once (a face is shared by two cells): the x-faces
// of each tile row and the y-faces of each tile column, into LDS.  Then each
// cell forms the 18 weak moments of d w / d x_l from its four faces and w-bar.
constexpr int RB_TX = 32, RB_TY = 8;

__global__ __launch_bounds__(RB_TX * RB_TY) void k_rbar2(Batch bt) {
    constexpr int NXF = RB_TY * (RB_TX + 1), NYF = (RB_TY + 1) * RB_TX;
    // per face and variable w: the Gauss average W0 = sum_G w_G h_G and the
    // first moment W1 = sum_G w_G x_G h_G of the interface average h
    __shared__ double hx[6][RB_TY][RB_TX + 1];   // [3 m + w][row][face i - 1/2]
    __shared__ double hy[6][RB_TY + 1][RB_TX];   // [3 m + w][face j - 1/2][column]
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    // tiles start at multiples of RB_TX columns of the ghosted grid (whole
    // cache lines per row segment); columns 0 and 1 are outside the region
    const int tiles_x = (g.NX - 2 + RB_TX - 1) / RB_TX;
    const int i0 = (lc.b % tiles_x) * RB_TX;
    const int j0 = 2 + (lc.b / tiles_x) * RB_TY;
    const long long N = g.ncell;
    for (int t = threadIdx.x; t < NXF + NYF; t += RB_TX * RB_TY) {
        const bool xd = t < NXF;
        const int q = xd ? t : t - NXF;
        // face between cells (ilo, jlo) and (i, j): i - 1/2 (x) or j - 1/2 (y)
        int i, j, ilo, jlo;
        if (xd) {
            i = i0 + q % (RB_TX + 1);
            j = j0 + q / (RB_TX + 1);
            ilo = i - 1;
            jlo = j;
            if (j > g.NY - 3 || i > g.NX - 2 || i < 2) continue;
        } else {
            i = i0 + q % RB_TX;
            j = j0 + q / RB_TX;
            ilo = i;
            jlo = j - 1;
            if (i > g.NX - 3 || j > g.NY - 2 || i < 2) continue;
        }
        const double* F = xd ? g.xf : g.yf;
        const long long lo = (long long)jlo * g.NX + ilo, hi = (long long)j * g.NX + i;
        double W0[3], W1[3];
        face_wavg(F, N, lo, hi, W0, W1);
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            if (xd) {
                hx[w][j - j0][i - i0] = W0[w];
                hx[3 + w][j - j0][i - i0] = W1[w];
            } else {
                hy[w][j - j0][i - i0] = W0[w];
                hy[3 + w][j - j0][i - i0] = W1[w];
            }
        }
    }
    __syncthreads();
    const int tx = threadIdx.x % RB_TX, ty = threadIdx.x / RB_TX;
    const int i = i0 + tx, j = j0 + ty;
    if (i < 2 || i > g.NX - 3 || j > g.NY - 3) return;
    const long long cell = (long long)j * g.NX + i;
#pragma unroll
    for (int l = 0; l < 2; ++l) {
        const double ih = l ? g.K.idy : g.K.idx;
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            const double W0lo = l ? hy[w][ty][tx] : hx[w][ty][tx];
            const double W0hi = l ? hy[w][ty + 1][tx] : hx[w][ty][tx + 1];
            const double W1lo = l ? hy[3 + w][ty][tx] : hx[3 + w][ty][tx];
            const double W1hi = l ? hy[3 + w][ty + 1][tx] : hx[3 + w][ty][tx + 1];
            double m[3];
            cell_wmom(W0lo, W0hi, W1lo, W1hi, g.wb[(l * 3 + w) * N + cell], ih, l, m);
            double* R = g.rb + ((l * 3 + w) * 3) * N + cell;
            R[0] = m[0];
            R[N] = m[1];       // xi moment
            R[2 * N] = m[2];   // eta moment
        }
    }
}

// ---------------------------------------------------------------------------
// Gradient reconstruction (eq. (3.9)) on halo ring 1, and on interior cells
// the volume-flux quadratures of eq. (3.2).
// ---------------------------------------------------------------------------
// The fluxes need the six gradients only in the combinations of
// stress_combos, each of a pair of them: (u_x, v_y), (v_x, u_y) and (e_x, e_y).
// A wavefront takes one pair k of 32 cells: its lower 32 lanes reconstruct the
// x-derivative and its upper 32 lanes the y-derivative; the halves then trade
// point values by lane swaps, and each lane forms its pair's combination at
// the six face points of its own direction and its pair's part of the volume
// flux of that direction.  So a block (NC cells, three wavefronts per 32) meets
// in LDS only for the energy component's sum (and the viscosities with mu(T)).
// A thread per component, exchanging every point value through LDS behind
// seven barriers, held this kernel to 105 us per stage at 1000x500.
constexpr int GW_MU = 9 * 64;   // LDS doubles per three wavefronts with mu(T)

// Component (2 w + l) of lane half l of pair k, as variable w of (u, v, e).
__device__ __forceinline__ int pair_var(int k, int l) { return k == 2 ? 2 : (k ^ l); }

// The two values of a pair from one value per half: afterwards x holds the
// lower half's x (low lanes) or y (high lanes), y the upper half's.
__device__ __forceinline__ void swap_halves(double& x, double& y) {
#ifdef __HIP_DEVICE_COMPILE__
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(x),
                                                     (unsigned)__double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(x),
                                                     (unsigned)__double2hiint(y), false, false);
    x = __hiloint2double((int)hi[0], (int)lo[0]);
    y = __hiloint2double((int)hi[1], (int)lo[1]);
#endif
}

// Stencil data a (17) of the lane's component -> gradients, their stores, and
// the volume flux.  k: the wavefront's pair (uniform); g3: which three
// wavefronts of the block; shm: NC / 32 * (3 * 64 (+ GW_MU)) doubles of LDS.
// Every thread of the block calls it (it holds barriers).
template <bool VarMu, bool FULL, bool SUMS = true>
__device__ __forceinline__ void grad_body(const Grid2& g, double* shm, const double* a, int k,
                                          bool valid, int j, int i) {
#pragma clang fp contract(off)
    const Consts& K = g.K;
    const long long N = g.ncell;
    const unsigned off = 8u * (unsigned)(j * g.NX + i);
    const int lane = threadIdx.x & 63;
    const int hi = lane >> 5;
    const bool inter = valid && j >= HALO && j < HALO + g.ny && i >= HALO && i < HALO + g.nx;
    // the pair's factor in the energy flux: the velocity normal to the face for
    // the normal stress, tangential for the shear, gamma / Pr for e
    gdouble* VC = g.vc + (hi ? VC_B : 0) * N;
    double pv[9];
    if constexpr (!SUMS) {
    } else if (k < 2) {
        gdouble* VV = VC + ((k ^ hi) == 0 ? 4 : 13) * N;
#pragma unroll
        for (int q = 0; q < 9; ++q) pv[q] = at(VV + q * N, off);
    } else {
#pragma unroll
        for (int q = 0; q < 9; ++q) pv[q] = K.gPr;
    }
    double C[15];
    hweno2d(a, grad_consts(K), C);
    double fx[6], fy[6], va[9], vb[9];
    eval_xface(C, fx);
    eval_yface(C, fy);
    eval_vol(C, va);
    if constexpr (FULL) {
        if (valid) {
            const int s = 2 * pair_var(k, hi) + hi;
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                at(g.gf + (p * 6 + s) * N, off) = fx[p];
                at(g.gf + ((6 + p) * 6 + s) * N, off) = fy[p];
            }
        }
    }
    if constexpr (!SUMS) return;
    // the pair's combination from the values of the lane's own direction and
    // the other one (stress_combos)
    const double co = k == 0 ? 4.0 / 3.0 : 1.0, ct = k == 0 ? -(2.0 / 3.0) : 1.0;
    auto combo = [&](double x, double y) {
        const double own = hi ? y : x, oth = hi ? x : y;
        return fma(co, own, ct * (k == 2 ? 0.0 : oth));
    };
    if constexpr (!FULL) {
#pragma unroll
        for (int p = 0; p < 6; ++p) {
            swap_halves(fx[p], fy[p]);
            const double v = combo(fx[p], fy[p]);
            if (valid) at(g.gf + ((hi * 6 + p) * 3 + k) * N, off) = v;
        }
    }
    // volume flux: viscous part of direction hi from this pair, at the points
    // of that direction's basis (the reconstruction kernel left the Gauss sum
    // of the convective flux and the velocities and temperatures)
    double mu[9];
    if constexpr (VarMu) {   // three of the nine points per wavefront
        double* M = shm + 3 * 64;
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if (inter) M[(3 * k + q) * 64 + lane] = viscosity_T(K, at(VC + (22 + 3 * k + q) * N, off));
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 9; ++q) mu[q] = M[q * 64 + lane];
    }
    double am = 0.0, ae = 0.0;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        vb[q] = va[q];
        swap_halves(va[q], vb[q]);
        const double w = (q / 3 == 1 ? GW1 : GW0) * (q % 3 == 1 ? GW1 : GW0);
        const double t = (VarMu ? mu[q] : K.mu_ref) * combo(va[q], vb[q]);
        am = fma(w, t, am);
        ae = fma(w, t * pv[q], ae);
    }
    shm[k * 64 + lane] = ae;
    __syncthreads();
    if (!inter) return;
    const int d = hi;
    if (k < 2) {
        // the normal stress enters the momentum along the direction
        const int c = k ^ d;
        at(g.vf + (d * 4 + 1 + c) * N, off) = at(VC + (1 + c) * N, off) - am;
    } else {
        at(g.vf + d * 4 * N, off) = at(VC, off);
        at(g.vf + (d * 4 + 3) * N, off) =
            at(VC + 3 * N, off) - (shm[lane] + shm[64 + lane] + shm[128 + lane]);
    }
}

// The gradient kernel of the reverse mode, which reads the weak moments itself
// (k_rbar2 leaves them in memory) and all six gradients: GR_CELLS cells per block.
// SUMS: the volume-flux quadratures too, from which a residual is formed.
template <int GR_CELLS, bool VarMu, bool SUMS>
__global__ __launch_bounds__(6 * GR_CELLS) void k_grad2(Batch bt) {
    constexpr int SH = 3 * 64 + (VarMu ? GW_MU : 0);
    __shared__ double shm[GR_CELLS / 32 * SH];
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k = wv % 3, l = (threadIdx.x >> 5) & 1, w = pair_var(k, l);
    const int wc = g.NX - 6;
    const int nreg = wc * (g.NY - 6);
    const int cid = lc.b * GR_CELLS + wv / 3 * 32 + (threadIdx.x & 31);
    const bool valid = cid < nreg;
    int j = 3, i = 3;
    if (valid) {
        j = 3 + cid / wc;
        i = 3 + cid % wc;
    }
    const long long N = g.ncell;
    gdouble* R = g.rb + (l * 3 + w) * 3 * N;
    const unsigned off = 8u * (unsigned)(j * g.NX + i), row = 8u * (unsigned)g.NX;
    double a[17];
#pragma unroll
    for (int q = 0; q < 9; ++q) a[q] = at(R, off + (q / 3 - 1) * row + 8u * (q % 3 - 1));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = 2 * e + 1;
        const unsigned nb = off + (q / 3 - 1) * row + 8u * (q % 3 - 1);
        a[9 + e] = at(R + N, nb);
        a[13 + e] = at(R + 2 * N, nb);
    }
    grad_body<VarMu, true, SUMS>(g, shm + wv / 3 * SH, a, k, valid, j, i);
}

// ---------------------------------------------------------------------------
// Weak moments and gradient reconstruction in one kernel (HWENO-GR, face
// gradients in the three combinations).  A block takes TX x TY = 32 cells of
// the gradient region and forms the weak moments of those cells and of the
// ring around them in LDS (the ring is formed again by the neighbouring
// tiles): first the interface data of every face of the ring's cells, then
// their 18 weak moments, then the gradient reconstruction reads its 3x3
// stencils from LDS.  Same arithmetic as k_rbar2 followed by k_grad2, without
// the weak moments' round trip through HBM.
// Bound: memory (54 planes read, 44 more of the volume points, 44 written;
// the ring's share of the first comes from the caches).  Blocks of three
// wavefronts overlap one's loads with another's arithmetic; 64 cells per block
// cost 204 us per stage at 1000x500.  Against the two kernels (with the same
// gradient body; sum of both, us): 64x64 11.9 -> 6.6, 500x100 22.9 -> 18.6,
// 256x256 27.7 -> 22.4, 512x512 93 -> 82, 1000x500 180 -> 172, 2048x1024 700 -> 697.
// Tiles 8x4 have the smaller ring, 16x2 the longer rows: up to RG_MAX_BLOCKS
// blocks of 16x2 the ring decides (64x64 6.6 against 7.1 us, 400x400, 5226
// blocks, 44.8 against 45.9), beyond, where the planes no longer stay in the
// caches, the rows (512x512, 8481 blocks, 87 against 82; 1000x500 187 against 172).
// ---------------------------------------------------------------------------
constexpr int RG_CELLS = 32;
constexpr unsigned RG_MAX_BLOCKS = 6144;

template <int TX, int TY, bool VarMu>
__global__ __launch_bounds__(6 * RG_CELLS) void k_rgrad2(Batch bt) {
    constexpr int RG_TX = TX, RG_TY = TY;
    constexpr int RG_RX = RG_TX + 2, RG_RY = RG_TY + 2;                         // tile + ring
    constexpr int RG_NXF = RG_RY * (RG_RX + 1), RG_NYF = (RG_RY + 1) * RG_RX;   // faces
    constexpr int RG_LDS = 6 * (RG_NXF + RG_NYF) + 18 * RG_RY * RG_RX;
    static_assert(TX * TY == RG_CELLS && RG_LDS >= 3 * 64 + GW_MU, "three wavefronts per tile");
    // phase 1: hx[6][RY][RX + 1] and hy[6][RY + 1][RX] (W0 for w = 0..2, then
    // W1), rbs[18][RY][RX] (index (l * 3 + w) * 3 + moment); phase 2: the
    // gradient body's exchange over the same memory
    __shared__ double lds[RG_LDS];
    double* const hx = lds;
    double* const hy = hx + 6 * RG_NXF;
    double* const rbs = hy + 6 * RG_NYF;
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const long long N = g.ncell;
    const int tiles_x = (g.NX - 6 + RG_TX - 1) / RG_TX;
    const int i0 = 3 + (lc.b % tiles_x) * RG_TX;   // first cell of the tile
    const int j0 = 3 + (lc.b / tiles_x) * RG_TY;
    constexpr int NT = 6 * RG_CELLS;
    // w-bar of the ring's cells, one task per (cell, l, w), asked for ahead of
    // the faces
    constexpr int NR = RG_RY * RG_RX, NQ = (6 * NR + NT - 1) / NT;
    double wb[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int t = threadIdx.x + q * NT, rc = t % NR;
        const int j = min(j0 - 1 + rc / RG_RX, g.NY - 3), i = min(i0 - 1 + rc % RG_RX, g.NX - 3);
        if (t < 6 * NR) wb[q] = g.wb[(t / NR) * N + (long long)j * g.NX + i];
    }
    // interface data of the faces of the ring's cells (j0 - 1 + r, i0 - 1 + c);
    // cells of weak moments lie in rows and columns 2 .. N - 3
    for (int t = threadIdx.x; t < RG_NXF + RG_NYF; t += NT) {
        const bool xd = t < RG_NXF;
        const int q = xd ? t : t - RG_NXF;
        int r, c, i, j, ilo, jlo;
        if (xd) {   // face i - 1/2 of row j
            r = q / (RG_RX + 1);
            c = q % (RG_RX + 1);
            j = j0 - 1 + r;
            i = i0 - 1 + c;
            ilo = i - 1;
            jlo = j;
            if (j > g.NY - 3 || i > g.NX - 2) continue;
        } else {    // face j - 1/2 of column i
            r = q / RG_RX;
            c = q % RG_RX;
            j = j0 - 1 + r;
            i = i0 - 1 + c;
            ilo = i;
            jlo = j - 1;
            if (i > g.NX - 3 || j > g.NY - 2) continue;
        }
        double W0[3], W1[3];
        face_wavg(xd ? g.xf : g.yf, N, (long long)jlo * g.NX + ilo, (long long)j * g.NX + i, W0,
                  W1);
        double* H = xd ? hx : hy;
        const int plane = xd ? RG_NXF : RG_NYF;
#pragma unroll
        for (int w = 0; w < 3; ++w) {
            H[w * plane + q] = W0[w];
            H[(3 + w) * plane + q] = W1[w];
        }
    }
    __syncthreads();
    // weak moments of the ring's cells
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int t = threadIdx.x + q * NT;
        const int lw = t / NR, rc = t % NR;
        const int l = lw / 3, w = lw % 3;
        const int r = rc / RG_RX, c = rc % RG_RX;
        if (t >= 6 * NR || j0 - 1 + r > g.NY - 3 || i0 - 1 + c > g.NX - 3) continue;
        double W0lo, W0hi, W1lo, W1hi;
        if (l == 0) {
            const int f = r * (RG_RX + 1) + c;
            W0lo = hx[w * RG_NXF + f];
            W0hi = hx[w * RG_NXF + f + 1];
            W1lo = hx[(3 + w) * RG_NXF + f];
            W1hi = hx[(3 + w) * RG_NXF + f + 1];
        } else {
            const int f = r * RG_RX + c;
            W0lo = hy[w * RG_NYF + f];
            W0hi = hy[w * RG_NYF + f + RG_RX];
            W1lo = hy[(3 + w) * RG_NYF + f];
            W1hi = hy[(3 + w) * RG_NYF + f + RG_RX];
        }
        double m[3];
        cell_wmom(W0lo, W0hi, W1lo, W1hi, wb[q],
                  l ? g.K.idy : g.K.idx, l, m);
#pragma unroll
        for (int k = 0; k < 3; ++k) rbs[(lw * 3 + k) * (RG_RY * RG_RX) + rc] = m[k];
    }
    __syncthreads();
    // gradient reconstruction: cell cl of the tile, variable w, direction l
    const int cl = threadIdx.x & 31;
    const int k = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = (threadIdx.x >> 5) & 1, w = pair_var(k, l);
    const int ty = cl / RG_TX, tx = cl % RG_TX;
    const int j = j0 + ty, i = i0 + tx;
    const bool valid = j <= g.NY - 4 && i <= g.NX - 4;
    const double* R = rbs + (long long)((l * 3 + w) * 3) * (RG_RY * RG_RX);
    double a[17];
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const int o = (ty + 1 + q / 3 - 1) * RG_RX + (tx + 1 + q % 3 - 1);
        a[q] = valid ? R[o] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = 2 * e + 1;
        const int o = (ty + 1 + q / 3 - 1) * RG_RX + (tx + 1 + q % 3 - 1);
        a[9 + e] = valid ? R[RG_RY * RG_RX + o] : 0.0;
        a[13 + e] = valid ? R[2 * RG_RY * RG_RX + o] : 0.0;
    }
    __syncthreads();   // the weak moments are in registers; the exchange reuses the LDS
    grad_body<VarMu, false>(g, lds, a, k, valid, valid ? j : 3, valid ? i : 3);
}

// The two Gauss moments of a face flux that the assembly of eq. (3.2) takes
// from a face, per component: A = sum_G w_G F_G and B = sum_G w_G x_G F_G
// (x_G = -s, 0, s in face units).  One definition for every kernel.
// Both are written so that exchanging the outer points (a mirror image of
// the face) gives the same A and the negated B bit for bit.
__device__ __forceinline__ void face_moments(double F0, double F1, double F2, double& A,
                                             double& B) {
#pragma clang fp contract(off)
    A = fma(GW0, F0 + F2, GW1 * F1);
    B = (GW0 * GS) * (F2 - F0);
}

// The three gradient combinations of face point p (0..5 x-face, 6..11
// y-face; direction d of that face) of a cell: read as stored, or formed from
// the six gradients of the full layout.
template <int d, bool FULL>
__device__ __forceinline__ void face_grad(const Grid2& g, int p, long long cell, double* dc) {
    const long long N = g.ncell;
    if constexpr (FULL) {
        double sq[6];
#pragma unroll
        for (int z = 0; z < 6; ++z) sq[z] = g.gf[(p * 6 + z) * N + cell];
        stress_combos<d>(sq, dc);
    } else {
#pragma unroll
        for (int z = 0; z < 3; ++z) dc[z] = g.gf[(p * 3 + z) * N + cell];
    }
}

// ---------------------------------------------------------------------------
// Face fluxes (eq. (3.3)): x-faces (j, i+1/2) for interior rows, i from the
// last ghost column; y-faces (j+1/2, i) likewise.  The LF coefficient is the
// max over the face's three Gauss points and both sides.
// ---------------------------------------------------------------------------
template <int d, int FX_FACES, bool VarMu, bool FULL>   // block = 3 Gauss points x FX_FACES faces
__global__ __launch_bounds__(3 * FX_FACES) void k_flux2(Batch bt) {
    __shared__ double shb[3 * FX_FACES];
    __shared__ double shf[4][3 * FX_FACES];
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const Consts& K = g.K;
    const int nfi = d == 0 ? g.nx + 1 : g.nx;
    const int nfj = d == 0 ? g.ny : g.ny + 1;
    const int G = threadIdx.x / FX_FACES;
    const int fl = threadIdx.x % FX_FACES;
    const long long t = (long long)lc.b * FX_FACES + fl;
    const bool valid = t < (long long)nfi * nfj;
    const long long N = g.ncell;
    long long cm = 0, cp = 0;
    double fs[4] = {0.0, 0.0, 0.0, 0.0}, du[4] = {0.0, 0.0, 0.0, 0.0};
    double beta = -INFINITY;
    if (valid) {
        const int fj = (int)(t / nfi), fi = (int)(t % nfi);
        const int j = d == 0 ? HALO + fj : HALO - 1 + fj;
        const int i = d == 0 ? HALO - 1 + fi : HALO + fi;
        cm = (long long)j * g.NX + i;
        cp = d == 0 ? cm + 1 : cm + g.NX;
        const double* F = d == 0 ? g.xf : g.yf;
        const int pg = d == 0 ? 0 : 6;
        double Um[4], Up[4], sm[3], sp[3], fm[4], fp[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            Um[c] = F[((3 + G) * 4 + c) * N + cm];
            Up[c] = F[(G * 4 + c) * N + cp];
        }
        face_grad<d, FULL>(g, pg + 3 + G, cm, sm);
        face_grad<d, FULL>(g, pg + G, cp, sp);
        beta = fmax(flux_speed2c<d, VarMu>(K, Um, sm, fm), flux_speed2c<d, VarMu>(K, Up, sp, fp));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            fs[c] = fm[c] + fp[c];
            du[c] = Up[c] - Um[c];
        }
    }
    shb[threadIdx.x] = beta;
    __syncthreads();
    // LF coefficient: max over the face's three Gauss points and both sides
    beta = fmax(fmax(shb[fl], shb[FX_FACES + fl]), shb[2 * FX_FACES + fl]);
    // the face's Gauss moments: the three points meet in LDS
#pragma unroll
    for (int c = 0; c < 4; ++c) shf[c][threadIdx.x] = 0.5 * fma(-beta, du[c], fs[c]);
    __syncthreads();
    if (valid && G == 0) {
        double* out = d == 0 ? g.fx : g.fy;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            double A, B;
            face_moments(shf[c][fl], shf[c][FX_FACES + fl], shf[c][2 * FX_FACES + fl], A, B);
            out[c * N + cm] = A;
            out[(4 + c) * N + cm] = B;
        }
    }
    red_max<3 * FX_FACES>(&g.red->beta_key, valid && G == 0 ? beta : -INFINITY);
}

// ---------------------------------------------------------------------------
// Assembly (eq. (3.2)) and stage update (eq. (2.12) in 2D form) of interior
// cell (ii, jj), t = jj * nx + ii.  ff(c, L, R, Bo, T) gives the Gauss
// moments (A, B) of component c of the fluxes of the cell's left, right,
// bottom and top faces (L[0] = A, L[1] = B, ...).  stage 0: R and Vhat out
// (interior layout); stage 1..3: SSP-RK3 stage.  rmin, pmin and bad receive
// the cell's share of the admissibility reductions (stages 1..3; solid cells
// give none).
// ---------------------------------------------------------------------------
// Component c of it: L, R, Bo and T as above.  nw: the new average and moments
// (stages 1..3) or the residual (stage 0), vh: the modified moments; stored by
// store_comp, so that a thread with several components issues every load
// before its first store.
__device__ __forceinline__ void update_comp(const Grid2& g, const Grid2& gsrc, long long t,
                                            long long cell, int c, int stage, int i0, int iin,
                                            double dt, const double* __restrict__ src,
                                            const double* L, const double* R, const double* Bo,
                                            const double* T, double* nw, double* vh) {
    // explicit fused multiply-adds, no automatic contraction: the same
    // rounding whichever kernel inlines this
#pragma clang fp contract(off)
    const double* __restrict__ S0 = gsrc.S[i0];
    const double* __restrict__ Sin = gsrc.S[iin];
    const long long nint = (long long)g.nx * g.ny;
    const long long N = g.ncell;
    const double idx = g.K.idx, idy = g.K.idy;
    const double dfx = R[0] - L[0], sfx = L[0] + R[0], dfxe = R[1] - L[1];
    const double dgy = T[0] - Bo[0], sgy = Bo[0] + T[0], dgyx = T[1] - Bo[1];
    double Fm[3];
    Fm[0] = fma(-dfx, idx, -dgy * idy);
    Fm[1] = fma(g.vf[c * N + cell], idx, fma(-sfx, 0.5 * idx, -dgyx * idy));
    Fm[2] = fma(g.vf[(4 + c) * N + cell], idy, fma(-dfxe, idx, -sgy * (0.5 * idy)));
    if (src) {   // prescribed source moments (layout of R; single grid)
#pragma unroll
        for (int m = 0; m < 3; ++m) Fm[m] += src[(m * 4 + c) * nint + t];
    }
    vh[0] = g.vk[c * N + cell];
    vh[1] = g.vk[(4 + c) * N + cell];
    if (stage == 0) {
#pragma unroll
        for (int m = 0; m < 3; ++m) nw[m] = Fm[m];
        return;
    }
    const double in0 = Sin[c * N + cell];
    if (stage == 1) {
        nw[0] = fma(dt, Fm[0], in0);
        nw[1] = fma(dt, Fm[1], vh[0]);
        nw[2] = fma(dt, Fm[2], vh[1]);
    } else {
        const double a = stage == 2 ? 0.75 : 1.0 / 3.0;
        const double bb = stage == 2 ? 0.25 : 2.0 / 3.0;
        nw[0] = fma(a, S0[c * N + cell], bb * fma(dt, Fm[0], in0));
        nw[1] = fma(a, g.vn[c * N + cell], bb * fma(dt, Fm[1], vh[0]));
        nw[2] = fma(a, g.vn[(4 + c) * N + cell], bb * fma(dt, Fm[2], vh[1]));
    }
}

__device__ __forceinline__ void reset_reduce(Reduce* r) {
    r->alpha_key = dkey(-INFINITY);
    r->beta_key = dkey(-INFINITY);
    r->pp_cells = 0;
    r->min_rho_key = dkey(INFINITY);
    r->min_p_key = dkey(INFINITY);
    r->bad[0] = r->bad[1] = r->bad[2] = r->bad[3] = 0;
}

// Step size of an update (StepRule).  In stage 1 every thread forms it from the
// wave speed, which no kernel after that stage's reconstruction changes;
// publish_step leaves it in the slots.
__device__ __forceinline__ double step_dt(const Grid2& g, const StepRule& r) {
    if (r.mode == 0) return g.red->dt;
    if (r.mode == 2) return r.dt;
    return fmin(fmin(r.cfl_h / dkey_inv(g.red->alpha_key), r.visc_dt), r.t_left);
}
__device__ __forceinline__ void publish_step(const Grid2& g, const StepRule& r, int block) {
    if (r.mode == 0 || block != 0 || threadIdx.x != 0) return;
    g.red->dt = step_dt(g, r);
    g.red->alpha1_key = g.red->alpha_key;
    if (r.clear) reset_reduce(r.clear);
}

__device__ __forceinline__ void store_comp(const Grid2& g, const Grid2& gsrc, long long t,
                                           long long cell, int c, int stage, int iout,
                                           double* __restrict__ Rout, double* __restrict__ Vout,
                                           const double* nw, const double* vh) {
    const long long nint = (long long)g.nx * g.ny;
    const long long N = g.ncell;
    if (stage == 0) {
#pragma unroll
        for (int m = 0; m < 3; ++m) Rout[(m * 4 + c) * nint + t] = nw[m];
        Vout[c * nint + t] = vh[0];
        Vout[(4 + c) * nint + t] = vh[1];
        return;
    }
    double* __restrict__ Sout = gsrc.S[iout];
#pragma unroll
    for (int m = 0; m < 3; ++m) Sout[(m * 4 + c) * N + cell] = nw[m];
    if (stage == 1) {   // kept for stages 2 and 3
        g.vn[c * N + cell] = vh[0];
        g.vn[(4 + c) * N + cell] = vh[1];
    }
}

// Solid cell of a masked domain: no residual, keeps the stage input, not
// checked.  Component c.
__device__ __forceinline__ void update_solid(const Grid2& g, const Grid2& gsrc, long long t,
                                             long long cell, int c, int stage, int iin, int iout,
                                             double* __restrict__ Rout,
                                             double* __restrict__ Vout) {
    const double* __restrict__ Sin = gsrc.S[iin];
    double* __restrict__ Sout = gsrc.S[iout];
    const long long nint = (long long)g.nx * g.ny;
    const long long N = g.ncell;
    if (stage == 0) {
#pragma unroll
        for (int m = 0; m < 3; ++m) Rout[(m * 4 + c) * nint + t] = 0.0;
        Vout[c * nint + t] = 0.0;
        Vout[(4 + c) * nint + t] = 0.0;
    } else {
#pragma unroll
        for (int m = 0; m < 3; ++m)
            Sout[(m * 4 + c) * N + cell] = Sin[(m * 4 + c) * N + cell];
    }
}

template <class FF>
__device__ __forceinline__ void update_cell(const Grid2& g, const Grid2& gsrc, long long t, int jj,
                                            int ii, int stage, int i0, int iin, int iout,
                                            double* __restrict__ Rout,
                                            double* __restrict__ Vout,
                                            const double* __restrict__ src, double dt,
                                            const FF& ff, double& rmin, double& pmin,
                                            unsigned int& bad) {
    const long long cell = (long long)(jj + HALO) * g.NX + ii + HALO;
    if (gsrc.solid && gsrc.solid[t]) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            update_solid(g, gsrc, t, cell, c, stage, iin, iout, Rout, Vout);
        return;
    }
    double nw[4][3], vh[4][2];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double L[2], R[2], Bo[2], T[2];
        ff(c, L, R, Bo, T);
        update_comp(g, gsrc, t, cell, c, stage, i0, iin, dt, src, L, R, Bo, T, nw[c], vh[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        store_comp(g, gsrc, t, cell, c, stage, iout, Rout, Vout, nw[c], vh[c]);
    if (stage == 0) return;
    const double p = pressure2(g.K, nw[0][0], nw[1][0], nw[2][0], nw[3][0]);
    rmin = nw[0][0];
    pmin = p;
    bool ok = nw[0][0] > 0.0 && p > 0.0;
#pragma unroll
    for (int q = 0; q < 12; ++q) ok = ok && isfinite(nw[q / 3][q % 3]);
    bad = ok ? 0u : 1u;
}

// Split path: the face fluxes come from k_flux2 through HBM.
__global__ __launch_bounds__(256) void k_update2(Batch bt, int stage, int i0, int iin, int iout,
                                                 double* __restrict__ Rout,
                                                 double* __restrict__ Vout,
                                                 const double* __restrict__ src,
                                                 StepRule rule) {
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    publish_step(g, rule, lc.b);
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)lc.b * blockDim.x + threadIdx.x;
    double rmin = INFINITY, pmin = INFINITY;
    unsigned int bad = 0;
    if (t < nint) {
        const int jj = (int)(t / g.nx), ii = (int)(t % g.nx);
        const long long N = g.ncell;
        const long long cell = (long long)(jj + HALO) * g.NX + ii + HALO;
        auto ff = [&](int c, double* L, double* R, double* Bo, double* T) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                R[m] = g.fx[(4 * m + c) * N + cell];
                L[m] = g.fx[(4 * m + c) * N + cell - 1];
                T[m] = g.fy[(4 * m + c) * N + cell];
                Bo[m] = g.fy[(4 * m + c) * N + cell - g.NX];
            }
        };
        update_cell(g, gsrc, t, jj, ii, stage, i0, iin, iout, Rout, Vout, src,
                    stage > 0 ? step_dt(g, rule) : 0.0, ff, rmin, pmin, bad);
    }
    if (stage > 0) reduce_update<256>(gsrc.red, stage, -INFINITY, rmin, pmin, bad != 0);
}

// ---------------------------------------------------------------------------
// Face fluxes fused with the assembly and the stage update.  A block of 256
// threads owns a tile of FU_TX x FU_TY cells (columns aligned to multiples of
// FU_TX in the ghosted grid; ghost cells in it stay idle).  First the two
// Gauss moments of the flux of every face of the tile go to LDS: thread
// (tx, ty) forms the x-face left of its cell and the y-face below it, and one
// more pass forms the x-faces right of the tile and the y-faces above it.
// Then each thread assembles and updates its cell.  A face on a tile edge is
// formed by both tiles that share it.  The arithmetic per face and per cell
// is that of k_flux2 and k_update2, so the two paths give the same bits.
// Constant viscosity, large launches; the others take k_fluxup2s below.
// ---------------------------------------------------------------------------
constexpr int FU_TX = 32, FU_TY = 8;

// Gauss moments (A into o[c * stride], B into o[(4 + c) * stride]) of the
// flux of the face between cells cm and cp (direction d); returns the LF
// coefficient (max over the three points and both sides).
template <int d, bool FULL>
__device__ __forceinline__ double face_flux3(const Grid2& g, long long cm, long long cp,
                                             double* o, int stride) {
    const Consts& K = g.K;
    const long long N = g.ncell;
    const double* F = d == 0 ? g.xf : g.yf;
    const int pg = d == 0 ? 0 : 6;
    double fs[3][4], du[3][4], bg[3];
#pragma unroll
    for (int G = 0; G < 3; ++G) {
        double Um[4], Up[4], sm[3], sp[3], fm[4], fp[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            Um[c] = F[((3 + G) * 4 + c) * N + cm];
            Up[c] = F[(G * 4 + c) * N + cp];
        }
        face_grad<d, FULL>(g, pg + 3 + G, cm, sm);
        face_grad<d, FULL>(g, pg + G, cp, sp);
        bg[G] = fmax(flux_speed2c<d, false>(K, Um, sm, fm), flux_speed2c<d, false>(K, Up, sp, fp));
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            fs[G][c] = fm[c] + fp[c];
            du[G][c] = Up[c] - Um[c];
        }
    }
    const double beta = fmax(fmax(bg[0], bg[1]), bg[2]);
    double Fg[3][4];   // the flux at each Gauss point
#pragma unroll
    for (int G = 0; G < 3; ++G)
#pragma unroll
        for (int c = 0; c < 4; ++c) Fg[G][c] = 0.5 * fma(-beta, du[G][c], fs[G][c]);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        face_moments(Fg[0][c], Fg[1][c], Fg[2][c], o[c * stride], o[(4 + c) * stride]);
    return beta;
}

template <bool FULL>
__global__ __launch_bounds__(FU_TX * FU_TY) void k_fluxup2(Batch bt, int stage, int i0, int iin,
                                                           int iout, double* __restrict__ Rout,
                                                           double* __restrict__ Vout,
                                                           const double* __restrict__ src,
                                                           StepRule rule) {
    constexpr int RX = FU_TX + 1;                              // x-face columns per row
    constexpr int SX = FU_TY * RX, SY = (FU_TY + 1) * FU_TX;   // plane sizes
    __shared__ double lx[8 * SX];    // [moment*4 + c][row][face column 0..FU_TX]
    __shared__ double ly[8 * SY];    // [moment*4 + c][face row 0..FU_TY][column]
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    publish_step(g, rule, lc.b);
    // tiles start at multiples of FU_TX columns of the ghosted grid, so that
    // their row segments are whole cache lines; the first tile's leading
    // columns are ghost cells and stay idle
    const int tiles_x = (g.nx + HALO + FU_TX - 1) / FU_TX;
    const int ii0 = (lc.b % tiles_x) * FU_TX - HALO, jj0 = (lc.b / tiles_x) * FU_TY;
    const int tx = threadIdx.x % FU_TX, ty = threadIdx.x / FU_TX;
    double bmax = -INFINITY;
    // x-face left of interior cell (ii0 + fc, jj0 + row); fc = FU_TX and
    // ii = nx (the domain's right boundary face) included
    auto xface = [&](int fc, int row) {
        const int ii = ii0 + fc, jj = jj0 + row;
        if (ii < 0 || ii > g.nx || jj >= g.ny) return;
        const long long cp = (long long)(jj + HALO) * g.NX + ii + HALO;
        bmax = fmax(bmax, face_flux3<0, FULL>(g, cp - 1, cp, lx + row * RX + fc, SX));
    };
    // y-face below interior cell (ii0 + col, jj0 + fr); fr = FU_TY and jj = ny
    // included
    auto yface = [&](int fr, int col) {
        const int ii = ii0 + col, jj = jj0 + fr;
        if (ii < 0 || ii >= g.nx || jj > g.ny) return;
        const long long cp = (long long)(jj + HALO) * g.NX + ii + HALO;
        bmax = fmax(bmax, face_flux3<1, FULL>(g, cp - g.NX, cp, ly + fr * FU_TX + col, SY));
    };
    xface(tx, ty);
    yface(ty, tx);
    if (threadIdx.x < FU_TX) yface(FU_TY, threadIdx.x);                  // wavefront 0
    else if (threadIdx.x >= 64 && threadIdx.x < 64 + FU_TY) xface(FU_TX, threadIdx.x - 64);
    __syncthreads();
    const int ii = ii0 + tx, jj = jj0 + ty;
    double rmin = INFINITY, pmin = INFINITY;
    unsigned int bad = 0;
    if (ii >= 0 && ii < g.nx && jj < g.ny) {
        auto ff = [&](int c, double* L, double* R, double* Bo, double* T) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const int q = 4 * m + c;
                L[m] = lx[q * SX + ty * RX + tx];
                R[m] = lx[q * SX + ty * RX + tx + 1];
                Bo[m] = ly[q * SY + ty * FU_TX + tx];
                T[m] = ly[q * SY + (ty + 1) * FU_TX + tx];
            }
        };
        update_cell(g, gsrc, (long long)jj * g.nx + ii, jj, ii, stage, i0, iin, iout, Rout, Vout,
                    src, stage > 0 ? step_dt(g, rule) : 0.0, ff, rmin, pmin, bad);
    }
    reduce_update<FU_TX * FU_TY>(gsrc.red, stage, bmax, rmin, pmin, bad != 0);
}

// The same with less work per thread: tiles of FU_TX x FS_TY cells, and a
// thread forms the flux at one Gauss point of one face instead of a whole face,
// then one component of one cell.  Same arithmetic, so the same bits.
// Small launches are bound by the latency of one block (its chain of loads and
// divisions), which this cuts: 64^2 15.8 -> 9.9 us, 104x88 14.5 -> 9.5,
// 500x100 17.4 -> 15.9, 256^2 21.5 -> 21.0, 360^2 32.5 -> 31.8; large ones move
// at the memory's rate with whole faces (1000x500 116 us, 5.3 TB/s, against
// 126 here: a third more edge faces are formed twice), so the line lies
// between 360^2 (540 blocks of the other kernel) and 512^2 (1088 blocks, 64
// against 69 us).  With mu(T) the power law's registers leave the whole-face
// kernel two wavefronts per SIMD, and this one is faster at every size (64^2
// 36 -> 17 us, 1000x500 158 -> 149).
constexpr int FS_TY = 4, FS_NT = 512;
constexpr unsigned FS_MAX_BLOCKS = 640;   // of k_fluxup2

// Flux sums of Gauss point G of the face between cells cm and cp (direction d):
// f- + f+ and U+ - U-; returns the larger wave-speed bound of the two sides.
template <int d, bool VarMu, bool FULL>
__device__ __forceinline__ double face_point(const Grid2& g, long long cm, long long cp, int G,
                                             double* fs, double* du) {
    const Consts& K = g.K;
    const long long N = g.ncell;
    const double* F = d == 0 ? g.xf : g.yf;
    const int pg = d == 0 ? 0 : 6;
    double Um[4], Up[4], sm[3], sp[3], fm[4], fp[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        Um[c] = F[((3 + G) * 4 + c) * N + cm];
        Up[c] = F[(G * 4 + c) * N + cp];
    }
    face_grad<d, FULL>(g, pg + 3 + G, cm, sm);
    face_grad<d, FULL>(g, pg + G, cp, sp);
    const double b = fmax(flux_speed2c<d, VarMu>(K, Um, sm, fm),
                          flux_speed2c<d, VarMu>(K, Up, sp, fp));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        fs[c] = fm[c] + fp[c];
        du[c] = Up[c] - Um[c];
    }
    return b;
}

template <bool VarMu, bool FULL>
__global__ __launch_bounds__(FS_NT) void k_fluxup2s(Batch bt, int stage, int i0, int iin, int iout,
                                                    double* __restrict__ Rout,
                                                    double* __restrict__ Vout,
                                                    const double* __restrict__ src,
                                                    StepRule rule) {
    constexpr int RX = FU_TX + 1;                              // x-face columns per row
    constexpr int NXF = FS_TY * RX, NYF = (FS_TY + 1) * FU_TX, NF = NXF + NYF;
    constexpr int NT = 3 * NF, NIT = (NT + FS_NT - 1) / FS_NT;
    __shared__ double shb[NT];        // wave-speed bound per Gauss point and face
    __shared__ double shf[4][NT];     // flux per component, Gauss point and face
    __shared__ double shu[4][FS_TY * FU_TX];   // new averages, for the admissibility check
    __shared__ unsigned char shk[4][FS_TY * FU_TX];
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    publish_step(g, rule, lc.b);
    const int tiles_x = (g.nx + HALO + FU_TX - 1) / FU_TX;
    const int ii0 = (lc.b % tiles_x) * FU_TX - HALO, jj0 = (lc.b / tiles_x) * FS_TY;
    double fs[NIT][4] = {}, du[NIT][4] = {}, bmax = -INFINITY;
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int t = threadIdx.x + it * FS_NT;
        const int G = t / NF, f = t - G * NF;
        if (t >= NT) continue;
        double b = -INFINITY;
        if (f < NXF) {   // x-face left of interior cell (ii, jj)
            const int ii = ii0 + f % RX, jj = jj0 + f / RX;
            if (ii >= 0 && ii <= g.nx && jj < g.ny) {
                const long long cp = (long long)(jj + HALO) * g.NX + ii + HALO;
                b = face_point<0, VarMu, FULL>(g, cp - 1, cp, G, fs[it], du[it]);
            }
        } else {         // y-face below it
            const int ii = ii0 + (f - NXF) % FU_TX, jj = jj0 + (f - NXF) / FU_TX;
            if (ii >= 0 && ii < g.nx && jj <= g.ny) {
                const long long cp = (long long)(jj + HALO) * g.NX + ii + HALO;
                b = face_point<1, VarMu, FULL>(g, cp - g.NX, cp, G, fs[it], du[it]);
            }
        }
        shb[t] = b;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int t = threadIdx.x + it * FS_NT;
        if (t >= NT) continue;
        const int f = t % NF;
        const double beta = fmax(fmax(shb[f], shb[NF + f]), shb[2 * NF + f]);
        bmax = fmax(bmax, beta);
#pragma unroll
        for (int c = 0; c < 4; ++c) shf[c][t] = 0.5 * fma(-beta, du[it][c], fs[it][c]);
    }
    __syncthreads();
    // thread (c, cell): component c of the tile's cell
    const int c = threadIdx.x / (FS_TY * FU_TX), ct = threadIdx.x % (FS_TY * FU_TX);
    const int tx = ct % FU_TX, ty = ct / FU_TX;
    const int ii = ii0 + tx, jj = jj0 + ty;
    const bool in = ii >= 0 && ii < g.nx && jj < g.ny;
    const long long t = (long long)jj * g.nx + ii;
    const bool solid = in && gsrc.solid && gsrc.solid[t];
    if (in) {
        const long long cell = (long long)(jj + HALO) * g.NX + ii + HALO;
        if (solid) {
            update_solid(g, gsrc, t, cell, c, stage, iin, iout, Rout, Vout);
        } else {
            auto mom = [&](int f, double* o) {
                face_moments(shf[c][f], shf[c][NF + f], shf[c][2 * NF + f], o[0], o[1]);
            };
            double L[2], R[2], Bo[2], T[2], nw[3], vh[2];
            mom(ty * RX + tx, L);
            mom(ty * RX + tx + 1, R);
            mom(NXF + ty * FU_TX + tx, Bo);
            mom(NXF + (ty + 1) * FU_TX + tx, T);
            update_comp(g, gsrc, t, cell, c, stage, i0, iin, stage > 0 ? step_dt(g, rule) : 0.0,
                        src, L, R, Bo, T, nw, vh);
            store_comp(g, gsrc, t, cell, c, stage, iout, Rout, Vout, nw, vh);
            shu[c][ct] = nw[0];
            shk[c][ct] = isfinite(nw[0]) && isfinite(nw[1]) && isfinite(nw[2]);
        }
    }
    __syncthreads();
    double rmin = INFINITY, pmin = INFINITY;
    bool bad = false;
    if (stage > 0 && c == 0 && in && !solid) {
        rmin = shu[0][ct];
        pmin = pressure2(g.K, rmin, shu[1][ct], shu[2][ct], shu[3][ct]);
        bad = !(rmin > 0.0 && pmin > 0.0 && shk[0][ct] && shk[1][ct] && shk[2][ct] && shk[3][ct]);
    }
    reduce_update<FS_NT>(gsrc.red, stage, bmax, rmin, pmin, bad);
}

__global__ void k_copy_in2(Grid2 g, const double* __restrict__ U, double* __restrict__ S) {
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nint * 12) return;
    const int q = (int)(t / nint);
    const long long r = t % nint;
    const int jj = (int)(r / g.nx), ii = (int)(r % g.nx);
    S[q * g.ncell + (long long)(jj + HALO) * g.NX + ii + HALO] = U[t];
}

__global__ void k_copy_out2(Grid2 g, const double* __restrict__ S, double* __restrict__ U) {
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nint * 12) return;
    const int q = (int)(t / nint);
    const long long r = t % nint;
    const int jj = (int)(r / g.nx), ii = (int)(r % g.nx);
    U[t] = S[q * g.ncell + (long long)(jj + HALO) * g.NX + ii + HALO];
}

// Input admissibility (finite values, positive density and pressure).
__global__ __launch_bounds__(256) void k_check2(Batch bt, int si) {
    const Loc lc = locate(bt);
    const Grid2& gsrc = bt.g[lc.p];   // arrays indexed at run time are read from here
    if (!gsrc.st->active) return;
    const Grid2 g = gsrc;
    const double* __restrict__ S = gsrc.S[si];
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)lc.b * blockDim.x + threadIdx.x;
    unsigned int bad = 0;
    if (t < nint && !(gsrc.solid && gsrc.solid[t])) {
        const int jj = (int)(t / g.nx), ii = (int)(t % g.nx);
        const long long cell = (long long)(jj + HALO) * g.NX + ii + HALO;
        double q[12];
        bool ok = true;
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            q[k] = S[k * g.ncell + cell];
            ok = ok && isfinite(q[k]);
        }
        ok = ok && q[0] > 0.0 && pressure2(g.K, q[0], q[1], q[2], q[3]) > 0.0;
        bad = ok ? 0u : 1u;
    }
    red_add32<256>(&g.red->bad[0], bad);
}

__global__ void k_reset(Reduce* r) {
    if (threadIdx.x == 0) reset_reduce(r);
}

__global__ void k_set_dt(Reduce* r, double dt) {
    if (threadIdx.x == 0) {
        r->alpha1_key = r->alpha_key;
        r->dt = dt;
    }
}

// Places the descriptors of an allocation-free call and resets its reductions:
// one launch, the descriptors its arguments (three copies from pageable memory
// and a reset, before).
__global__ __launch_bounds__(256) void k_place2(Place2 a) {
    auto put = [&](void* to, const void* from, int bytes) {
        for (int k = threadIdx.x; k < bytes / 4; k += 256)
            ((unsigned*)to)[k] = ((const unsigned*)from)[k];
    };
    put(a.dg, &a.g, sizeof(a.g));
    put(a.dst, &a.st, sizeof(a.st));
    put(a.dstart, a.start, sizeof(a.start));
    if (threadIdx.x == 0) reset_reduce((Reduce*)a.g.red);
}

// Per-instance kernels of a batch: thread p serves the instance in slot p.
__global__ void k_reset2(const Grid2* __restrict__ gs, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < n) reset_reduce((Reduce*)gs[p].red);
}

// Trial step of the time-step rule from the stage-1 wave speed, halved once
// per rejected attempt of the current step.
__global__ void k_dt2(const Grid2* __restrict__ gs, int n) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const InstState* st = gs[p].st;
    if (!st->active) return;
    Reduce* r = gs[p].red;
    r->alpha1_key = r->alpha_key;
    double dt = fmin(st->cfl_h / dkey_inv(r->alpha_key), st->visc_dt);
    if (st->t_final > 0.0) dt = fmin(dt, st->t_final - st->t);
    r->dt = ldexp(dt, -st->halvings);
}

__device__ __forceinline__ bool accepted(const Grid2& g) {
    const Reduce* r = g.red;
    const double dt = r->dt;
    return r->bad[1] == 0 && r->bad[2] == 0 && r->bad[3] == 0 && dt > 0.0 && isfinite(dt);
}

// Accepted instances: interior of S[1] (the stage-3 output) -> S[0].
__global__ __launch_bounds__(256) void k_commit_copy(Batch bt) {
    const Loc lc = locate(bt);
    const Grid2 g = bt.g[lc.p];
    if (!g.st->active || !accepted(g)) return;
    const long long nint = (long long)g.nx * g.ny;
    const long long t = (long long)lc.b * blockDim.x + threadIdx.x;
    if (t >= nint) return;
    const int jj = (int)(t / g.nx), ii = (int)(t % g.nx);
    const long long cell = (long long)(jj + HALO) * g.NX + ii + HALO;
#pragma unroll
    for (int q = 0; q < 12; ++q) g.S[0][q * g.ncell + cell] = g.S[1][q * g.ncell + cell];
}

__global__ void k_commit_state(const Grid2* __restrict__ gs, int n, int code_inadmissible,
                               int code_nonfinite) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const Grid2& g = gs[p];
    InstState* st = g.st;
    if (!st->active) return;
    const Reduce* r = g.red;
    st->alpha = dkey_inv(r->alpha1_key);
    st->beta_max = dkey_inv(r->beta_key);
    st->min_rho = dkey_inv(r->min_rho_key);
    st->min_p = dkey_inv(r->min_p_key);
    if (!(r->dt > 0.0) || !isfinite(r->dt)) {
        // no usable step size (a non-finite wave speed): stop the instance
        // as the single-grid driver stops, instead of halving a NaN
        st->status = code_nonfinite;
        st->active = 0;
        return;
    }
    if (accepted(g)) {
        st->t += r->dt;
        st->dt_last = r->dt;
        st->steps += 1;
        st->halvings = 0;
        st->pp_cells += r->pp_cells;
        const bool at_end = st->t_final > 0.0 && !(st->t < st->t_final);
        if (st->steps >= st->target || at_end) st->active = 0;
    } else {
        st->restarts += 1;
        if (st->halvings >= st->max_halvings) {
            st->status = code_inadmissible;
            st->active = 0;
        } else {
            st->halvings += 1;
        }
    }
}

inline unsigned nblk(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_reset(Reduce* red, hipStream_t st) {
    k_reset<<<1, 64, 0, st>>>(red);
    return hipGetLastError();
}

hipError_t launch_set_dt(Reduce* red, double dt, hipStream_t st) {
    k_set_dt<<<1, 64, 0, st>>>(red, dt);
    return hipGetLastError();
}

void batch_blocks(const Grid2* hg, int n, const Tiles& t, int* out) {
    for (int k = 0; k < KB_COUNT; ++k) {
        int* st = out + k * (n + 1);
        st[0] = 0;
        for (int p = 0; p < n; ++p) {
            const Grid2& g = hg[p];
            long long work = 0;
            int per = 256;
            switch (k) {
                case KB_GHOST: work = (long long)(g.ny + g.NX) * 2 * HALO; break;
                case KB_RECON:   // tiles of t.recon x (64 / t.recon) cells, aligned to
                                 // ghosted columns
                    work = (long long)((g.NX - 1 + t.recon - 1) / t.recon) *
                           ((g.NY - 2 + 64 / t.recon - 1) / (64 / t.recon));
                    per = 1;
                    break;
                case KB_RBAR:    // tiles of RB_TX x RB_TY cells, aligned to ghosted columns
                    work = (long long)((g.NX - 2 + RB_TX - 1) / RB_TX) *
                           ((g.NY - 4 + RB_TY - 1) / RB_TY);
                    per = 1;
                    break;
                case KB_GRAD:
                    work = (long long)(g.NX - 6) * (g.NY - 6);
                    per = t.grad == 64 ? 64 : 32;
                    break;
                case KB_RGRAD:   // tiles of 16 x 2 cells of the gradient region
                    work = (long long)((g.NX - 6 + 15) / 16) * ((g.NY - 6 + 1) / 2);
                    per = 1;
                    break;
                case KB_RGRADS:   // tiles of 8 x 4 cells
                    work = (long long)((g.NX - 6 + 7) / 8) * ((g.NY - 6 + 3) / 4);
                    per = 1;
                    break;
                case KB_FLUX0:   // none when the update kernel forms the fluxes
                    work = t.flux ? (long long)(g.nx + 1) * g.ny : 0;
                    per = t.flux ? t.flux : 1;
                    break;
                case KB_FLUX1:
                    work = t.flux ? (long long)g.nx * (g.ny + 1) : 0;
                    per = t.flux ? t.flux : 1;
                    break;
                case KB_FLUXUP:  // tiles of FU_TX x FU_TY cells, aligned to ghosted columns
                    work = (long long)((g.nx + HALO + FU_TX - 1) / FU_TX) *
                           ((g.ny + FU_TY - 1) / FU_TY);
                    per = 1;
                    break;
                case KB_FLUXUPS:   // tiles of FU_TX x FS_TY cells
                    work = (long long)((g.nx + HALO + FU_TX - 1) / FU_TX) *
                           ((g.ny + FS_TY - 1) / FS_TY);
                    per = 1;
                    break;
                default: work = (long long)g.nx * g.ny; break;
            }
            st[p + 1] = st[p] + (int)nblk(work, per);
        }
    }
}

hipError_t launch_check2(const BatchL& b, int si, hipStream_t st) {
    k_check2<<<b.blocks(KB_CELLS), 256, 0, st>>>(b.arg(KB_CELLS), si);
    return hipGetLastError();
}

hipError_t launch_solid2(const Grid2* g, int n, int si, hipStream_t st) {
    if (n > 0) k_solid2<<<nblk(n, 256), 256, 0, st>>>(g, si);
    return hipGetLastError();
}

hipError_t launch_copy_in2(const Grid2& g, const double* U, double* S, hipStream_t st) {
    const long long n = (long long)g.nx * g.ny * 12;
    k_copy_in2<<<nblk(n, 256), 256, 0, st>>>(g, U, S);
    return hipGetLastError();
}

hipError_t launch_copy_out2(const Grid2& g, const double* S, double* U, hipStream_t st) {
    const long long n = (long long)g.nx * g.ny * 12;
    k_copy_out2<<<nblk(n, 256), 256, 0, st>>>(g, S, U);
    return hipGetLastError();
}

// Launch of a kernel that is a timing class of its own: when the class is
// timed, the kernel records the two events itself at the start and end of
// its execution; otherwise a plain launch (the one graphs record).
template <typename F, typename... Args>
void tlaunch(Timer* tm, int k, F kern, unsigned grid, unsigned block, hipStream_t st,
             Args... args) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (tm) tm->ext(k, &e0, &e1);
    if (e0) hipExtLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, st, e0, e1, 0, args...);
    else hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, st, args...);
}

hipError_t launch_ghost2(const BatchL& b, int si, hipStream_t st, Timer* tm, int stage) {
    tlaunch(tm, KC_GHOST, k_ghost2, b.blocks(KB_GHOST), 256, st, b.arg(KB_GHOST), si, stage);
    return hipGetLastError();
}

// The split face-flux kernels of both directions for the launch's tiles.
template <bool FULL>
void launch_flux2(const BatchL& b, hipStream_t st) {
    const Batch a0 = b.arg(KB_FLUX0), a1 = b.arg(KB_FLUX1);
    const unsigned n0 = b.blocks(KB_FLUX0), n1 = b.blocks(KB_FLUX1);
    if (b.tiles.flux == 128) {
        if (b.var_mu) {
            k_flux2<0, 128, true, FULL><<<n0, 384, 0, st>>>(a0);
            k_flux2<1, 128, true, FULL><<<n1, 384, 0, st>>>(a1);
        } else {
            k_flux2<0, 128, false, FULL><<<n0, 384, 0, st>>>(a0);
            k_flux2<1, 128, false, FULL><<<n1, 384, 0, st>>>(a1);
        }
    } else {
        if (b.var_mu) {
            k_flux2<0, 64, true, FULL><<<n0, 192, 0, st>>>(a0);
            k_flux2<1, 64, true, FULL><<<n1, 192, 0, st>>>(a1);
        } else {
            k_flux2<0, 64, false, FULL><<<n0, 192, 0, st>>>(a0);
            k_flux2<1, 64, false, FULL><<<n1, 192, 0, st>>>(a1);
        }
    }
}

// full_grad: the reverse mode also stores the full volume values.
template <int TX>
void launch_recon2(const BatchL& b, int si, int alpha, int gst, const double* U, hipStream_t st,
                   Timer* tm) {
    const unsigned n = b.blocks(KB_RECON);
    const Batch a = b.arg(KB_RECON);
    auto launch = [&](auto f) { tlaunch(tm, KC_RECON, f, n, 256, st, a, si, alpha, gst, U); };
    if (b.full_grad && !b.sums) launch(k_recon2<TX, false, 2, false>);
    else if (b.full_grad) launch(b.var_mu ? k_recon2<TX, true, 1, false> : k_recon2<TX, false, 1, false>);
    else if (gst == GHOSTS_FILLED) launch(b.var_mu ? k_recon2<TX, true, 0, false> : k_recon2<TX, false, 0, false>);
    else launch(b.var_mu ? k_recon2<TX, true, 0, true> : k_recon2<TX, false, 0, true>);
}

template <bool VarMu>
void launch_rgrad2(const BatchL& b, hipStream_t st, Timer* tm) {
    if (b.blocks(KB_RGRAD) <= RG_MAX_BLOCKS)
        tlaunch(tm, KC_GRAD, k_rgrad2<8, 4, VarMu>, b.blocks(KB_RGRADS), 6 * RG_CELLS, st,
                b.arg(KB_RGRADS));
    else
        tlaunch(tm, KC_GRAD, k_rgrad2<16, 2, VarMu>, b.blocks(KB_RGRAD), 6 * RG_CELLS, st,
                b.arg(KB_RGRAD));
}

template <int TX>
void launch_recon2_dr(const BatchL& b, int si, bool alpha, int gst, const double* U,
                      hipStream_t st, Timer* tm) {
    auto launch = [&](auto f) {
        tlaunch(tm, KC_RECON, f, b.blocks(KB_RECON), 256, st, b.arg(KB_RECON), si, (int)alpha, gst,
                U);
    };
    if (gst == GHOSTS_FILLED)
        launch(b.var_mu ? k_recon2_dr<TX, true, false> : k_recon2_dr<TX, false, false>);
    else
        launch(b.var_mu ? k_recon2_dr<TX, true, true> : k_recon2_dr<TX, false, true>);
}

hipError_t launch_residual2(const BatchL& b, int si, int gst, hipStream_t st, Timer* tm, bool alpha,
                            const double* U) {
    const unsigned ng = b.blocks(KB_GRAD);
    if (b.dr) {   // HWENO-DR: gradients and volume fluxes come with the reconstruction
        if (b.tiles.recon == 16) launch_recon2_dr<16>(b, si, alpha, gst, U, st, tm);
        else launch_recon2_dr<32>(b, si, alpha, gst, U, st, tm);
    } else if (b.tiles.recon == 16) {
        launch_recon2<16>(b, si, alpha, gst, U, st, tm);
    } else {
        launch_recon2<32>(b, si, alpha, gst, U, st, tm);
    }
    if (!b.dr && !b.full_grad) {   // HWENO-GR: gradients from the weak moments
        if (b.var_mu) launch_rgrad2<true>(b, st, tm);
        else launch_rgrad2<false>(b, st, tm);
    } else if (!b.dr) {   // the reverse mode reads the weak moments and all six gradients
        tlaunch(tm, KC_RBAR, k_rbar2, b.blocks(KB_RBAR), RB_TX * RB_TY, st, b.arg(KB_RBAR));
        auto launch = [&](auto f, unsigned threads) {
            tlaunch(tm, KC_GRAD, f, ng, threads, st, b.arg(KB_GRAD));
        };
        if (b.tiles.grad == 64) {
            if (!b.sums) launch(k_grad2<64, false, false>, 384);
            else launch(b.var_mu ? k_grad2<64, true, true> : k_grad2<64, false, true>, 384);
        } else {
            if (!b.sums) launch(k_grad2<32, false, false>, 192);
            else launch(b.var_mu ? k_grad2<32, true, true> : k_grad2<32, false, true>, 192);
        }
        if (!b.sums) return hipGetLastError();
    }
    if (b.tiles.flux == 0) return hipGetLastError();   // fluxes formed by the update kernel
    tbeg(tm, KC_FLUX, st);
    if (b.full_grad) launch_flux2<true>(b, st);
    else launch_flux2<false>(b, st);
    tend(tm, st);
    return hipGetLastError();
}

template <bool VarMu, bool FULL>
void launch_fluxup2(const BatchL& b, int stage, int i0, int iin, int iout, double* R, double* Vhat,
                    hipStream_t st, Timer* tm, const double* src, const StepRule& rule) {
    if (VarMu || b.blocks(KB_FLUXUP) <= FS_MAX_BLOCKS)
        tlaunch(tm, KC_FLUXUP, k_fluxup2s<VarMu, FULL>, b.blocks(KB_FLUXUPS), FS_NT, st,
                b.arg(KB_FLUXUPS), stage, i0, iin, iout, R, Vhat, src, rule);
    else
        tlaunch(tm, KC_FLUXUP, k_fluxup2<FULL>, b.blocks(KB_FLUXUP), FU_TX * FU_TY, st,
                b.arg(KB_FLUXUP), stage, i0, iin, iout, R, Vhat, src, rule);
}

hipError_t launch_update2(const BatchL& b, int stage, int i0, int iin, int iout, double* R,
                          double* Vhat, hipStream_t st, Timer* tm, const double* src,
                          const StepRule& rule) {
    if (b.tiles.flux == 0) {
        auto launch = [&](auto f) { f(b, stage, i0, iin, iout, R, Vhat, st, tm, src, rule); };
        if (b.full_grad) launch(b.var_mu ? launch_fluxup2<true, true> : launch_fluxup2<false, true>);
        else launch(b.var_mu ? launch_fluxup2<true, false> : launch_fluxup2<false, false>);
    } else {
        tlaunch(tm, KC_UPDATE, k_update2, b.blocks(KB_CELLS), 256, st, b.arg(KB_CELLS), stage, i0,
                iin, iout, R, Vhat, src, rule);
    }
    return hipGetLastError();
}

hipError_t launch_place2(const Place2& a, hipStream_t st) {
    k_place2<<<1, 256, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_reset2(const BatchL& b, hipStream_t st) {
    k_reset2<<<nblk(b.n, 64), 64, 0, st>>>(b.dg, b.n);
    return hipGetLastError();
}

hipError_t launch_dt2(const BatchL& b, hipStream_t st) {
    k_dt2<<<nblk(b.n, 64), 64, 0, st>>>(b.dg, b.n);
    return hipGetLastError();
}

hipError_t launch_commit2(const BatchL& b, hipStream_t st) {
    k_commit_copy<<<b.blocks(KB_CELLS), 256, 0, st>>>(b.arg(KB_CELLS));
    k_commit_state<<<nblk(b.n, 64), 64, 0, st>>>(b.dg, b.n, 4, 5);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Scratch of the allocation-free residual: a file-scope array in device
// memory, one per device the library runs on.  Host code never passes the
// array's name to a kernel (on the host it only names a stand-in); it takes
// the device address from hipGetSymbolAddress, once per device with that
// device current, and hands that pointer on.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

hipError_t static_scratch(void** out) {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* addr[MAX_DEVICES] = {};
    *out = nullptr;
    int d = 0;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess) return e;
    if (d < 0 || d >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[d]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[d] = p;
    }
    *out = addr[d];
    return hipSuccess;
}

}  // namespace hw
