// Generated by gen_tables.py from exact rational derivations of the
// unified-stencil HWENO candidate p0 (Appendix A of the paper).  Do not edit.
#pragma once

namespace hweno_gen {

// 1D quartic p0, eq. (A.1).  a = {ubar_{i-1}, ubar_i, ubar_{i+1}, vbar_{i-1},
// vbar_{i+1}} -> c[k], coefficient of xi^k.
__device__ __forceinline__ void p0_1d(const double* __restrict__ a, double* __restrict__ c) {
    const double um = a[0], uc = a[1], up = a[2], vm = a[3], vp = a[4];
    c[0] = 1.2239583333333333 * (uc)
        + 0.421875 * (-vm + vp)
        + 0.11197916666666667 * (-um - up);
    c[1] = 3.9473684210526314 * (-vm - vp)
        + 0.8289473684210527 * (-um + up);
    c[2] = 5.625 * (vm - vp)
        + 2.875 * (-uc)
        + 1.4375 * (um + up);
    c[3] = 3.1578947368421053 * (vm + vp)
        + 0.2631578947368421 * (um - up);
    c[4] = 3.75 * (-vm + vp)
        + 1.25 * (uc)
        + 0.625 * (-um - up);
}

// Sobolev smoothness indicator of a 1D quartic with coefficients c.
__device__ __forceinline__ double sobolev_1d(const double* __restrict__ c) {
    double b = 0.0;
    b = fma(1.0, c[1] * c[1], b);
    b = fma(0.5, c[1] * c[3], b);
    b = fma(4.333333333333333, c[2] * c[2], b);
    b = fma(4.2, c[2] * c[4], b);
    b = fma(39.1125, c[3] * c[3], b);
    b = fma(625.8357142857143, c[4] * c[4], b);
    return b;
}

// 2D quartic p0, eq. (A.4), constrained least squares.  a[0..8] = averages of
// cells 1..9 (row-major from (i-1,j-1)), a[9..12] = xi-moments of cells
// 2,4,6,8, a[13..16] = eta-moments of cells 2,4,6,8 -> c[15] in monomial order.
__device__ __forceinline__ void p0_2d(const double* __restrict__ a, double* __restrict__ c) {
#pragma clang fp contract(on)
    const double a1 = a[0];
    const double a2 = a[1];
    const double a3 = a[2];
    const double a4 = a[3];
    const double a5 = a[4];
    const double a6 = a[5];
    const double a7 = a[6];
    const double a8 = a[7];
    const double a9 = a[8];
    const double x2 = a[9];
    const double x4 = a[10];
    const double x6 = a[11];
    const double x8 = a[12];
    const double y2 = a[13];
    const double y4 = a[14];
    const double y6 = a[15];
    const double y8 = a[16];
    c[0] = 1.4548611111111112 * (a5)
        + 0.421875 * (-x4 + x6 - y2 + y8)
        + 0.1154513888888889 * (-a2 - a4 - a6 - a8)
        + 0.001736111111111111 * (a1 + a3 + a7 + a9);
    c[1] = 3.9473684210526314 * (-x4 - x6)
        + 0.8706140350877193 * (-a4 + a6)
        + 0.020833333333333332 * (a1 - a3 + a7 - a9);
    c[2] = 3.9473684210526314 * (-y2 - y8)
        + 0.8706140350877193 * (-a2 + a8)
        + 0.020833333333333332 * (a1 + a3 - a7 - a9);
    c[3] = 5.625 * (x4 - x6)
        + 2.9583333333333335 * (-a5)
        + 1.4791666666666667 * (a4 + a6)
        + 0.041666666666666664 * (a2 + a8)
        + 0.020833333333333332 * (-a1 - a3 - a7 - a9);
    c[4] = 6.818181818181818 * (-x2 + x8 - y4 + y6)
        + 0.3181818181818182 * (-a1 + a3 + a7 - a9);
    c[5] = 5.625 * (y2 - y8)
        + 2.9583333333333335 * (-a5)
        + 1.4791666666666667 * (a2 + a8)
        + 0.041666666666666664 * (a4 + a6)
        + 0.020833333333333332 * (-a1 - a3 - a7 - a9);
    c[6] = 3.1578947368421053 * (x4 + x6)
        + 0.2631578947368421 * (a4 - a6);
    c[7] = 0.5 * (a2 - a8)
        + 0.25 * (-a1 - a3 + a7 + a9);
    c[8] = 0.5 * (a4 - a6)
        + 0.25 * (-a1 + a3 - a7 + a9);
    c[9] = 3.1578947368421053 * (y2 + y8)
        + 0.2631578947368421 * (a2 - a8);
    c[10] = 3.75 * (-x4 + x6)
        + 1.25 * (a5)
        + 0.625 * (-a4 - a6);
    c[11] = 5.454545454545454 * (x2 - x8)
        + 0.22727272727272727 * (a1 - a3 - a7 + a9);
    c[12] = 1.0 * (a5)
        + 0.5 * (-a2 - a4 - a6 - a8)
        + 0.25 * (a1 + a3 + a7 + a9);
    c[13] = 5.454545454545454 * (y4 - y6)
        + 0.22727272727272727 * (a1 - a3 - a7 + a9);
    c[14] = 3.75 * (-y2 + y8)
        + 1.25 * (a5)
        + 0.625 * (-a2 - a8);
}

// Sobolev smoothness indicator of a 2D quartic with coefficients c.
__device__ __forceinline__ double sobolev_2d(const double* __restrict__ c) {
    double b = 0.0;
    b = fma(1.0, c[1] * c[1], b);
    b = fma(0.5, c[1] * c[6], b);
    b = fma(0.16666666666666666, c[1] * c[8], b);
    b = fma(1.0, c[2] * c[2], b);
    b = fma(0.16666666666666666, c[2] * c[7], b);
    b = fma(0.5, c[2] * c[9], b);
    b = fma(4.333333333333333, c[3] * c[3], b);
    b = fma(4.2, c[3] * c[10], b);
    b = fma(0.7222222222222222, c[3] * c[12], b);
    b = fma(1.1666666666666667, c[4] * c[4], b);
    b = fma(0.5666666666666667, c[4] * c[11], b);
    b = fma(0.5666666666666667, c[4] * c[13], b);
    b = fma(4.333333333333333, c[5] * c[5], b);
    b = fma(0.7222222222222222, c[5] * c[12], b);
    b = fma(4.2, c[5] * c[14], b);
    b = fma(39.1125, c[6] * c[6], b);
    b = fma(0.041666666666666664, c[6] * c[8], b);
    b = fma(4.706944444444445, c[7] * c[7], b);
    b = fma(0.041666666666666664, c[7] * c[9], b);
    b = fma(4.706944444444445, c[8] * c[8], b);
    b = fma(39.1125, c[9] * c[9], b);
    b = fma(625.8357142857143, c[10] * c[10], b);
    b = fma(0.35, c[10] * c[12], b);
    b = fma(42.37410714285714, c[11] * c[11], b);
    b = fma(0.1375, c[11] * c[13], b);
    b = fma(18.886111111111113, c[12] * c[12], b);
    b = fma(0.35, c[12] * c[14], b);
    b = fma(42.37410714285714, c[13] * c[13], b);
    b = fma(625.8357142857143, c[14] * c[14], b);
    return b;
}

}  // namespace hweno_gen
