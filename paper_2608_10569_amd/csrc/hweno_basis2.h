// Characteristic bases of the 2D reconstruction in (normal, tangential)
// coordinates, and the projection of an LDS stencil tile onto a field; shared by
// the forward reconstruction and its adjoint.
#pragma once

#include "hweno_device.h"

namespace hw {

// Characteristic basis at a cell average in (rho, m_n, m_t, E) ordering.
struct Basis2 {
    double un, ut, q2, c, ic, H, b1, b2;
};
__device__ __forceinline__ Basis2 basis2(const Consts& K, double r, double mn, double mt,
                                         double E) {
#pragma clang fp contract(on)
    Basis2 e;
    const double ir = rcp(r);
    e.un = mn * ir;
    e.ut = mt * ir;
    e.q2 = e.un * e.un + e.ut * e.ut;
    const double p = K.gm1 * (E - 0.5 * r * e.q2);
    e.c = sqrt(K.gamma * p * ir);
    e.ic = rcp(e.c);
    e.H = (E + p) * ir;
    e.b1 = K.gm1 * e.ic * e.ic;
    e.b2 = 0.5 * e.b1 * e.q2;
    return e;
}
// Row k of L and column k of R = L^-1 (k uniform).
__device__ __forceinline__ void field_rows(const Basis2& e, int k, double* L, double* R) {
#pragma clang fp contract(on)
    if (k == 1) {
        L[0] = 1.0 - e.b2; L[1] = e.b1 * e.un; L[2] = e.b1 * e.ut; L[3] = -e.b1;
        R[0] = 1.0; R[1] = e.un; R[2] = e.ut; R[3] = 0.5 * e.q2;
    } else if (k == 2) {
        L[0] = -e.ut; L[1] = 0.0; L[2] = 1.0; L[3] = 0.0;
        R[0] = 0.0; R[1] = 0.0; R[2] = 1.0; R[3] = e.ut;
    } else {
        const double sc = k == 0 ? -e.c : e.c, si = k == 0 ? -e.ic : e.ic;
        L[0] = 0.5 * (e.b2 - e.un * si);
        L[1] = 0.5 * (si - e.b1 * e.un);
        L[2] = -0.5 * e.b1 * e.ut;
        L[3] = 0.5 * e.b1;
        R[0] = 1.0; R[1] = e.un + sc; R[2] = e.ut; R[3] = e.H + e.un * sc;
    }
}

// Adjoint of the basis.  The conserved components at a point, u = sum_k x[k] R_k,
// depend on it through these sums over the points of (cotangents y of u) times
// (field values x).
struct PointSums2 {
    double a1 = 0.0, a2 = 0.0, a3 = 0.0, a4 = 0.0, a5 = 0.0, a6 = 0.0;
};
// One point: its share of the sums, and the cotangents z[k] = y . R_k of its fields.
__device__ __forceinline__ void cons2_vjp(const Basis2& e, const double* x, const double* y,
                                          PointSums2& a, double* z) {
    const double sm = x[0] + x[3], df = x[3] - x[0], al = sm + x[1];
    a.a1 += y[1] * al;
    a.a2 += y[2] * al + y[3] * x[2];
    a.a3 += y[1] * df;
    a.a4 += y[3] * df;
    a.a5 += y[3] * sm;
    a.a6 += y[3] * x[1];
    const double s0 = y[0] + e.un * y[1] + e.ut * y[2];
    const double sa = s0 + e.H * y[3], sd = e.c * (y[1] + e.un * y[3]);
    z[0] = sa - sd;
    z[1] = s0 + 0.5 * e.q2 * y[3];
    z[2] = y[2] + e.ut * y[3];
    z[3] = sa + sd;
}
// Cotangents of the members of Basis2 (H's is the sum a5).
struct Basis2Bar {
    double un, ut, c, q2, b1 = 0.0, b2 = 0.0, ic = 0.0;
    __device__ __forceinline__ Basis2Bar(const Basis2& e, const PointSums2& a)
        : un(a.a1 + e.c * a.a4), ut(a.a2), c(a.a3 + e.un * a.a4), q2(0.5 * a.a6) {}
};
// Adds the share of row k of L (k uniform) with cotangents Lb.
__device__ __forceinline__ void row2_vjp(const Basis2& e, int k, const double* Lb, Basis2Bar& g) {
    if (k == 1) {
        g.b2 -= Lb[0];
        g.b1 += e.un * Lb[1] + e.ut * Lb[2] - Lb[3];
        g.un += e.b1 * Lb[1];
        g.ut += e.b1 * Lb[2];
    } else if (k == 2) {
        g.ut -= Lb[0];
    } else {
        const double sg = k == 0 ? -1.0 : 1.0, si = sg * e.ic;
        g.b2 += 0.5 * Lb[0];
        g.un -= 0.5 * (si * Lb[0] + e.b1 * Lb[1]);
        g.ic += 0.5 * sg * (Lb[1] - e.un * Lb[0]);
        g.b1 += 0.5 * (Lb[3] - e.un * Lb[1] - e.ut * Lb[2]);
        g.ut -= 0.5 * e.b1 * Lb[2];
    }
}
// Back through basis2 to the cell average (r, mn, mt, E): adds to ub.
__device__ __forceinline__ void basis2_vjp(const Consts& K, const Basis2& e, double r, double mn,
                                           double mt, double E, double a5, Basis2Bar g,
                                           double* ub) {
    const double ir = rcp(r), p = K.gm1 * (E - 0.5 * r * e.q2);
    g.b1 += 0.5 * e.q2 * g.b2;
    g.q2 += 0.5 * e.b1 * g.b2;
    g.ic += 2.0 * K.gm1 * e.ic * g.b1;
    g.c -= e.ic * e.ic * g.ic;
    const double c2b = 0.5 * e.ic * g.c;
    const double pb = ir * a5 + K.gamma * ir * c2b;
    double irb = (E + p) * a5 + K.gamma * p * c2b;
    g.q2 -= 0.5 * K.gm1 * r * pb;
    g.un += 2.0 * e.un * g.q2;
    g.ut += 2.0 * e.ut * g.q2;
    irb += mn * g.un + mt * g.ut;
    ub[0] -= 0.5 * K.gm1 * e.q2 * pb + ir * ir * irb;
    ub[1] += ir * g.un;
    ub[2] += ir * g.ut;
    ub[3] += ir * a5 + K.gm1 * pb;
}

// A wavefront's half: its points and the slots of the exchange it owns (the face
// points and the moment, or the volume points).
template <int h>
struct Part {
    static constexpr int value = h, points = h ? 9 : 6, slots = h ? 9 : 7;
};

// The 17 stencil data of the field with left eigenvector L: sh holds 12
// fields of PL doubles, rows of TW; basis b's normal direction is x (b = 0)
// or y (b = 1).
template <int b, int TW, int PL>
__device__ __forceinline__ void project2(const double* sh, const double* L, double* a) {
#pragma clang fp contract(on)
    constexpr int sn = b ? TW : 1, st = b ? 1 : TW;   // strides: normal, tangential
    constexpr int cm[4] = {0, b ? 2 : 1, b ? 1 : 2, 3};
    constexpr int mn = b ? 8 : 4, mt = b ? 4 : 8;     // moment fields: normal, tangential
#pragma unroll
    for (int s = 0; s < 9; ++s) {
        const double* q = sh + (s % 3 - 1) * sn + (s / 3 - 1) * st;
        double acc = L[0] * q[cm[0] * PL];
#pragma unroll
        for (int c = 1; c < 4; ++c) acc += L[c] * q[cm[c] * PL];
        a[s] = acc;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int s = 2 * e + 1;
        const double* q = sh + (s % 3 - 1) * sn + (s / 3 - 1) * st;
        double an = L[0] * q[(mn + cm[0]) * PL], at_ = L[0] * q[(mt + cm[0]) * PL];
#pragma unroll
        for (int c = 1; c < 4; ++c) {
            an += L[c] * q[(mn + cm[c]) * PL];
            at_ += L[c] * q[(mt + cm[c]) * PL];
        }
        a[9 + e] = an;
        a[13 + e] = at_;
    }
}

}  // namespace hw
