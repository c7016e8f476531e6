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
