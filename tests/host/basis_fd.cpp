// CPU unit test of the eigenvector adjoint that the reconstruction adjoint runs
// (hweno_basis2.h): the cotangents of the cell average and of the characteristic
// values against central differences (fourth order) of a scalar formed from the
// forward functions,
//   J(U, x) = sum_k L_k(U) . l_k  +  sum_q y_q . sum_k x_qk R_k(U),
// rows L_k and columns R_k of field_rows at the basis of the average U, l_k and y_q
// random, x_qk the fields' values at a few points q.  Built with g++ against a host
// stand-in of the HIP runtime header.  Prints: <name> <worst relative error> <OK|FAIL>
#include <cstdio>
#include <random>
#include <vector>

#include "hweno_basis2.h"

using namespace hw;
using Vec = std::vector<double>;

static std::mt19937_64 rng(2608);
static double nrm() { return std::normal_distribution<double>(0.0, 1.0)(rng); }
static double uni() { return std::uniform_real_distribution<double>()(rng); }
static int failures = 0;

constexpr int POINTS = 3;
static double l[4][4], y[POINTS][4];   // cotangents of the rows and of the points

static Consts consts(double gamma) {
    Consts K{};
    K.gamma = gamma;
    K.gm1 = gamma - 1.0;
    return K;
}

// v = (rho, m_n, m_t, E), then the points' four field values
static double forward(const Consts& K, const Vec& v) {
    const Basis2 e = basis2(K, v[0], v[1], v[2], v[3]);
    double J = 0.0;
    for (int k = 0; k < 4; ++k) {
        double L[4], R[4];
        field_rows(e, k, L, R);
        for (int c = 0; c < 4; ++c) {
            J += L[c] * l[k][c];
            for (int q = 0; q < POINTS; ++q) J += y[q][c] * v[4 + 4 * q + k] * R[c];
        }
    }
    return J;
}

static void reverse(const Consts& K, const Vec& v, Vec& vb) {
    const Basis2 e = basis2(K, v[0], v[1], v[2], v[3]);
    PointSums2 a;
    for (int q = 0; q < POINTS; ++q) cons2_vjp(e, v.data() + 4 + 4 * q, y[q], a, vb.data() + 4 + 4 * q);
    Basis2Bar g(e, a);
    for (int k = 0; k < 4; ++k) row2_vjp(e, k, l[k], g);
    basis2_vjp(K, e, v[0], v[1], v[2], v[3], a.a5, g, vb.data());
}

static void check(const char* name, double gamma, double mach, double tol) {
    double worst = 0.0;
    for (int t = 0; t < 60; ++t) {
        const Consts K = consts(gamma);
        Vec v(4 + 4 * POINTS);
        const double r = 0.2 + 1.8 * uni(), p = 0.2 + 1.8 * uni(), c = sqrt(gamma * p / r);
        const double un = mach * c * nrm(), ut = mach * c * nrm();
        v[0] = r;
        v[1] = r * un;
        v[2] = r * ut;
        v[3] = p / K.gm1 + 0.5 * r * (un * un + ut * ut);
        for (size_t q = 4; q < v.size(); ++q) v[q] = nrm();
        for (auto& row : l)
            for (double& z : row) z = nrm();
        for (auto& row : y)
            for (double& z : row) z = nrm();
        Vec vb(v.size(), 0.0);
        reverse(K, v, vb);
        for (size_t q = 0; q < v.size(); ++q) {
            const double h = 1e-4 * fmax(1e-2, fabs(v[q]));
            auto at = [&](double s) {
                Vec z = v;
                z[q] += s * h;
                return forward(K, z);
            };
            const double fd = (8.0 * (at(1) - at(-1)) - (at(2) - at(-2))) / (12.0 * h);
            const double e = fabs(fd - vb[q]) / fmax(1.0, fmax(fabs(fd), fabs(vb[q])));
            worst = std::isfinite(vb[q]) ? fmax(worst, e) : INFINITY;
        }
    }
    if (!(worst <= tol)) ++failures;
    printf("%s %.3e %s\n", name, worst, worst <= tol ? "OK" : "FAIL");
}

int main() {
    // the bound of the other adjoint checks against differences of this order
    check("basis2_vjp_subsonic", 1.4, 0.5, 1e-7);
    check("basis2_vjp_at_rest", 1.4, 0.0, 1e-7);
    check("basis2_vjp_monatomic", 5.0 / 3.0, 1.0, 1e-7);
    printf("failures %d\n", failures);
    return failures ? 1 : 0;
}
