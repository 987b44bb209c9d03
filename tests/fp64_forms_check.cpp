// Accuracy of the FP64 forms of the force, the velocity and the collisions
// (csrc/lbm_kernels.hpp) on the CPU.  forms.hpp, cut from that header, is
// compiled here for double twice: in the forms with fewer operations and in the
// forms the reduced-precision modes use.  Both step the same droplets, and the
// populations are compared with the equations evaluated in 80 bits:
// prints the rms error of the first and of the second, then how far each is
// from the equations evaluated as written in 64 bits.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>
#include <type_traits>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline
using std::fma;
constexpr int kQ = 9;
template <class R> constexpr bool kNoRef = true;
template <class R> R recip(R v) { return R(1) / v; }

namespace fewer {
template <class R> constexpr bool kFewerOps = true;
#include "forms.hpp"
}
namespace plain {
template <class R> constexpr bool kFewerOps = false;
#include "forms.hpp"
}

template <class X>
static X weight(int q) { return q == 0 ? X(4) / 9 : (q < 5 ? X(1) / 9 : X(1) / 36); }
static const int CX[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1}, CY[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
static const int M[9][9] = {{1, 1, 1, 1, 1, 1, 1, 1, 1},      {-4, -1, -1, -1, -1, 2, 2, 2, 2},
                            {4, -2, -2, -2, -2, 1, 1, 1, 1},  {0, 1, 0, -1, 0, 1, -1, -1, 1},
                            {0, -2, 0, 2, 0, 1, -1, -1, 1},   {0, 0, 1, 0, -1, 1, 1, -1, -1},
                            {0, 0, -2, 0, 2, 1, 1, -1, -1},   {0, 1, -1, 1, -1, 0, 0, 0, 0},
                            {0, 0, 0, 0, 0, 1, -1, 1, -1}};
static const int NORM[9] = {9, 36, 36, 6, 12, 6, 12, 4, 4};

// Carnahan-Starling EOS with all its constants 1, G = -1, eps = 1.73.
struct Lattice {
    int nx, ny;
    double tau, sigma, T;
    bool mrt;
    double te, tz, tq;
};
const double kA = 1, kB = 1, kEps = 1.73;

static int at(const Lattice &L, int x, int y)
{
    return (y + L.ny) % L.ny * L.nx + (x + L.nx) % L.nx;
}

#define STEP(NS)                                                                              \
    static void step_##NS(const Lattice &L, std::vector<double> &f)                           \
    {                                                                                         \
        NS::Coeffs c{};                                                                       \
        c.omega = 1 / L.tau, c.guo = 1 - 1 / (2 * L.tau), c.eos_b = kB, c.kcT = L.T;          \
        c.ka = kA, c.invG = -1, c.cSC = 6;                                                    \
        c.cA = -9 * (1.5 * kEps - L.sigma + 1), c.cB = -9 * (L.sigma - 1);                    \
        c.s_e = 1 / L.te, c.s_z = 1 / L.tz, c.s_q = 1 / L.tq;                                 \
        const NS::Phys<double> P(c);                                                          \
        const int n = L.nx * L.ny;                                                            \
        std::vector<double> rho(n), psi(n), out(9 * (size_t)n);                               \
        for (int i = 0; i < n; ++i) {                                                         \
            const double *d = &f[9 * (size_t)i];                                              \
            const double r =                                                                  \
                (((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7]))) + d[8];   \
            const double br = P.eos_b * r, om = 1 - br;                                       \
            const double num = fma(br, fma(br, om, 1.0), 1.0);                                \
            rho[i] = r;                                                                       \
            psi[i] = std::sqrt(                                                               \
                r * fma(P.g_kcT, num / (om * om * om), -fma(P.g_ka, r, P.g_third)));          \
        }                                                                                     \
        for (int y = 0; y < L.ny; ++y)                                                        \
            for (int x = 0; x < L.nx; ++x) {                                                  \
                const int i = y * L.nx + x;                                                   \
                double s[9], d[9], Fx, Fy, ux, uy, Jx, Jy;                                    \
                for (int q = 0; q < 9; ++q) {                                                 \
                    s[q] = psi[at(L, x + CX[q], y + CY[q])];                                  \
                    d[q] = f[9 * (size_t)i + q];                                              \
                }                                                                             \
                NS::force<double>(s, P, Fx, Fy);                                              \
                NS::velocity<double>(d, rho[i], Fx, Fy, ux, uy, Jx, Jy);                      \
                if (L.mrt)                                                                    \
                    NS::collide_mrt<double>(d, rho[i], ux, uy, Jx, Jy, Fx, Fy, P);            \
                else                                                                          \
                    NS::collide<double>(d, 0.0, rho[i], ux, uy, Jx, Jy, Fx, Fy, P);           \
                for (int q = 0; q < 9; ++q)                                                   \
                    out[9 * (size_t)at(L, x + CX[q], y + CY[q]) + q] = d[q];                  \
            }                                                                                 \
        f.swap(out);                                                                          \
    }
STEP(fewer)
STEP(plain)

// The equations as they are written, in the type X.
template <class X>
static void step_literal(const Lattice &L, std::vector<X> &f)
{
    const int n = L.nx * L.ny;
    std::vector<X> rho(n), psi(n), out(9 * (size_t)n);
    const X om = 1 / (X)L.tau, guo = 1 - om / 2;
    const X lam[9] = {1, 1 / (X)L.te, 1 / (X)L.tz, 1, 1 / (X)L.tq, 1, 1 / (X)L.tq, om, om};
    for (int i = 0; i < n; ++i) {
        X r = 0;
        for (int q = 0; q < 9; ++q) r += f[9 * (size_t)i + q];
        const X br = kB * r;
        const X p = L.T * r * (1 + br + br * br - br * br * br) / ((1 - br) * (1 - br) * (1 - br)) -
                    kA * r * r;
        rho[i] = r;
        psi[i] = std::sqrt(-(p - r / 3));
    }
    for (int y = 0; y < L.ny; ++y)
        for (int x = 0; x < L.nx; ++x) {
            const int i = y * L.nx + x;
            X m1x = 0, m1y = 0, xx = 0, yy = 0, xy = 0, jx = 0, jy = 0;
            for (int q = 0; q < 9; ++q) {
                const X s = weight<X>(q) * psi[at(L, x + CX[q], y + CY[q])];
                m1x += CX[q] * s, m1y += CY[q] * s, xy += CX[q] * CY[q] * s;
                xx += (CX[q] * CX[q] - X(1) / 3) * s, yy += (CY[q] * CY[q] - X(1) / 3) * s;
                jx += CX[q] * f[9 * (size_t)i + q], jy += CY[q] * f[9 * (size_t)i + q];
            }
            const X cA = -9 * (X(1.5) * (X)kEps - (X)L.sigma + 1), cB = -9 * ((X)L.sigma - 1);
            const X Fx = 6 * psi[i] * m1x + cA * (m1x * xx + m1y * xy) + cB * m1x * (xx + yy);
            const X Fy = 6 * psi[i] * m1y + cA * (m1x * xy + m1y * yy) + cB * m1y * (xx + yy);
            const X ux = (jx + Fx / 2) / rho[i], uy = (jy + Fy / 2) / rho[i];
            X df[9], S[9], g[9];
            for (int q = 0; q < 9; ++q) {
                const X cu = CX[q] * ux + CY[q] * uy, cF = CX[q] * Fx + CY[q] * Fy;
                const X feq =
                    weight<X>(q) * rho[i] * (1 + 3 * cu + X(4.5) * cu * cu - X(1.5) * (ux * ux + uy * uy));
                g[q] = f[9 * (size_t)i + q];
                df[q] = g[q] - feq;
                S[q] = weight<X>(q) * (3 * cF + 9 * cF * cu - 3 * (ux * Fx + uy * Fy));
            }
            if (!L.mrt)
                for (int q = 0; q < 9; ++q) g[q] += guo * S[q] - om * df[q];
            else
                for (int k = 0; k < 9; ++k) {
                    X a = 0, b = 0;
                    for (int q = 0; q < 9; ++q) a += M[k][q] * df[q], b += M[k][q] * S[q];
                    for (int q = 0; q < 9; ++q)
                        g[q] += M[k][q] * ((1 - lam[k] / 2) * b - lam[k] * a) / NORM[k];
                }
            for (int q = 0; q < 9; ++q) out[9 * (size_t)at(L, x + CX[q], y + CY[q]) + q] = g[q];
        }
    f.swap(out);
}

// usage: nx ny tau sigma T mrt tau_e tau_zeta tau_q rho_gas rho_liquid steps seeds
int main(int argc, char **argv)
{
    if (argc != 14) return 2;
    auto v = [&](int k) { return std::atof(argv[k]); };
    const Lattice L{(int)v(1), (int)v(2), v(3), v(4), v(5), v(6) != 0, v(7), v(8), v(9)};
    const double rg = v(10), rl = v(11);
    const int n = L.nx * L.ny;
    double e_fewer = 0, e_plain = 0, d_fewer = 0, d_plain = 0;
    for (int seed = 0; seed < (int)v(13); ++seed) {
        std::mt19937_64 gen(1000 + seed);
        std::uniform_real_distribution<double> noise(-1e-3, 1e-3);
        std::vector<double> a(9 * (size_t)n);
        for (int y = 0; y < L.ny; ++y)
            for (int x = 0; x < L.nx; ++x) {
                const double r = std::hypot(x - (L.nx - 1) / 2.0, y - (L.ny - 1) / 2.0);
                const double rho = 0.5 * (rl + rg) -
                                   0.5 * (rl - rg) * std::tanh(r - 0.25 * std::min(L.nx, L.ny)) +
                                   noise(gen);
                for (int q = 0; q < 9; ++q)
                    a[9 * (size_t)(y * L.nx + x) + q] = weight<double>(q) * rho;
            }
        std::vector<double> b = a, w = a;
        std::vector<long double> e(a.begin(), a.end());
        for (int s = 0; s < (int)v(12); ++s) {
            step_fewer(L, a);
            step_plain(L, b);
            step_literal(L, w);
            step_literal(L, e);
        }
        auto add = [](double &sum, long double d) { sum += (double)(d * d); };
        for (size_t k = 0; k < e.size(); ++k) {
            add(e_fewer, a[k] - e[k]), add(e_plain, b[k] - e[k]);
            add(d_fewer, a[k] - w[k]), add(d_plain, b[k] - w[k]);
        }
    }
    const double count = 9.0 * n * v(13);
    printf("%.3e %.3e %.3e %.3e\n", std::sqrt(e_fewer / count), std::sqrt(e_plain / count),
           std::sqrt(d_fewer / count), std::sqrt(d_plain / count));
    return 0;
}
