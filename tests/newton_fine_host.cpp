// Host build of the dual Newton polish where its right-hand side or torque
// arms are large: kappa is a parameter, and the forces come from where the
// solve leaves them (the store's centre, or u).
#include "../paper_2412_16490_amd/csrc/bodex_newton.h"

#include <algorithm>

using namespace bodex;

// One grasp with m <= 8 contacts (p, n [m][3], mu [m]) and s right-hand sides
// bt [s][6], cold: forces f [s][3 m], info [s][2] (solved, Newton steps).
template <bool CONE>
static void solve(int m, const double* p, const double* n, const double* mu, const double* bt, int s, double kappa,
                  double eps, double fmax, int max_steps, double* f, int* info) {
    constexpr int MM = 8;
    for (int j = 0; j < s; ++j, bt += 6, f += 3 * m, info += 2) {
        double geo[MM * 12] = {}, centre[3 * MM] = {}, qp[NewtonStore<MM>::kQp], u[6];
        NewtonStore<MM> st;
        NewtonFriction Fr[MM];
        st.cp = centre;
        st.q = qp;
        st.cs = st.qs = 1;
        for (int i = 0; i < MM; ++i) {
            st.geo[i] = geo + 12 * i;
            if (i < m) newton_contact(p + 3 * i, n + 3 * i, kappa, geo + 12 * i);
            Fr[i] = newton_friction((i < m ? mu[i] : 0.5) * (CONE ? 1.0 : kC8));
        }
        for (int r = 0; r < 6; ++r) st.bt(r) = bt[r];
        const NewtonOut o = newton_solve<1, MM, CONE>(st, Fr, m, fmax, eps, max_steps, u);
        if (!o.forces)
            for (int i = 0; i < m; ++i) {
                double y[3];
                newton_gt(st.contact(i), u, y);
                const NewtonFold Y = newton_fold<CONE>(y[0] / eps, y[1] / eps, y[2] / eps);
                newton_keep(st, i, Y, newton_project<CONE>(Y, Fr[i], fmax));
            }
        for (int i = 0; i < m; ++i)
            for (int t = 0; t < 3; ++t) f[3 * i + t] = st.centre(i, t);
        info[0] = o.ok;
        info[1] = o.steps;
    }
}

extern "C" void host_newton_fine(int cone, int m, const double* p, const double* n, const double* mu, const double* bt,
                                 int s, double kappa, double eps, double fmax, int max_steps, double* f, int* info) {
    (cone ? solve<true> : solve<false>)(m, p, n, mu, bt, s, kappa, eps, fmax, max_steps, f, info);
}

// The minimiser in 128 bits: Newton's method on F(u) = G P_C(G^T u / eps) + u - bt
// from u = bt - G f0, with its own projection; returns |F| at the end (the dual
// is strictly convex, so F = 0 is the minimiser's certificate).
using Quad = __float128;
static Quad quad_sqrt(Quad x) {
    if (!(x > 0)) return 0;
    Quad r = std::sqrt(double(x));
    for (int i = 0; i < 4; ++i) r = (r + x / r) / 2;
    return r;
}

extern "C" double host_newton_exact(int cone, int m, const double* p, const double* n, const double* mu,
                                    const double* bt, double kappa, double eps, double fmax, const double* f0,
                                    double* f) {
    Quad G[6][24], u[6], x[24];
    const Quad r2 = quad_sqrt(2), c8 = quad_sqrt((2 + r2) / 4), s8 = quad_sqrt((2 - r2) / 4);
    for (int i = 0; i < m; ++i) {
        const Quad len = quad_sqrt(Quad(n[3 * i]) * n[3 * i] + Quad(n[3 * i + 1]) * n[3 * i + 1] +
                                   Quad(n[3 * i + 2]) * n[3 * i + 2]);
        const Quad a = n[3 * i] / len, b = n[3 * i + 1] / len, c = n[3 * i + 2] / len, s = c < 0 ? -1 : 1, h = -1 / (s + c);
        const Quad R[3][3] = {{a, b, c}, {1 + s * a * a * h, s * a * b * h, -s * a}, {a * b * h, s + b * b * h, -b}};
        for (int t = 0; t < 3; ++t)
            for (int q = 0; q < 3; ++q) {
                G[q][3 * i + t] = R[t][q];
                G[3 + q][3 * i + t] = Quad(kappa) * (Quad(p[3 * i + (q + 1) % 3]) * R[t][(q + 2) % 3] -
                                                     Quad(p[3 * i + (q + 2) % 3]) * R[t][(q + 1) % 3]);
            }
    }
    for (int r = 0; r < 6; ++r) {
        u[r] = bt[r];
        for (int c = 0; c < 3 * m; ++c) u[r] -= G[r][c] * f0[c];
    }
    double res = INFINITY;
    for (int it = 0; it < 60; ++it) {
        Quad F[6], M[6][6] = {};
        for (int r = 0; r < 6; ++r) {
            F[r] = u[r] - bt[r];
            M[r][r] = eps;
        }
        for (int i = 0; i < m; ++i) {
            Quad y[3] = {0, 0, 0}, V[3][6];
            for (int t = 0; t < 3; ++t)
                for (int r = 0; r < 6; ++r) y[t] += G[r][3 * i + t] * u[r] / eps;
            // (e_p, e_q): the nearest facet's normal (the radius) and across
            Quad a = 1, b = 0, k = mu[i], kt = 0;
            if (cone) {
                const Quad r = quad_sqrt(y[1] * y[1] + y[2] * y[2]);
                if (r > 0) a = y[1] / r, b = y[2] / r;
            } else {
                const bool up = (y[1] < 0 ? -y[1] : y[1]) < (y[2] < 0 ? -y[2] : y[2]);
                a = (up ? s8 : c8) * (y[1] < 0 ? -1 : 1);
                b = (up ? c8 : s8) * (y[2] < 0 ? -1 : 1);
                k *= c8;
                kt = k * s8 / c8;
            }
            const Quad P = a * y[1] + b * y[2], Q = a * y[2] - b * y[1], sq = Q < 0 ? -1 : 1;
            const Quad facet = (y[0] + k * P) / (1 + k * k), edge = (y[0] + k * P + kt * sq * Q) / (1 + k * k + kt * kt);
            const bool on_edge = !cone && edge > facet;
            const Quad far = std::max(facet, on_edge ? edge : facet), top = std::max(y[0], far);
            const Quad f1 = std::min(std::max(top, Quad(0)), Quad(fmax)), fp = std::min(P, k * f1);
            const Quad fq = cone ? Quad(0) : sq * std::min(sq * Q, kt * f1);
            x[3 * i] = f1, x[3 * i + 1] = a * fp - b * fq, x[3 * i + 2] = b * fp + a * fq;
            // its derivative's three directions, each scaled by a root of its weight
            const bool inside = y[0] >= far, moves = top > 0 && top < fmax;
            const Quad gp = inside ? Quad(0) : k, gq = inside || !on_edge ? Quad(0) : sq * kt;
            const Quad w1 = moves ? 1 / (1 + gp * gp + gq * gq) : Quad(0), w2 = P < k * f1 ? 1 : 0;
            const Quad w3 = cone ? (P < k * f1 ? Quad(1) : (P > 0 ? fp / P : Quad(0))) : Quad(sq * Q < kt * f1 ? 1 : 0);
            const Quad w[3] = {w1, w2, w3};
            for (int r = 0; r < 6; ++r) {
                const Quad vp = G[r][3 * i + 1] * a + G[r][3 * i + 2] * b, vq = G[r][3 * i + 2] * a - G[r][3 * i + 1] * b;
                V[0][r] = G[r][3 * i] + gp * vp + gq * vq, V[1][r] = vp, V[2][r] = vq;
                for (int t = 0; t < 3; ++t) F[r] += G[r][3 * i + t] * x[3 * i + t];
            }
            for (int t = 0; t < 3; ++t)
                for (int r = 0; r < 6; ++r)
                    for (int c = 0; c < 6; ++c) M[r][c] += w[t] * V[t][r] * V[t][c];
        }
        res = 0.0;
        for (int r = 0; r < 6; ++r) res = std::max(res, std::fabs(double(F[r])));
        if (res < 1e-24) break;
        for (int r = 0; r < 6; ++r) F[r] *= -Quad(eps);
        for (int j = 0; j < 6; ++j)
            for (int i = j + 1; i < 6; ++i) {
                const Quad l = M[i][j] / M[j][j];
                for (int c = j; c < 6; ++c) M[i][c] -= l * M[j][c];
                F[i] -= l * F[j];
            }
        for (int i = 5; i >= 0; --i) {
            for (int c = i + 1; c < 6; ++c) F[i] -= M[i][c] * F[c];
            F[i] /= M[i][i];
            u[i] += F[i];
        }
    }
    for (int c = 0; c < 3 * m; ++c) f[c] = double(x[c]);
    return res;
}
