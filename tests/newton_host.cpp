// Host build of the dual Newton polish (the header the GPU kernels use, one
// thread per QP), for CPU tests.
#include "../paper_2412_16490_amd/csrc/bodex_newton.h"

using namespace bodex;

namespace {

template <bool CONE>
void solve_one(int m, const double* p, const double* n, const double* mu, const double* t, const double* x0,
               double eps, double fmax, int max_steps, double* f, int* info) {
    constexpr int MM = 8;
    double geo[MM * 12] = {}, centre[3 * MM] = {}, qp[NewtonStore<MM>::kQp], u[6];
    NewtonStore<MM> st;
    NewtonFriction Fr[MM];
    st.cp = centre;
    st.cs = 1;
    st.q = qp;
    st.qs = 1;
    for (int i = 0; i < MM; ++i) {
        st.geo[i] = geo + 12 * i;
        if (i < m) newton_contact(p + 3 * i, n + 3 * i, 20.0, geo + 12 * i);
        Fr[i] = newton_friction((i < m ? mu[i] : 0.5) * (CONE ? 1.0 : kC8));
        for (int k = 0; k < 3; ++k) st.centre(i, k) = i < m ? x0[3 * i + k] : 0.0;
    }
    for (int r = 0; r < 6; ++r) st.bt(r) = t[r];
    const NewtonOut o = newton_solve<1, MM, CONE>(st, Fr, m, fmax, eps, max_steps, u);
    for (int i = 0; i < m; ++i) {
        double y[3];
        newton_gt(st.contact(i), u, y);
        const NewtonFold Y = newton_fold<CONE>(y[0] / eps, y[1] / eps, y[2] / eps);
        const NewtonProj P = newton_project<CONE>(Y, Fr[i], fmax);
        f[3 * i] = P.f1;
        f[3 * i + 1] = Y.a * P.fp - Y.b * P.fq;
        f[3 * i + 2] = Y.b * P.fp + Y.a * P.fq;
    }
    info[0] = o.ok;
    info[1] = o.steps;
}

}  // namespace

extern "C" {

// One grasp with m <= 8 contacts (p, n [m][3], mu [m]) and s wrenches t
// [s][6], from the points x0 [s][3 m]: forces f [s][3 m], info [s][2] (solved,
// Newton steps).
void host_newton_grasp(int cone, int m, const double* p, const double* n, const double* mu, const double* t, int s,
                       const double* x0, double eps, double fmax, int max_steps, double* f, int* info) {
    for (int j = 0; j < s; ++j)
        (cone ? solve_one<true> : solve_one<false>)(m, p, n, mu, t + 6 * j, x0 + 3 * m * j, eps, fmax, max_steps,
                                                    f + 3 * m * j, info + 2 * j);
}

// Projection of one contact's point y and its derivative (3 x 3, row-major)
// as the method composes it.
void host_newton_project(int cone, const double* y, double mu, double fmax, double* f, double* d) {
    auto go = [&](auto tag) {
        constexpr bool CONE = decltype(tag)::value;
        const NewtonFriction Fr = newton_friction(mu * (CONE ? 1.0 : kC8));
        const NewtonFold Y = newton_fold<CONE>(y[0], y[1], y[2]);
        const NewtonProj P = newton_project<CONE>(Y, Fr, fmax);
        const NewtonDeriv D = newton_deriv<CONE>(Y, P, Fr, fmax);
        f[0] = P.f1;
        f[1] = Y.a * P.fp - Y.b * P.fq;
        f[2] = Y.b * P.fp + Y.a * P.fq;
        const double ep[3] = {0.0, Y.a, Y.b}, eq[3] = {0.0, -Y.b, Y.a};
        double g[3];
        for (int t = 0; t < 3; ++t) g[t] = (t == 0 ? 1.0 : 0.0) + D.gp * ep[t] + D.gq * eq[t];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j)
                d[3 * i + j] = D.w1 * g[i] * g[j] + D.w2 * ep[i] * ep[j] + D.w3 * eq[i] * eq[j];
    };
    if (cone)
        go(std::true_type{});
    else
        go(std::false_type{});
}
}
