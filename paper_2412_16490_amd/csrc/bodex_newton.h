// bodex_newton.h -- FP64 solution of one contact-force QP in its dual, by a
// semismooth Newton method (no active-set bookkeeping).
//
// With u = beta t - G f the minimiser of |G f - beta t|^2 + eps |f|^2 over
// the contacts' friction cones C = prod C_i is f = P_C(G^T u / eps), the
// projection taken contact by contact in closed form, so the whole QP is six
// equations in six unknowns,
//     F(u) = G P_C(G^T u / eps) + u - beta t = 0,
// the gradient of a strictly convex, piecewise quadratic function of u
// (truncated pyramid; piecewise smooth for the circular cone).  Its
// generalised Hessian is I + G Pi G^T / eps with Pi the derivative of the
// projection (per contact: the projector onto the face that P_C hit), the
// same 6 x 6 matrix that an active-set method factors for that set of rows;
// a Newton step changes any number of rows of every contact at once, needs
// no multipliers and takes the same path on every lane.
//
// Globalisation: an exact line search along the Newton direction (the slope
// is a sum of per-contact terms: no matrix work), and, first, proximal steps
// of falling weight: with f' the last point and weight s,
//     f = P_C((G^T u + s f') / (eps + s)),
// whose regions are wider by (eps + s) / eps.  Over the ellipsoid workload (5
// contacts, 16 wrenches) from the 20-iteration ADMM point a QP takes 12.4
// Newton steps and 26 slopes on average (99 % within 21 steps, the longest
// 31), against 13 factorisations, 9 row steps and 6.5 row searches, each with
// its own passes over the contacts, for the active-set polish.
//
// Rounding: y = G^T u / eps carries that of u, 1e-16 |beta t| / eps, which at
// long torque arms or a large beta t exceeds what F has to fall below.  Such a
// QP (newton_solve) is ended by newton_fine, which carries u and y in two
// doubles each.
//
// Mapping: GS lanes per QP (1, 2, 4 or 8), lane `sub` owns the contacts sub,
// sub + GS, ...; u, the 6 x 6 factor and the line search are replicated, the
// sums over contacts are butterflies of DPP moves, whose pairwise additions
// give every lane of the group the same bits, so its control flow is uniform.
#pragma once

#include "bodex_gpolish.h"
#include "bodex_math.h"

namespace bodex {

constexpr double kTan8 = 0.41421356237309504880;  // tan(pi/8)

// A contact as the method reads it: its frame (rows n, d, e) and kappa p, and
// the friction terms: the facet coefficient k = mu cos(pi/8) (the cone's mu),
// kt = k tan(pi/8) and the inverse squared lengths of a facet's and an edge's
// directions.
struct NewtonContact {
    double R[9], kp[3];
};
struct NewtonFriction {
    double k, kt, i1, i2;
};

BODEX_FI NewtonFriction newton_friction(double k) {
    NewtonFriction F;
    F.k = k;
    F.kt = k * kTan8;
    F.i1 = 1.0 / (1.0 + k * k);
    F.i2 = 1.0 / (1.0 + k * k + F.kt * F.kt);
    return F;
}

// Geometry of the contact at p with normal n: its frame, kappa p.
BODEX_FI void newton_contact(const double p[3], const double n[3], double kappa, double* geo) {
    double R[9];
    contact_frame<double>(n[0], n[1], n[2], R, R + 3, R + 6);
#pragma unroll
    for (int t = 0; t < 9; ++t) geo[t] = R[t];
#pragma unroll
    for (int t = 0; t < 3; ++t) geo[9 + t] = kappa * p[t];
}

// What is kept in memory between its uses (LDS on the GPU; in registers it
// would cost a third of the occupancy): the geometry of the lane's contacts
// (12 doubles each, shared by the grasp's QPs), the proximal centre of its
// contacts (entry e at centre[e * cs]), and the QP's beta t and schedule,
// which the lanes of a group share (they write the same bits; entry e at
// q[e * qs]; in registers the two last cost another 1 % at 131,072 QPs).
template <int NC>
struct NewtonStore {
    static constexpr int kGeo = 12, kCentre = 3 * NC, kQp = 18;
    const double* geo[NC];
    double* cp;
    int cs;
    double* q;
    int qs;
    BODEX_FI NewtonContact contact(int c) const {
        NewtonContact C;
#pragma unroll
        for (int t = 0; t < 9; ++t) C.R[t] = geo[c][t];
#pragma unroll
        for (int t = 0; t < 3; ++t) C.kp[t] = geo[c][9 + t];
        return C;
    }
    BODEX_FI double& centre(int c, int t) const { return cp[(3 * c + t) * cs]; }
    BODEX_FI double& bt(int r) const { return q[r * qs]; }
    BODEX_FI double& tol() const { return q[6 * qs]; }
    BODEX_FI double& scale() const { return q[7 * qs]; }
    BODEX_FI double& ratio() const { return q[8 * qs]; }  // of the proximal weight, and
    BODEX_FI double& last() const { return q[9 * qs]; }   // its last value before zero
    BODEX_FI double& ref(int r) const { return q[(10 + r) * qs]; }  // u some steps back
    BODEX_FI double& end() const { return q[16 * qs]; }   // F's tolerance at the end,
    BODEX_FI double& fine() const { return q[17 * qs]; }  // and whether newton_fine is the end
};

// A number as the sum of two doubles (hi the rounded value), by error-free
// transformations: Knuth's sum, products with fma.  No contraction: the
// compiler must not fuse one of their products into the sum that follows.
struct NewtonTwo {
    double hi, lo;
};
#if defined(__clang__)
#define BODEX_NO_CONTRACT _Pragma("clang fp contract(off)")
#else
#define BODEX_NO_CONTRACT
#endif
BODEX_FI NewtonTwo two_sum(double a, double b) {
    BODEX_NO_CONTRACT
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
BODEX_FI NewtonTwo two_add(NewtonTwo a, NewtonTwo b) {
    BODEX_NO_CONTRACT
    const NewtonTwo s = two_sum(a.hi, b.hi);
    const double lo = s.lo + (a.lo + b.lo), hi = s.hi + lo;
    return {hi, lo - (hi - s.hi)};
}
BODEX_FI NewtonTwo two_mul(double a, NewtonTwo b) {
    BODEX_NO_CONTRACT
    const double p = a * b.hi, lo = fma(a, b.hi, -p) + a * b.lo, hi = p + lo;
    return {hi, lo - (hi - p)};
}

// R^T-rotated wrench: the contact's three rows of G^T w.
BODEX_FI void newton_gt(const NewtonContact& C, const double* w, double* v) {
    const double h[3] = {w[0] + (w[4] * C.kp[2] - w[5] * C.kp[1]), w[1] + (w[5] * C.kp[0] - w[3] * C.kp[2]),
                         w[2] + (w[3] * C.kp[1] - w[4] * C.kp[0])};
#pragma unroll
    for (int t = 0; t < 3; ++t) v[t] = C.R[3 * t] * h[0] + C.R[3 * t + 1] * h[1] + C.R[3 * t + 2] * h[2];
}

// The same of w + dw.
BODEX_FI void newton_gt_two(const NewtonContact& C, const double* w, const double* dw, NewtonTwo* v) {
    NewtonTwo W[6], h[3];
#pragma unroll
    for (int r = 0; r < 6; ++r) W[r] = two_sum(w[r], dw[r]);
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int a = (t + 1) % 3, b = (t + 2) % 3;
        h[t] = two_add(W[t], two_add(two_mul(C.kp[b], W[3 + a]), two_mul(-C.kp[a], W[3 + b])));
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
        v[t] = two_add(two_mul(C.R[3 * t], h[0]), two_add(two_mul(C.R[3 * t + 1], h[1]), two_mul(C.R[3 * t + 2], h[2])));
}

// The contact's vector v (normal, d, e) in the world frame.
BODEX_FI void newton_world(const NewtonContact& C, double v1, double v2, double v3, double* w) {
#pragma unroll
    for (int t = 0; t < 3; ++t) w[t] = C.R[t] * v1 + C.R[3 + t] * v2 + C.R[6 + t] * v3;
}

// A contact's point y on the half plane its projection works in: y1 along
// the axis, p along the nearest facet's normal (the radius for the cone), q
// across; (a, b) the direction of p in the tangent plane, q along (-b, a).
struct NewtonFold {
    double y1, p, q, a, b;
};

template <bool CONE>
BODEX_FI NewtonFold newton_fold(double y1, double y2, double y3) {
    NewtonFold f;
    f.y1 = y1;
    if constexpr (CONE) {
        const double r2 = y2 * y2 + y3 * y3;
        const double ir = r2 > 0.0 ? 1.0 / sqrt(r2) : 0.0;
        f.a = r2 > 0.0 ? y2 * ir : 1.0;
        f.b = y3 * ir;
        f.p = r2 * ir;
        f.q = 0.0;
    } else {
        const bool sw = fabs(y3) > fabs(y2);
        f.a = copysign(sw ? kS8 : kC8, y2);
        f.b = copysign(sw ? kC8 : kS8, y3);
        f.p = f.a * y2 + f.b * y3;
        f.q = f.a * y3 - f.b * y2;
    }
    return f;
}

// Projection of a folded point onto the truncated cone.  With ff and fe the
// axial positions of the nearest points on the facet's plane and on the edge's
// line, f1 is the largest of y1 (inside), ff (facet) and fe (edge), clamped to
// [0, fmax] (apex, cap), and the tangential part is y's, cut off at the section
// there: every region of the projection without a case distinction.
struct NewtonProj {
    double f1, fp, fq;  // the projection
    double m, ff, fe;   // unclamped f1 and its candidates
};

template <bool CONE>
BODEX_FI NewtonProj newton_project(const NewtonFold& y, const NewtonFriction& C, double fmax) {
    NewtonProj P;
    const double t = y.y1 + C.k * y.p;
    P.ff = t * C.i1;
    P.m = __builtin_fmax(y.y1, P.ff);
    P.fe = 0.0;
    if constexpr (!CONE) {
        P.fe = (t + C.kt * fabs(y.q)) * C.i2;
        P.m = __builtin_fmax(P.m, P.fe);
    }
    P.f1 = __builtin_fmin(__builtin_fmax(P.m, 0.0), fmax);
    P.fp = __builtin_fmin(y.p, C.k * P.f1);
    P.fq = CONE ? 0.0 : copysign(__builtin_fmin(fabs(y.q), C.kt * P.f1), y.q);
    return P;
}

// Fold and projection of a point in two doubles: far from the cone f1 is what
// is left of terms many times its size.
template <bool CONE>
BODEX_FI NewtonProj newton_project_two(const NewtonTwo (&y)[3], const NewtonFriction& C, double fmax, NewtonFold& Y) {
    Y = newton_fold<CONE>(y[0].hi, y[1].hi, y[2].hi);
    NewtonTwo p, q = {0.0, 0.0};
    if constexpr (CONE) {  // the radius: a Newton step for the square root from its rounded value
        const NewtonTwo sq = two_add(two_add(two_mul(y[1].hi, y[1]), two_mul(y[2].hi, y[2])),
                                     {y[1].lo * y[1].hi + y[2].lo * y[2].hi, 0.0});
        const double over = two_add(sq, two_mul(-Y.p, {Y.p, 0.0})).hi;
        p = Y.p > 0.0 ? two_sum(Y.p, 0.5 * over / Y.p) : q;
    } else {
        p = two_add(two_mul(Y.a, y[1]), two_mul(Y.b, y[2]));
        q = two_add(two_mul(Y.a, y[2]), two_mul(-Y.b, y[1]));
        Y.q = q.hi;
        if (q.hi < 0.0) q = {-q.hi, -q.lo};
    }
    Y.p = p.hi;
    NewtonProj P;
    const NewtonTwo t = two_add(y[0], two_mul(C.k, p));
    P.ff = t.hi * C.i1;
    P.m = __builtin_fmax(Y.y1, P.ff);
    P.fe = 0.0;
    if constexpr (!CONE) {
        P.fe = two_add(t, two_mul(C.kt, q)).hi * C.i2;
        P.m = __builtin_fmax(P.m, P.fe);
    }
    P.f1 = __builtin_fmin(__builtin_fmax(P.m, 0.0), fmax);
    P.fp = __builtin_fmin(Y.p, C.k * P.f1);
    P.fq = CONE ? 0.0 : copysign(__builtin_fmin(q.hi, C.kt * P.f1), Y.q);
    return P;
}

// Its derivative w1 g g^T + w2 e_p e_p^T + w3 e_q e_q^T, g = (1, gp, gq).
struct NewtonDeriv {
    double w1, gp, gq, w2, w3;
};

template <bool CONE>
BODEX_FI NewtonDeriv newton_deriv(const NewtonFold& y, const NewtonProj& P, const NewtonFriction& C, double fmax) {
    NewtonDeriv D;
    const bool moves = P.m > 0.0 && P.m < fmax, free = P.m == y.y1;
    const bool edge = !CONE && P.fe > P.ff;
    D.w1 = !moves ? 0.0 : (free ? 1.0 : (edge ? C.i2 : C.i1));
    D.gp = free ? 0.0 : C.k;
    D.gq = (free || !edge) ? 0.0 : copysign(C.kt, y.q);
    D.w2 = y.p < C.k * P.f1 ? 1.0 : 0.0;
    if constexpr (CONE)
        D.w3 = y.p < C.k * P.f1 ? 1.0 : (y.p > 0.0 ? P.fp / y.p : 0.0);  // turning about the axis: |f_t| / |y_t|
    else
        D.w3 = fabs(y.q) < C.kt * P.f1 ? 1.0 : 0.0;
    return D;
}

// Which rows are active at a projection.
enum NewtonFace { kNwFree, kNwFacet, kNwEdge, kNwApex, kNwCap, kNwCapFacet, kNwCapEdge };
template <bool CONE>
BODEX_FI int newton_face(const NewtonFold& y, const NewtonProj& P, const NewtonFriction& C, double fmax) {
    if (!(P.m > 0.0)) return kNwApex;
    const bool side = !(y.p < C.k * P.f1) && (P.m != y.y1 || P.m > fmax);
    const bool corner = !CONE && side && !(fabs(y.q) < C.kt * P.f1);
    return (P.m > fmax ? kNwCap : kNwFree) + (corner ? 2 : (side ? 1 : 0));
}

// Adds a contact's image G f to s[0..5] and its block G Pi G^T to s[6..26].
BODEX_FI void newton_terms(const NewtonContact& C, const NewtonFold& Y, const NewtonProj& P, const NewtonDeriv& D,
                           double* s) {
    const double* kp = C.kp;
    double w[3];
    newton_world(C, P.f1, Y.a * P.fp - Y.b * P.fq, Y.b * P.fp + Y.a * P.fq, w);
#pragma unroll
    for (int t = 0; t < 3; ++t) s[t] += w[t];
    s[3] += kp[1] * w[2] - kp[2] * w[1];
    s[4] += kp[2] * w[0] - kp[0] * w[2];
    s[5] += kp[0] * w[1] - kp[1] * w[0];
    // S = Pi in the world frame (3 x 3), then its force, torque-force
    // and torque blocks with [kp]x
    double ep[3], eq[3], g[3];
    newton_world(C, 0.0, Y.a, Y.b, ep);
    newton_world(C, 0.0, -Y.b, Y.a, eq);
#pragma unroll
    for (int t = 0; t < 3; ++t) g[t] = C.R[t] + D.gp * ep[t] + D.gq * eq[t];
    double S[3][3], w1g[3], w2p[3], w3q[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        w1g[t] = D.w1 * g[t];
        w2p[t] = D.w2 * ep[t];
        w3q[t] = D.w3 * eq[t];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
            S[i][j] = w1g[i] * g[j] + w2p[i] * ep[j] + w3q[i] * eq[j];
            S[j][i] = S[i][j];
        }
    double* M = s + 6;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) M[lo_idx(i, j)] += S[i][j];
    double T[3][3];  // K S, K = [kp]x
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        T[0][j] = kp[1] * S[2][j] - kp[2] * S[1][j];
        T[1][j] = kp[2] * S[0][j] - kp[0] * S[2][j];
        T[2][j] = kp[0] * S[1][j] - kp[1] * S[0][j];
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j) M[lo_idx(3 + i, j)] += T[i][j];
        // (K S) K^T, lower triangle: row i of T crossed with kp
        M[lo_idx(3 + i, 3)] += T[i][2] * kp[1] - T[i][1] * kp[2];
        if (i >= 1) M[lo_idx(3 + i, 4)] += T[i][0] * kp[2] - T[i][2] * kp[0];
        if (i >= 2) M[lo_idx(3 + i, 5)] += T[i][1] * kp[0] - T[i][0] * kp[1];
    }
}

// Reciprocal to the last bits (pivots of the factorisation, positive).
BODEX_FI double newton_rcp(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
#else
    return 1.0 / x;
#endif
}

// M = L D L^T in place (packed lower, unit L; the diagonal holds 1 / D), and
// the solve.  False when a pivot is not positive.
BODEX_FI bool ldl6(double* M) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        double c[6];  // L_jl D_l
        double d = M[lo_idx(j, j)];
#pragma unroll
        for (int l = 0; l < j; ++l) {
            c[l] = M[lo_idx(j, l)];
            M[lo_idx(j, l)] = c[l] * M[lo_idx(l, l)];
            d -= c[l] * M[lo_idx(j, l)];
        }
        ok = ok && d > 0.0;
        M[lo_idx(j, j)] = newton_rcp(d);
#pragma unroll
        for (int i = j + 1; i < 6; ++i)
#pragma unroll
            for (int l = 0; l < j; ++l) M[lo_idx(i, j)] -= M[lo_idx(i, l)] * M[lo_idx(j, l)];
    }
    return ok;
}

BODEX_FI void ldl6_solve(const double* L, double* v) {
#pragma unroll
    for (int i = 1; i < 6; ++i)
#pragma unroll
        for (int l = 0; l < i; ++l) v[i] -= L[lo_idx(i, l)] * v[l];
#pragma unroll
    for (int i = 5; i >= 0; --i) {
        v[i] *= L[lo_idx(i, i)];
#pragma unroll
        for (int l = i + 1; l < 6; ++l) v[i] -= L[lo_idx(l, i)] * v[l];
    }
}

// Sums over the lanes of a group (bits equal on all of them).  The third
// stage takes the mirrored lane of the eight, which after the first two holds
// the other quad's sum.
#if defined(__HIPCC__)
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_mov_dpp(int(b), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(int(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
#endif
template <int GS, int N>
BODEX_FI void group_sum(double (&v)[N]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if constexpr (GS >= 2) v[j] += dpp_move<0xB1>(v[j]);   // quad_perm [1,0,3,2]
        if constexpr (GS >= 4) v[j] += dpp_move<0x4E>(v[j]);   // quad_perm [2,3,0,1]
        if constexpr (GS >= 8) v[j] += dpp_move<0x141>(v[j]);  // row_half_mirror
    }
#elif !defined(__HIPCC__)
    static_assert(GS == 1, "the host build runs one thread per QP");
#endif
}

// Schedule of the proximal weight, in units of the mean squared length of a
// contact's three wrenches: from `first`, times `ratio` per Newton step, and
// zero below `last`.  The cone starts lower (its ADMM point is three digits
// closer) and falls faster.  Swept on the 131,072 QPs of the ellipsoid workload
// for the largest step and slope counts among 8 neighbouring QPs (which share
// a wave) and the length of the tail: ratios 0.4 / 0.5 / 0.6 / 0.7 take 10.3 /
// 11.0 / 12.4 / 14.3 steps and 40 / 33 / 26 / 24 slopes per QP.
struct ProxSchedule {
    double first, ratio, last;
};
constexpr ProxSchedule kProxPyramid = {0.1, 0.6, 2e-4}, kProxCone = {1e-3, 0.3, 1e-5},
                       kProxRestart = {3e-4, 0.6, 3e-6};
// At weight zero the steps of a few QPs (0.3 % of the ellipsoid workload) run
// in cycles of two or three between the walls of one contact's force range,
// drifting slowly along a valley; every kZigzag steps the method therefore
// searches along the last kZigzag steps' sum instead, with no bound on its
// length (pyramid only: the longest QP of the workload 51 -> 31 steps).  A QP
// not done within kProxStuck steps goes round again from kProxRestart, at most
// kProxRounds times.
constexpr int kZigzagFrom = 2, kZigzag = 6, kProxStuck = 40, kProxRounds = 3;
// The line search ends once the slope is this small against the one at the
// start of the step, with and without a proximal weight.  At weight zero the
// search has to land inside the thin regions between two faces.
constexpr double kSlopeProx = 0.1, kSlopeZero = 0.005;
constexpr double kNewtonTol = 2e-9;  // |F|_inf relative to |beta t|

constexpr int kNewtonSteps = 200;      // cap on the Newton steps of a QP

// The last proximal weight is at most this many eps.  Beyond a mean squared
// length of 20 (the workloads' contacts reach 8) the schedules above would
// leave a wider and wider gap down to eps, which the line search at weight
// zero has to bridge: torque_scale 400 / 1000 / 4000, slopes per QP 160 / 219 /
// 279 without the limit, 85 / 97 / 111 with it.
constexpr double kProxLast = 4000.0;

// A QP is ended by newton_fine when the rounding of y exceeds kFineForce (the
// forces' own error against it: 1e-10 up to there), or that of F its
// tolerance; F's tolerance until then: kFineTol times its rounding.
constexpr double kFineForce = 1e-9, kFineTol = 4.0;
constexpr int kFineSteps = 6;

struct NewtonOut {
    int ok, steps, evals, slopes;
    int forces;  // the forces are in the store's centre (newton_fine; always of the cone)
};

// Algorithmic FP64 flops of one solve (FMA = 2, add/mul/div = 1, selects and
// compares 0) at m contacts: start and outputs 27 m + 227 m, an evaluation of
// F and its matrix 236 m (G^T u 27, point 9, fold and projection 26, image 30,
// derivative 78, blocks 66), a Newton step 30 m + 235 (factor 91, solve 66,
// scalars), a slope 51 m + 9.  Moves of the proximal centre are not counted.
BODEX_FI double newton_flops(int m, int steps, int evals, int slopes) {
    return 254.0 * m + evals * (236.0 * m) + steps * (30.0 * m + 235.0) + slopes * (51.0 * m + 9.0);
}

// Puts a contact's projection into the store's centre.
template <int NC>
BODEX_FI void newton_keep(const NewtonStore<NC>& st, int c, const NewtonFold& Y, const NewtonProj& P) {
    st.centre(c, 0) = P.f1;
    st.centre(c, 1) = Y.a * P.fp - Y.b * P.fq;
    st.centre(c, 2) = Y.b * P.fp + Y.a * P.fq;
}

// Newton steps at weight zero on u + lo, with y and its projection in two
// doubles: F then falls to the rounding of its own sum, whatever |u| / eps.  The
// forces, which u alone does not hold, are left in the store's centre.  Largest
// force error of 4800 QPs (5 contacts, cold starts) without / with it: beta 100
// 2e-8 / 7e-15, beta 1000 1e-7 / 5e-14; torque arms of 50: 123 QPs above the
// tolerance after 128 steps / none, of 200: 829 / none.  Whole solve on the GPU,
// 131,072 QPs, torque_scale 400 / 1000 / 4000: 10.6 / 16.9 / 20.4 ms without, 1.05
// / 1.16 / 1.41 with; at beta 100, where it adds an iteration, 0.60 / 0.63.
template <int GS, int NC, bool CONE>
BODEX_FI bool newton_fine(const NewtonStore<NC>& st, const NewtonFriction (&Fr)[NC], double fm, double eps,
                          const double (&u)[6], NewtonOut& out) {
    const double ie = 1.0 / eps;
    double lo[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int k = 0;; ++k) {
        BODEX_SPLIT();
        ++out.evals;
        double s[27];
#pragma unroll
        for (int j = 0; j < 27; ++j) s[j] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const NewtonContact C = st.contact(c);
            NewtonTwo y[3];
            newton_gt_two(C, u, lo, y);
#pragma unroll
            for (int t = 0; t < 3; ++t) y[t] = two_mul(ie, y[t]);
            NewtonFold Y;
            const NewtonProj P = newton_project_two<CONE>(y, Fr[c], fm, Y);
            newton_terms(C, Y, P, newton_deriv<CONE>(Y, P, Fr[c], fm), s);
            newton_keep(st, c, Y, P);
            BODEX_SPLIT();
        }
        group_sum<GS>(s);
        double res = 0.0, all = 0.0, d[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            d[r] = s[r] + ((u[r] - st.bt(r)) + lo[r]);
            res = __builtin_fmax(res, fabs(d[r]));
            all += fabs(d[r]);
        }
        if (!(all < INFINITY)) return false;
        if ((k > 0 && res <= 1e-3 * st.end()) || k == kFineSteps) return res <= st.end();
        double* M = s + 6;
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            d[r] *= -eps;
            M[lo_idx(r, r)] += eps;
        }
        if (!ldl6(M)) return false;
        ldl6_solve(M, d);
#pragma unroll
        for (int r = 0; r < 6; ++r) lo[r] += d[r];
        ++out.steps;
    }
}

// Solve one QP: u <- the dual solution (NewtonOut::forces: the forces are in the
// centre, and of u only its rounding).  st holds the lane's contacts, beta t
// and the starting forces (the proximal centre, overwritten), Fr the contacts'
// friction terms, m the contacts of the grasp.  Every lane of the group calls it.
template <int GS, int NC, bool CONE>
BODEX_FI NewtonOut newton_solve(const NewtonStore<NC>& st, const NewtonFriction (&Fr)[NC], int m, double fm, double eps,
                                int max_steps, double (&u)[6]) {
    NewtonOut out = {0, 0, 0, 0, 0};
    // u = beta t - G f
    double len[1] = {0.0};
    {
#pragma unroll
        for (int r = 0; r < 6; ++r) u[r] = 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const NewtonContact C = st.contact(c);
            double w[3];
            newton_world(C, st.centre(c, 0), st.centre(c, 1), st.centre(c, 2), w);
            const double* kp = C.kp;
            const double n2 = C.R[0] * C.R[0] + C.R[1] * C.R[1] + C.R[2] * C.R[2];  // 1, padding 0
            len[0] += 3.0 * n2 + 2.0 * (kp[0] * kp[0] + kp[1] * kp[1] + kp[2] * kp[2]);
#pragma unroll
            for (int t = 0; t < 3; ++t) u[t] += w[t];
            u[3] += kp[1] * w[2] - kp[2] * w[1];
            u[4] += kp[2] * w[0] - kp[0] * w[2];
            u[5] += kp[0] * w[1] - kp[1] * w[0];
        }
        group_sum<GS>(u);
#pragma unroll
        for (int r = 0; r < 6; ++r) u[r] = st.bt(r) - u[r];
    }
    double t2 = 0.0;
#pragma unroll
    for (int r = 0; r < 6; ++r) t2 += st.bt(r) * st.bt(r);
    // the second term grows neither with an fmax that no force reaches nor against
    // a small beta t; the third ends a solve of beta t = 0 from other forces
    st.end() = kNewtonTol * sqrt(t2) + 1e-12 * fmin(fm, 1.0) * fmin(1e3 * sqrt(t2), 1.0) + 1e-24;
    group_sum<GS>(len);
    st.scale() = len[0] / m;
    {
        // 2^-53 |beta t| / eps is the rounding of u / eps, times a row of G that
        // of y, times its square that of F (compared squared: no root or
        // division on the way of the QPs that it does not concern)
        const double sc = st.scale();
        const bool fine = 0x1p-106 * t2 * sc > kFineForce * kFineForce * eps * eps || 0x1p-53 * sc > kNewtonTol * eps;
        st.fine() = fine ? 1.0 : 0.0;
        st.tol() = fine ? fmax(st.end(), kFineTol * 0x1p-53 * sqrt(t2) / eps * sc) : st.end();
    }
    const ProxSchedule first = CONE ? kProxCone : kProxPyramid;
    st.ratio() = first.ratio;
    st.last() = fmax(fmin(first.last * st.scale(), kProxLast * eps), 10.0 * eps);
    double prox = first.first * st.scale();
    if (prox < 10.0 * eps) prox = 0.0;
    int at_zero = 0, rounds = 0;
#pragma unroll 1
    for (;;) {
        BODEX_SPLIT();  // the store is read anew
        const double e = eps + prox, ie = 1.0 / e;
        ++out.evals;
        // F and the matrix e I + G Pi G^T at u
        double s[27];
#pragma unroll
        for (int j = 0; j < 27; ++j) s[j] = 0.0;
        double y[NC][3];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const NewtonContact C = st.contact(c);
            newton_gt(C, u, y[c]);
#pragma unroll
            for (int t = 0; t < 3; ++t) y[c][t] = (y[c][t] + prox * st.centre(c, t)) * ie;
            const NewtonFold Y = newton_fold<CONE>(y[c][0], y[c][1], y[c][2]);
            const NewtonProj P = newton_project<CONE>(Y, Fr[c], fm);
            const NewtonDeriv D = newton_deriv<CONE>(Y, P, Fr[c], fm);
            newton_terms(C, Y, P, D, s);
        }
        group_sum<GS>(s);
        double res = 0.0, all = 0.0, d[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            d[r] = s[r] + (u[r] - st.bt(r));
            res = __builtin_fmax(res, fabs(d[r]));
            all += fabs(d[r]);
        }
        if (!(all < INFINITY)) break;
        const bool small = res <= (prox > 0.0 ? 1e3 * st.tol() : st.tol());
        if (small && prox == 0.0) {
            out.ok = 1;
            if constexpr (CONE) {
                out.forces = 1;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const NewtonFold Y = newton_fold<CONE>(y[c][0], y[c][1], y[c][2]);
                    newton_keep(st, c, Y, newton_project<CONE>(Y, Fr[c], fm));
                }
            }
            break;
        }
        if (out.steps >= max_steps) break;
        double al = 0.0, dy[NC][3];
        if (!small) {
            double F[6], g0 = 0.0;
            double* M = s + 6;
#pragma unroll
            for (int r = 0; r < 6; ++r) F[r] = d[r];
            const bool mark = !CONE && prox == 0.0 && at_zero >= kZigzagFrom && (at_zero - kZigzagFrom) % kZigzag == 0;
            bool along = mark && at_zero > kZigzagFrom;
            if (along) {  // the sum of the last kZigzag steps
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    d[r] = u[r] - st.ref(r);
                    g0 += F[r] * d[r];
                }
                along = g0 < 0.0;
            }
            if (mark) {
#pragma unroll
                for (int r = 0; r < 6; ++r) st.ref(r) = u[r];
            }
            if (!along) {
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    d[r] = -e * F[r];
                    M[lo_idx(r, r)] += e;
                }
                if (!ldl6(M)) break;
                ldl6_solve(M, d);
                g0 = 0.0;
#pragma unroll
                for (int r = 0; r < 6; ++r) g0 += F[r] * d[r];
            }
            ++out.steps;
            BODEX_SPLIT();
            double du = 0.0, dd = 0.0;
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                du += d[r] * (u[r] - st.bt(r));
                dd += d[r] * d[r];
            }
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                newton_gt(st.contact(c), d, dy[c]);
#pragma unroll
                for (int t = 0; t < 3; ++t) dy[c][t] *= ie;
            }
            // line search: the zero of the slope in (0, 1] (the slope rises
            // from g0 < 0; not above zero at 1: the full step)
            const double lim = (prox > 0.0 ? kSlopeProx : kSlopeZero) * fabs(g0);
            double lo = 0.0, hi = along ? INFINITY : 1.0, glo = g0;
            al = 1.0;
#pragma unroll 1
            for (int k = 0; k < 48; ++k) {
                double v[2] = {0.0, 0.0};  // slope and curvature
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const NewtonFold Y = newton_fold<CONE>(y[c][0] + al * dy[c][0], y[c][1] + al * dy[c][1],
                                                           y[c][2] + al * dy[c][2]);
                    const NewtonProj P = newton_project<CONE>(Y, Fr[c], fm);
                    const double dp = Y.a * dy[c][1] + Y.b * dy[c][2], dq = Y.a * dy[c][2] - Y.b * dy[c][1];
                    v[0] += dy[c][0] * P.f1 + dp * P.fp + dq * P.fq;
                    const NewtonDeriv D = newton_deriv<CONE>(Y, P, Fr[c], fm);
                    const double gd = dy[c][0] + D.gp * dp + D.gq * dq;
                    v[1] += D.w1 * gd * gd + D.w2 * dp * dp + D.w3 * dq * dq;
                }
                group_sum<GS>(v);
                ++out.slopes;
                const double gs = e * v[0] + (du + al * dd), cu = e * v[1] + dd;
                if (fabs(gs) <= lim || (k == 0 && !along && gs <= 0.0)) break;
                if (gs > 0.0)
                    hi = al;
                else {
                    lo = al;
                    glo = gs;
                }
                double nx = al - gs * newton_rcp(cu);
                if (!(hi < INFINITY)) {
                    nx = 8.0 * al;
                } else if (!(nx > lo && nx < hi)) {
                    if (k == 0)
                        nx = lo - glo * (hi - lo) * newton_rcp(gs - glo);
                    else
                        nx = lo > 0.0 ? double(sqrtf(float(lo) * float(hi))) : 0.05 * hi;
                    if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
                }
                if (!(nx > lo && nx < hi)) break;
                al = nx;
            }
#pragma unroll
            for (int r = 0; r < 6; ++r) u[r] += al * d[r];
        }
        // next proximal centre and weight
        bool recentre = prox > 0.0;
        if (prox == 0.0 && ++at_zero >= kProxStuck) {
            if (rounds == kProxRounds) break;
            ++rounds;
            at_zero = 0;
            recentre = true;
            prox = kProxRestart.first / kProxRestart.ratio * st.scale();
            st.ratio() = kProxRestart.ratio;
            st.last() = fmax(fmin(kProxRestart.last * st.scale(), kProxLast * eps), 10.0 * eps);
        }
        if (recentre) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                double v[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) v[t] = al == 0.0 ? y[c][t] : y[c][t] + al * dy[c][t];
                const NewtonFold Y = newton_fold<CONE>(v[0], v[1], v[2]);
                newton_keep(st, c, Y, newton_project<CONE>(Y, Fr[c], fm));
            }
            prox *= st.ratio();
            if (prox < st.last()) prox = 0.0;
        }
    }
    if (out.ok && st.fine() != 0.0) out.ok = out.forces = newton_fine<GS, NC, CONE>(st, Fr, fm, eps, u, out) ? 1 : 0;
    return out;
}

}  // namespace bodex
