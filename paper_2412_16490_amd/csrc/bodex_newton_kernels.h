// bodex_newton_kernels.h -- gfx950 kernels of the dual Newton polish: the
// solve of every QP (newton_kernel) and the outputs of the solved ones
// (newton_out_kernel).
#pragma once

#include "bodex_kernels.h"
#include "bodex_newton.h"

namespace bodex {

// The cone's force c of a QP between the two kernels: its words in row c of z
// and of y at state column sw.
__device__ __forceinline__ void cone_keep(const KArgs& a, int c, size_t sw, double f) {
    const long long b = __double_as_longlong(f);
    a.z[size_t(c) * a.sW + sw] = __int_as_float(int(b));
    a.y[size_t(c) * a.sW + sw] = __int_as_float(int(b >> 32));
}
template <bool CONE>
__device__ __forceinline__ void newton_keep_word(const KArgs& a, int w, int word) {
    if constexpr (CONE)
        a.qobj[w] = __int_as_float(word);
    else
        a.ninfo[w] = word;
}
__device__ __forceinline__ double cone_kept(const KArgs& a, int c, size_t sw) {
    const unsigned lo = unsigned(__float_as_int(a.z[size_t(c) * a.sW + sw]));
    const unsigned hi = unsigned(__float_as_int(a.y[size_t(c) * a.sW + sw]));
    return __longlong_as_double((static_cast<long long>(hi) << 32) | lo);
}

// Solve: GS lanes per QP, 64 / GS QPs per one-wave workgroup; the GS parts of
// a tile are separate workgroups, so a hard QP holds up no more than the
// other groups of its wave.  Bound by FP64 issue and the dependent chain of
// the 6 x 6 factor and of the slopes; HBM traffic is the ADMM point in (12 m B
// per QP) and u out (52 B; the forces, 24 m B, of QPs that newton_fine ended and
// of the cone).  The contacts' geometry, the proximal centre and the
// group's scalars are in LDS: an early form with everything in registers (256,
// and spills) took 1105 us at 5 contacts and 131,072 QPs, with these in LDS 862
// (8 lanes per QP) and 734 (2 lanes).  At 629 us now (2 lanes), it and
// newton_out_kernel (35 us) replace, for the pyramid, the one-lane and
// contact-parallel active-set passes (1157 + 466 + 58 us).
template <int MM, int GS, bool CONE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) newton_kernel(const KArgs a) {
    constexpr int NC = (MM + GS - 1) / GS, PER = kWave / GS;
    using Store = NewtonStore<NC>;
    extern __shared__ __align__(16) double sGeo[];  // [slots MM + 1 (padding)][12]
    __shared__ double sCentre[Store::kCentre * kWave], sQp[Store::kQp * PER];
    __shared__ SlotInfo sInfo[kMaxSlots];
    const int lane = threadIdx.x, sub = lane % GS, grp = lane / GS;
    const int t = int(blockIdx.x) / GS, part = int(blockIdx.x) % GS;
    int nsl;
    load_slots(a, t, sInfo, nsl);
    for (int e = lane; e < nsl * MM + 1; e += kWave) {
        double* geo = sGeo + e * Store::kGeo;
        const int i = e % MM;
        if (e < nsl * MM && i < sInfo[e / MM].m) {
            const size_t base = (size_t(sInfo[e / MM].g) * a.ms + i) * 3;
            const double p[3] = {a.points[base], a.points[base + 1], a.points[base + 2]};
            const double n[3] = {a.normals[base], a.normals[base + 1], a.normals[base + 2]};
            newton_contact(p, n, double(a.kappa), geo);
        } else {
#pragma unroll
            for (int q = 0; q < Store::kGeo; ++q) geo[q] = 0.0;
        }
    }
    __syncthreads();
    int slot, j;
    lane_slot(sInfo, nsl, part * PER + grp, slot, j);
    if (slot < 0) return;  // the whole group
    const SlotInfo si = sInfo[slot];
    const int w = si.w0 + j;
    if (a.status[w] & kStNonfinite) {
        if (sub == 0) newton_keep_word<CONE>(a, w, 0);
        return;
    }
    const size_t sw = state_col(a, si, j);
    Store store;
    store.cp = sCentre + lane;
    store.cs = kWave;
    store.q = sQp + grp;
    store.qs = PER;
    NewtonFriction Fr[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int i = sub + GS * c;
        const bool live = i < si.m;
        store.geo[c] = sGeo + (live ? slot * MM + i : nsl * MM) * Store::kGeo;
#pragma unroll
        for (int q = 0; q < 3; ++q) store.centre(c, q) = live ? (a.x + size_t(3 * i + q) * a.sW)[sw] : 0.f;
        const double mu = live ? a.mu[size_t(si.g) * a.ms + i] : 0.5f;
        Fr[c] = newton_friction(CONE ? mu : mu * kC8);
    }
    double u[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) store.bt(r) = double(a.beta) * double(a.wrench[size_t(w) * 6 + r]);
    const NewtonOut o = newton_solve<GS, NC, CONE>(store, Fr, si.m, double(a.fmax), double(a.eps),
                                                   min(a.polish_steps, kNewtonSteps), u);
    if (o.ok && o.forces) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const int i = sub + GS * c;
            if (i < si.m)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    if constexpr (CONE)
                        cone_keep(a, 3 * i + q, sw, store.centre(c, q));
                    else
                        a.nu[size_t(3 * i + q) * a.W + w] = store.centre(c, q);
                }
        }
    } else if (!CONE && sub == 0) {
#pragma unroll
        for (int r = 0; r < 6; ++r) a.nu[size_t(r) * a.W + w] = u[r];
    }
    if (sub == 0) newton_keep_word<CONE>(a, w, newton_info(o));
}

// Multipliers of a pyramid contact's nine rows from its normal-cone vector
// N = 2 (G^T u - eps f) (folded: N1, along the nearest facet's normal, and
// across).  At the apex, where the eight facets leave a choice, the two
// nearest carry the tangential part and all eight share the rest of the
// normal one.
struct NewtonRows {
    int ka, kb;          // nearest facet, its neighbour
    double la, lb, ls, l8;  // their multipliers, the share of every facet, the bound row's
};

__device__ inline NewtonRows newton_rows(int face, const NewtonFold& Y, double N1, double N2, double N3, double k) {
    constexpr double kS45 = 0.70710678118654752440, kIS45 = 1.41421356237309504880;
    NewtonRows L;
    // at the apex the facet nearest to N itself, elsewhere y's
    NewtonFold F = Y;
    if (face == kNwApex) F = newton_fold<false>(N1, N2, N3);
    const double np = F.a * N2 + F.b * N3, nq = F.a * N3 - F.b * N2;
    const bool wide = fabs(F.a) > fabs(F.b);  // first and last facet of a quadrant
    const int quad = F.b < 0.0 ? (F.a < 0.0 ? 2 : 3) : (F.a < 0.0 ? 1 : 0);
    L.ka = 2 * quad + ((quad & 1) ? (wide ? 1 : 0) : (wide ? 0 : 1));
    const bool two = face == kNwEdge || face == kNwCapEdge || face == kNwApex;
    const bool up = face == kNwApex ? nq > 0.0 : F.q > 0.0;
    L.kb = (L.ka + (up ? 1 : 7)) & 7;
    L.lb = two ? fmax((up ? nq : -nq) * kIS45, 0.0) : 0.0;
    L.la = (face == kNwFree || face == kNwCap) ? 0.0 : fmax(np - L.lb * kS45, 0.0);
    const double rest = N1 + k * (L.la + L.lb);  // what the facets leave of the normal part
    L.l8 = face >= kNwCap ? fmax(rest, 0.0) : 0.0;
    L.ls = face == kNwApex ? fmax(-rest, 0.0) / (8.0 * k) : 0.0;
    return L;
}

// Outputs: forces and multipliers from u (or from the stored forces), objective, energy, the ADMM-form
// state of the point and its relative KKT residual (rel_kkt64's, of the
// rounded state, without reading it back).  Streams the state out: 4 (6 m +
// 18 m) B per QP at the pyramid's nine rows per contact.  QPs the Newton
// method left are counted in KArgs::nfail and keep their ADMM point; their
// outputs come from the finalize launch that follows.  Bound by HBM writes; at
// three waves per SIMD (166 registers) nothing spills, at four 140 B a lane
// did: 5 contacts, 131,072 QPs 43 -> 35 us, 951,279 QPs 417 -> 347, 8 contacts,
// 8547 QPs 36 -> 22.
template <int MM, bool CONE>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) newton_out_kernel(const KArgs a) {
    constexpr int NV = 3 * MM, NG = 6 * NV, RW = CONE ? 3 : 9;
    extern __shared__ __align__(16) unsigned char smem[];
    FinPtrs<MM> P;
    P.G = reinterpret_cast<double*>(smem);
    P.muc = P.G + size_t(a.slots) * NG;
    P.red = P.muc + size_t(a.slots) * 8;
    P.work = P.Gbar = nullptr;
    P.info = reinterpret_cast<SlotInfo*>(P.red + kWave);
    P.flag = reinterpret_cast<int*>(P.info + kMaxSlots);
    const int lane = threadIdx.x;
    int nsl;
    load_slots(a, blockIdx.x, P.info, nsl);
    int slot, j;
    lane_slot(P.info, nsl, lane, slot, j);
    const bool act = slot >= 0;
    SlotInfo si = {0, 0, 1, 0};
    if (act) si = P.info[slot];
    const bool good = fin_setup<MM>(a, P, nsl, slot, j, si, CONE);
    double Q = 0.0;
    if (act) {
        const double* Gs = P.G + size_t(slot) * NG;
        const double* muc = P.muc + slot * 8;
        const int w = si.w0 + j;
        const size_t W_ = size_t(a.sW), sw = state_col(a, si, j);
        unsigned char st = a.status[w];
        const int info = newton_word<CONE>(a, w);
        const bool finite_in = good && !(st & kStNonfinite);
        double bt[6];
#pragma unroll
        for (int r = 0; r < 6; ++r) bt[r] = double(a.beta) * double(a.wrench[size_t(w) * 6 + r]);
        if (finite_in && (info & kNewtonOk)) {
            const double eps = double(a.eps), ie = 1.0 / eps, fm = double(a.fmax);
            const bool forces = CONE || (info & kNewtonForces);
            double u[6];  // (of a QP whose forces are stored: below)
#pragma unroll
            for (int r = 0; r < 6; ++r) u[r] = CONE ? 0.0 : a.nu[size_t(r) * a.W + w];
            NewtonFriction Fr;  // of contact i
            // contact i's G^T u, folded point and projection
            auto contact = [&](int i, double* gu, NewtonFold& Y) -> NewtonProj {
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    double s = 0.0;
#pragma unroll
                    for (int r = 0; r < 6; ++r) s += Gs[r * NV + 3 * i + t] * u[r];
                    gu[t] = s;
                }
                Fr = newton_friction(muc[i]);
                Y = newton_fold<CONE>(gu[0] * ie, gu[1] * ie, gu[2] * ie);
                return newton_project<CONE>(Y, Fr, fm);
            };
            // its forces: as stored, or that projection's
            auto force = [&](int i, const NewtonFold& Y, const NewtonProj& p, double* f) {
                f[0] = p.f1;
                f[1] = Y.a * p.fp - Y.b * p.fq;
                f[2] = Y.b * p.fp + Y.a * p.fq;
                if (forces) {
#pragma unroll
                    for (int t = 0; t < 3; ++t)
                        f[t] = CONE ? cone_kept(a, 3 * i + t, sw) : a.nu[size_t(3 * i + t) * a.W + w];
                }
            };
            double r6[6], gx[6], ff = 0.0, s1 = 0.0;
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                r6[r] = -bt[r];
                gx[r] = 0.0;
            }
#pragma unroll 1
            for (int i = 0; i < a.ms; ++i) {
                double f[3] = {0.0, 0.0, 0.0};
                if (i < si.m) {
                    double gu[3];
                    NewtonFold Y;
                    const NewtonProj p = contact(i, gu, Y);
                    force(i, Y, p, f);
#pragma unroll
                    for (int t = 0; t < 3; ++t)
#pragma unroll
                        for (int r = 0; r < 6; ++r) {
                            const double g = Gs[r * NV + 3 * i + t];
                            r6[r] += g * f[t];
                            gx[r] += g * double(float(f[t]));
                        }
                    s1 += f[0];
                }
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    ff += f[t] * f[t];
                    a.x[size_t(3 * i + t) * W_ + sw] = float(f[t]);
                    a.forces[size_t(w) * 3 * a.ms + 3 * i + t] = float(f[t]);
                }
            }
            if (forces) {
#pragma unroll
                for (int r = 0; r < 6; ++r) u[r] = -r6[r];
            }
            // z, y and the residual of the rounded state
            double rp = 0, nAx = 0, nz = 0, rd = 0, nPx = 0, nAty = 0, nq = 0, t1 = 0.0;
#pragma unroll 1
            for (int i = 0; i < a.ms; ++i) {
                float zv[RW], yv[RW];
#pragma unroll
                for (int q = 0; q < RW; ++q) zv[q] = yv[q] = 0.f;
                if (i < si.m) {
                    double gu[3];
                    NewtonFold Y;
                    const NewtonProj p = contact(i, gu, Y);
                    const double k = muc[i];
                    const int face = newton_face<CONE>(Y, p, Fr, fm);
                    double f[3], N[3], x[3], aty[3] = {0.0, 0.0, 0.0};
                    force(i, Y, p, f);
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        N[t] = 2.0 * (gu[t] - eps * f[t]);
                        x[t] = double(float(f[t]));
                    }
                    if constexpr (CONE) {
#pragma unroll
                        for (int t = 0; t < 3; ++t) {
                            zv[t] = float(f[t]);
                            yv[t] = float(N[t]);
                            aty[t] = double(yv[t]);
                            nAx = fmax(nAx, fabs(x[t]));
                        }
                    } else {
                        const NewtonRows L = newton_rows(face, Y, N[0], N[1], N[2], k);
                        const bool on_a = face != kNwFree && face != kNwCap;
                        const bool on_b = face == kNwEdge || face == kNwCapEdge;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            const double ck = facet_cos<double>(q), sk = facet_sin<double>(q);
                            const bool on = face == kNwApex || (on_a && q == L.ka) || (on_b && q == L.kb);
                            const double l = L.ls + (q == L.ka ? L.la : 0.0) + (q == L.kb ? L.lb : 0.0);
                            zv[q] = on ? 0.f : fminf(float(ck * f[1] + sk * f[2] - k * f[0]), 0.f);
                            yv[q] = float(l);
                            const double ax = ck * x[1] + sk * x[2] - k * x[0], zk = double(zv[q]), yk = double(yv[q]);
                            rp = fmax(rp, fabs(ax - zk));
                            nAx = fmax(nAx, fabs(ax));
                            nz = fmax(nz, fabs(zk));
                            aty[0] -= k * yk;
                            aty[1] += ck * yk;
                            aty[2] += sk * yk;
                        }
                        zv[8] = face >= kNwCap ? a.fmax : fminf(fmaxf(float(f[0]), 0.f), a.fmax);
                        yv[8] = float(L.l8);
                        aty[0] += double(yv[8]);
                        rp = fmax(rp, fabs(x[0] - double(zv[8])));
                        nAx = fmax(nAx, fabs(x[0]));
                        nz = fmax(nz, fabs(double(zv[8])));
                    }
                    t1 += x[0];
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        double s = eps * x[t], qc = 0.0;
#pragma unroll
                        for (int r = 0; r < 6; ++r) {
                            const double g = Gs[r * NV + 3 * i + t];
                            s += g * gx[r];
                            qc += g * bt[r];
                        }
                        rd = fmax(rd, fabs(2.0 * s - 2.0 * qc + aty[t]));
                        nPx = fmax(nPx, fabs(2.0 * s));
                        nAty = fmax(nAty, fabs(aty[t]));
                        nq = fmax(nq, fabs(2.0 * qc));
                    }
                }
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    a.z[size_t(RW * i + q) * W_ + sw] = zv[q];
                    a.y[size_t(RW * i + q) * W_ + sw] = yv[q];
                }
            }
            const float zg = fmaxf(float(s1), a.gamma);
            a.z[size_t(RW * a.ms) * W_ + sw] = zg;
            a.y[size_t(RW * a.ms) * W_ + sw] = 0.f;
            if constexpr (CONE) nz = nAx;  // z = x
            rp = fmax(rp, fabs(t1 - double(zg)));
            nAx = fmax(nAx, fabs(t1));
            nz = fmax(nz, fabs(double(zg)));
            const double rel = fmax(rp / (1.0 + fmax(nAx, nz)), rd / (1.0 + fmax(fmax(nPx, nAty), nq)));
            double rr2 = 0.0;
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                rr2 += r6[r] * r6[r];
                if (a.resid) a.resid[size_t(r) * W_ + sw] = float(r6[r]);
            }
            Q = rr2 + eps * ff;
            st |= kStPolished;
            st &= ~kStPolishRej;
            st = rel <= double(a.tol) ? (st | kStConverged) : (st & ~kStConverged);
            a.status[w] = st;
            a.kkt[w] = float(rel);
            a.qobj[w] = float(Q);
            if (a.pflops) a.pflops[w] = float(newton_info_flops(si.m, info));
        } else {
            atomicAdd(a.nfail, 1);
        }
    }
    P.red[lane] = Q;
    __syncthreads();
    if (act && j == 0) {
        double E = 0.0;
        for (int l = lane; l < lane + si.s; ++l) E += P.red[l];
        a.energy[si.g] = float(E);
    }
}

template <int MM>
size_t newton_lds(int slots) {
    return size_t(slots * MM + 1) * NewtonStore<1>::kGeo * sizeof(double);
}

template <int MM>
size_t newton_out_lds(int slots) {
    return size_t(slots) * (6 * 3 * MM + 8) * 8 + kWave * 8 + kMaxSlots * 32 + 64;
}

}  // namespace bodex
