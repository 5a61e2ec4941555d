// xf_vjp64.hpp -- the face VJP in FP64: the backward of the forms of
// xf_face64.hpp (face_vjp of xf_vjp.hpp is its FP32 counterpart, with the
// same interface).
//
// What bounds it: one wave per SIMD (the backward of a face holds about 200
// live values), so the time is the length of a wave's instruction stream.
// Against the plain forms:
//   * a WENO5 side and its backward run on the four first differences with
//     one reciprocal (the weights' denominator times the product of the three
//     indicators) instead of four: 73 operations instead of about 125;
//   * per-cell sums over species are not differentiated species by species:
//     with t = E - u.m + q^2/2 rho - sum_s e_s rho_s and S = sum_s R_s rho_s
//     the projection is DU = Gi t + Ti S, DF = u_n DU + Gi p (u_n - u~_n),
//     and a partial density's cotangent is (T~/Gamma R_s - e_s) tbar;
//   * the acoustic pair is taken back together, and a partial density's
//     contributions of one loop go to LDS in one add.
#pragma once

#include "xf_face64.hpp"

namespace xf {

struct WenoVjpK : WenoK {
    double c55, c25, c24;
    XF_HD WenoVjpK() : c55(in_sgpr(5.5)), c25(in_sgpr(2.5)), c24(in_sgpr(-2.4375)) {}
};

// WENO5-JS on differences (weno5_diff) and its backward: returns V, the value
// minus the centre, and db = hb dV/dd.  V = sum_k w_k q_k / 6 with the
// normalised weights w_k ~ d_k / s_k^2, so dV = sum_k w_k dq_k / 6 -
// 2 sum_k w_k (q_k / 6 - V) ds_k / s_k.
XF_HD double weno5_vjp(const WenoVjpK &K, const double *d, double eps, double hb, double *db) {
    const double h1 = fma(K.h * d[1], d[1], eps), h2 = fma(K.h * d[2], d[2], eps);
    const double z0 = fma(K.a, d[1], d[0]), z1 = fma(K.b, d[2], d[1]), z2 = fma(K.a, d[2], d[3]);
    const double s0 = fma(z0, z0, h1), s1 = fma(z1, z1, h2), s2 = fma(z2, z2, h2);
    const double p0 = s1 * s2, p1 = s0 * s2, p2 = s0 * s1;
    const double v0 = p0 * p0, v1 = K.c6 * (p1 * p1), v2 = K.c3 * (p2 * p2);
    const double D = v0 + v1 + v2, s = p0 * s0, Q = D * s;
    double w0, w1, w2, i0, i1, i2;   // the weights, 1 / s_k
    if (Q < kWideProduct) {
        const double r = rcp_nr(Q), iD = r * s, iS = r * D;
        w0 = v0 * iD;
        w1 = v1 * iD;
        w2 = v2 * iD;
        i0 = iS * p0;
        i1 = iS * p1;
        i2 = iS * p2;
    } else {                         // indicators whose products leave the range
        i0 = rcp_nr(s0);
        i1 = rcp_nr(s1);
        i2 = rcp_nr(s2);
        const double a0 = i0 * i0, a1 = 6.0 * i1 * i1, a2 = 3.0 * i2 * i2, r = rcp_nr(a0 + a1 + a2);
        w0 = a0 * r;
        w1 = a1 * r;
        w2 = a2 * r;
    }
    // candidates minus the centre, times 6
    const double q0 = fma(K.c5, d[1], -2.0 * d[0]), q1 = fma(2.0, d[2], d[1]), q2 = fma(4.0, d[2], -d[3]);
    const double V6 = fma(w2, q2, fma(w1, q1, w0 * q0));
    const double hs = hb * K.sixth;
    const double g0 = hs * w0, g1 = hs * w1, g2 = hs * w2;
    // X_k = -1/2 the cotangent of s_k, t_k = X_k z_k
    const double X0 = g0 * (q0 - V6) * i0, X1 = g1 * (q1 - V6) * i1, X2 = g2 * (q2 - V6) * i2;
    const double t0 = X0 * z0, t1 = X1 * z1, t2 = X2 * z2;
    db[0] = fma(-4.0, t0, -2.0 * g0);
    db[1] = fma(K.c24, d[1] * X0, fma(-4.0, t1, fma(K.c55, t0, fma(K.c5, g0, g1))));
    db[2] = fma(K.c24, d[2] * (X1 + X2), fma(K.c55, t2, fma(K.c25, t1, fma(4.0, g2, 2.0 * g1))));
    db[3] = fma(-4.0, t2, -g2);
    return V6 * K.sixth;
}

// One characteristic field h = W(g+) + W(g-), g+- = wF +- a wU (taken times
// SCALE) and the cotangent hb of h: returns h and the cotangents sF of wF and
// aU of wU.
template <bool CU6, int SCALE>
XF_HD double field_vjp(const WenoVjpK &K, double a, const double *wU, const double *wF, double hb, double *sF,
                       double *aU) {
    if constexpr (CU6) {
        double gp[6], gm[6], pb[6] = {}, mb[6] = {};
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            gp[m] = fma(a, wU[m], wF[m]) * (1.0 / SCALE);
            gm[m] = fma(-a, wU[m], wF[m]) * (1.0 / SCALE);
        }
        const double h = cu6_bwd(gp[0], gp[1], gp[2], gp[3], gp[4], gp[5], hb, pb[0], pb[1], pb[2], pb[3], pb[4], pb[5]) +
                         cu6_bwd(gm[5], gm[4], gm[3], gm[2], gm[1], gm[0], hb, mb[5], mb[4], mb[3], mb[2], mb[1], mb[0]);
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            sF[m] = (pb[m] + mb[m]) * (1.0 / SCALE);
            aU[m] = (pb[m] - mb[m]) * (a / SCALE);
        }
        return h;
    } else {
        constexpr double eps = 0.75e-6 * (SCALE * SCALE);
        const double hs = hb * (1.0 / SCALE);
        double g[5], d[4], db[4], pb[5], h;
#pragma unroll
        for (int k = 0; k < 5; ++k) g[k] = fma(a, wU[k], wF[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = g[k + 1] - g[k];
        h = g[2] + weno5_vjp(K, d, eps, hs, db);
        pb[0] = -db[0];
        pb[1] = db[0] - db[1];
        pb[2] = (db[1] - db[2]) + hs;
        pb[3] = db[2] - db[3];
        pb[4] = db[3];
#pragma unroll
        for (int k = 0; k < 5; ++k) g[k] = fma(-a, wU[5 - k], wF[5 - k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = g[k + 1] - g[k];
        h += g[2] + weno5_vjp(K, d, eps, hs, db);
        // slots 5..1 of the mirrored side: -db0, db0 - db1, db1 - db2 + hs, db2 - db3, db3
        const double m4 = db[0] - db[1], m3 = (db[1] - db[2]) + hs, m2 = db[2] - db[3], m1 = db[3];
        sF[0] = pb[0];
        aU[0] = a * pb[0];
        sF[1] = pb[1] + m1;
        aU[1] = a * (pb[1] - m1);
        sF[2] = pb[2] + m2;
        aU[2] = a * (pb[2] - m2);
        sF[3] = pb[3] + m3;
        aU[3] = a * (pb[3] - m3);
        sF[4] = pb[4] + m4;
        aU[4] = a * (pb[4] - m4);
        sF[5] = -db[0];
        aU[5] = a * db[0];
        return h * (1.0 / SCALE);
    }
}

template <int NS, int DIR, bool CU6, class St, class Bar, class Out>
__device__ __forceinline__ void face_vjp_f64(St st, const ThermoK<double> &th, const Bar &Fb, const Out &out,
                                             const Dissip &ds) {
    constexpr int IM = NS;
    constexpr int IE = NS + 3;
    constexpr int KN = Axes<DIR>::n, K1 = Axes<DIR>::t1, K2 = Axes<DIR>::t2;
    constexpr int IN = NS + KN, I1 = NS + K1, I2 = NS + K2;
    const WenoVjpK K;

    // ================= forward: Roe state and per-cell sums ==================
    const double iL = st.p(3, 2), iR = st.p(3, 3);
    const double qL = iL * rsqrt_nr(iL), qR = iR * rsqrt_nr(iR);
    const double wL = qR * rcp_nr(qL + qR), wR = 1.0 - wL;
    const double aL = wL * iL, aR = wR * iR;
    double ut[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) ut[k] = aL * st.u(IM + k, 2) + aR * st.u(IM + k, 3);
    const double Ht = aL * (st.u(IE, 2) + st.p(1, 2)) + aR * (st.u(IE, 3) + st.p(1, 3));
    const double Tt = wL * st.p(0, 2) + wR * st.p(0, 3);
    double rh[6], un[6], DU[6], DF[6];
    double Gam, S1, Sb, Rb, cvb, ic, ct, aM = 0.0, a0 = 0.0, aP = 0.0, SYF = 0.0;
    const double q2 = ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2], hq = 0.5 * q2;
    const double utn = ut[KN];
    {
        double Se[6], SR[6], cvL = 0.0, cvR = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) rh[m] = Se[m] = SR[m] = 0.0;
#pragma unroll 1
        for (int s = 0; s < NS; ++s) {
            const double es = e_uniform(th, s, Tt), cs = cv_uniform(th, s, Tt), Rs = th.Rs[s];
            double r[6];
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                r[m] = st.u(s, m);
                rh[m] += r[m];
                Se[m] = fma(es, r[m], Se[m]);
                SR[m] = fma(Rs, r[m], SR[m]);
            }
            cvL = fma(cs, r[2], cvL);
            cvR = fma(cs, r[3], cvR);
            SYF = fma(fma(aL, r[2], aR * r[3]), Fb(s), SYF);   // sum_s Y_s Fbar_s
        }
        Rb = fma(aL, SR[2], aR * SR[3]);
        cvb = fma(aL, cvL, aR * cvR);
        S1 = fma(aL, rh[2], aR * rh[3]);
        Sb = fma(aL, Se[2], aR * Se[3]);
        Gam = Rb * rcp_nr(cvb);
        const double c2 = Gam * (Ht - q2) + Gam * (hq * S1 - Sb) + Tt * Rb;
        ic = rsqrt_nr(c2);
        ct = c2 * ic;
        const double ic2 = ic * ic, Gi = Gam * ic2, Ti = Tt * ic2;
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            const double pm = st.p(1, m), cm = st.p(2, m);
            un[m] = st.u(IN, m) * st.p(3, m);
            double t = fma(-ut[0], st.u(IM, m), st.u(IE, m));
            t = fma(-ut[1], st.u(IM + 1, m), t);
            t = fma(-ut[2], st.u(IM + 2, m), t);
            t += fma(hq, rh[m], -Se[m]);
            DU[m] = fma(Gi, t, Ti * SR[m]);
            DF[m] = fma(un[m], DU[m], (Gi * pm) * (un[m] - utn));
            aM = fmax(aM, fabs(un[m] - cm));
            a0 = fmax(a0, fabs(un[m]));
            aP = fmax(aP, fabs(un[m] + cm));
        }
    }
    if (ds.type == kViscRoe) {   // speeds of the Roe state, held fixed like the LLF ones
        aM = fabs(utn - ct);
        a0 = fabs(utn);
        aP = fabs(utn + ct);
    } else if (ds.type == kViscGlf) {
        aM = ds.glf[0];
        a0 = ds.glf[1];
        aP = ds.glf[2];
    }

    XF_PHASE(st);
    // ================= back-projection ======================================
    // F_s = Y_s A + h_s; F_m = u (A + gsum) + c n D + t1 h1 + t2 h2;
    // F_E = H A + u_n c D + u_t1 h1 + u_t2 h2 + sum_s (q^2/2 + e_s - KT R_s) h_s,
    // A = h_- + h_+, D = h_+ - h_-, KT = T~ / Gamma.
    const double FbE = Fb(IE);
    const double Fbm[3] = {Fb(IM), Fb(IM + 1), Fb(IM + 2)};
    const double uF = fma(ut[0], Fbm[0], fma(ut[1], Fbm[1], ut[2] * Fbm[2]));
    const double A_b = fma(Ht, FbE, uF) + SYF, FbN = fma(utn, FbE, Fbm[KN]), D_b = ct * FbN;

    // ================= acoustic pair ========================================
    double un_b[6], DU_b[6], DF_b[6], rh_b[6];
    double A, Dd, ic_b = 0.0, utn_b = 0.0;
    {
        double sFm[6], aUm[6], sFp[6], aUp[6], wU[6], wF[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            const double XU = fma(-utn, rh[m], st.u(IN, m)), XF = fma(un[m], XU, st.p(1, m));
            wU[m] = fma(-ic, XU, DU[m]);
            wF[m] = fma(-ic, XF, DF[m]);
        }
        const double hm = field_vjp<CU6, 4>(K, aM, wU, wF, A_b - D_b, sFm, aUm);
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            wU[m] = fma(2.0, DU[m], -wU[m]);
            wF[m] = fma(2.0, DF[m], -wF[m]);
        }
        const double hp = field_vjp<CU6, 4>(K, aP, wU, wF, A_b + D_b, sFp, aUp);
        A = hm + hp;
        Dd = hp - hm;
        XF_PHASE(st);
        // w = D -+ X / c, X_U = m_n - u~_n rho, X_F = u_n X_U + p
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            DU_b[m] = aUm[m] + aUp[m];
            DF_b[m] = sFm[m] + sFp[m];
            const double dU = aUp[m] - aUm[m], dF = sFp[m] - sFm[m];
            const double XU = fma(-utn, rh[m], st.u(IN, m)), XF = fma(un[m], XU, st.p(1, m));
            ic_b = fma(XU, dU, fma(XF, dF, ic_b));
            const double XFb = ic * dF, xb = fma(un[m], XFb, ic * dU);
            un_b[m] = XU * XFb;
            rh_b[m] = -utn * xb;
            utn_b = fma(-rh[m], xb, utn_b);
            out.u(IN, m, xb);
            out.p(kSinkP, m, XFb);
        }
    }
    double ut_b[3];
    ut_b[KN] = fma(ct * Dd, FbE, utn_b);
    double ct_b = Dd * FbN;
    double Ht_b = A * FbE;

    // ================= tangential pair ======================================
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        XF_PHASE(st);
        const int I = a == 0 ? I1 : I2, Kk = a == 0 ? K1 : K2;
        const double uta = ut[Kk];
        double wU[6], wF[6], sF[6], aU[6];
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            wU[m] = fma(-uta, rh[m], st.u(I, m));
            wF[m] = un[m] * wU[m];
        }
        const double ha = field_vjp<CU6, 2>(K, a0, wU, wF, fma(uta, FbE, Fbm[Kk]), sF, aU);
        double ub = ha * FbE;
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            const double wb = fma(un[m], sF[m], aU[m]);
            un_b[m] = fma(wU[m], sF[m], un_b[m]);
            rh_b[m] = fma(-uta, wb, rh_b[m]);
            ub = fma(-rh[m], wb, ub);
            out.u(I, m, wb);
        }
        ut_b[Kk] = ub;
    }

    // ================= species fields =======================================
    const double iGam = cvb * rcp_nr(Rb), KT = Tt * iGam;
    double gsum = 0.0, CH = 0.0, RH = 0.0;   // sums of h_s, cv_s h_s, R_s h_s
    double aL_b = 0.0, aR_b = 0.0;
    {
        const double hb0 = fma(hq, FbE, uF);
#pragma unroll 1
        for (int s = 0; s < NS; ++s) {
            XF_PHASE(st);
            const double Fbs = Fb(s), Rs = th.Rs[s];
            double r[6], wU[6], wF[6], sF[6], aU[6];
#pragma unroll
            for (int m = 0; m < 6; ++m) r[m] = st.u(s, m);
            const double Ys = fma(aL, r[2], aR * r[3]);
            const double hsb = fma(fma(-KT, Rs, e_uniform(th, s, Tt)), FbE, hb0 + Fbs);
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                wU[m] = fma(-Ys, DU[m], r[m]);
                wF[m] = fma(-Ys, DF[m], r[m] * un[m]);
            }
            const double hs = field_vjp<CU6, 2>(K, a0, wU, wF, hsb, sF, aU);
            gsum += hs;
            CH = fma(cv_uniform(th, s, Tt), hs, CH);
            RH = fma(Rs, hs, RH);
            double yb = A * Fbs;   // cotangent of Y_s
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                un_b[m] = fma(r[m], sF[m], un_b[m]);
                yb = fma(-DU[m], aU[m], fma(-DF[m], sF[m], yb));
                DU_b[m] = fma(-Ys, aU[m], DU_b[m]);
                DF_b[m] = fma(-Ys, sF[m], DF_b[m]);
            }
#pragma unroll
            for (int m = 0; m < 6; ++m) {
                double v = fma(un[m], sF[m], aU[m]);
                if (m == 2) v = fma(aL, yb, v);
                if (m == 3) v = fma(aR, yb, v);
                out.u(s, m, v);
            }
            aL_b = fma(r[2], yb, aL_b);
            aR_b = fma(r[3], yb, aR_b);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) ut_b[k] = fma(A + gsum, Fbm[k], ut_b[k]);
    double hq_b = gsum * FbE;
    const double KT_b = -FbE * RH;
    double Tt_b = fma(CH, FbE, iGam * KT_b);
    double Gam_b = -KT * iGam * KT_b;

    // ================= per-cell projections =================================
    const double ic2 = ic * ic, Gi = Gam * ic2, Ti = Tt * ic2;
    double Gi_b = 0.0, DD = 0.0;   // DD = sum_m DU DUbar
#pragma unroll
    for (int m = 0; m < 6; ++m) {
        XF_PHASE(st);
        const double pm = st.p(1, m), du = un[m] - utn;
        const double db = fma(un[m], DF_b[m], DU_b[m]);     // all of DU's cotangent
        DU_b[m] = db;
        DD = fma(DU[m], db, DD);
        const double pF = pm * DF_b[m];
        Gi_b = fma(du, pF, Gi_b);
        out.p(kSinkP, m, Gi * du * DF_b[m]);
        const double ub = fma(DU[m], DF_b[m], fma(Gi, pF, un_b[m]));   // u_n = m_n / rho
        ut_b[KN] = fma(-Gi, pF, ut_b[KN]);
        const double tb = Gi * db;
        hq_b = fma(rh[m], tb, hq_b);
        const double rinv = st.p(3, m), ur = rinv * ub;
        rh_b[m] = fma(hq, tb, fma(-un[m], ur, rh_b[m]));
        out.p(kSinkRho, m, rh_b[m]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            ut_b[k] = fma(-st.u(IM + k, m), tb, ut_b[k]);
            out.u(IM + k, m, k == KN ? fma(-ut[k], tb, ur) : -ut[k] * tb);
        }
        out.u(IE, m, tb);
    }
    // sums over species of R_s and cv_s times sum_m rho_s DUbar
    double SX = 0.0, CX = 0.0;
#pragma unroll 1
    for (int s = 0; s < NS; ++s) {
        double x = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) x = fma(st.u(s, m), DU_b[m], x);
        SX = fma(th.Rs[s], x, SX);
        CX = fma(cv_uniform(th, s, Tt), x, CX);
    }
    // DU = Gi t + Ti S: sum t DUbar = (sum DU DUbar - Ti sum S DUbar) / Gi
    const double c2 = ct * ct;
    Gi_b = fma(fma(-Ti, SX, DD), c2 * iGam, Gi_b);
    Tt_b = fma(ic2, SX, fma(-Gi, CX, Tt_b));
    Gam_b = fma(ic2, Gi_b, Gam_b);
    const double ic2_b = fma(Gam, Gi_b, Tt * SX);

    XF_PHASE(st);
    // ================= Roe state: c, Gamma, averages =========================
    // c = c2 / sqrt(c2), 1 / c and 1 / c^2 from c2
    const double c2_b = 0.5 * ic * (ct_b - ic2 * ic_b) - ic2 * ic2 * ic2_b;
    Gam_b = fma(Ht - q2 + (hq * S1 - Sb), c2_b, Gam_b);
    Ht_b = fma(Gam, c2_b, Ht_b);
    hq_b = fma(Gam * S1, c2_b, hq_b);
    const double q2_b = fma(0.5, hq_b, -Gam * c2_b);
    Tt_b = fma(fma(-Gam, cvb, Rb), c2_b, Tt_b);
    const double icv = rcp_nr(cvb), Rb_b = Gam_b * icv, cvb_b = -Gam * Rb_b;
    const double kR = fma(Tt, c2_b, Rb_b), kc = Gam * c2_b;
#pragma unroll 1
    for (int s = 0; s < NS; ++s) {
        XF_PHASE(st);
        const double rL = st.u(s, 2), rR = st.u(s, 3), Rs = th.Rs[s];
        const double es = e_uniform(th, s, Tt);
        const double T = Tt;
        const double dcv = fma(T, fma(T, fma(T, 4.0 * th.cv[s][4], 3.0 * th.cv[s][3]), 2.0 * th.cv[s][2]), th.cv[s][1]);
        const double yb = fma(cv_uniform(th, s, Tt), cvb_b, fma(Rs, kR, kc * (hq - es)));
        Tt_b = fma(fma(aL, rL, aR * rR) * dcv, cvb_b, Tt_b);
        const double k = Gi * fma(KT, Rs, -es);
#pragma unroll
        for (int m = 0; m < 6; ++m) {
            double v = k * DU_b[m];
            if (m == 2) v = fma(aL, yb, v);
            if (m == 3) v = fma(aR, yb, v);
            out.u(s, m, v);
        }
        aL_b = fma(rL, yb, aL_b);
        aR_b = fma(rR, yb, aR_b);
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) ut_b[k] = fma(2.0 * ut[k], q2_b, ut_b[k]);

    XF_PHASE(st);
    aL_b = fma(st.u(IE, 2) + st.p(1, 2), Ht_b, aL_b);
    aR_b = fma(st.u(IE, 3) + st.p(1, 3), Ht_b, aR_b);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        aL_b = fma(st.u(IM + k, 2), ut_b[k], aL_b);
        aR_b = fma(st.u(IM + k, 3), ut_b[k], aR_b);
        out.u(IM + k, 2, aL * ut_b[k]);
        out.u(IM + k, 3, aR * ut_b[k]);
    }
    out.u(IE, 2, aL * Ht_b);
    out.u(IE, 3, aR * Ht_b);
    out.p(kSinkP, 2, aL * Ht_b);
    out.p(kSinkP, 3, aR * Ht_b);
    out.p(kSinkT, 2, wL * Tt_b);
    out.p(kSinkT, 3, wR * Tt_b);
    // aL = wL / rho_L, aR = wR / rho_R, T~ = wL T_L + wR T_R, and
    // dwL = wL wR (drho_L / rho_L - drho_R / rho_R) / 2
    const double jL = st.p(3, 2), jR = st.p(3, 3);
    const double w_b = (st.p(0, 2) * Tt_b + jL * aL_b) - (st.p(0, 3) * Tt_b + jR * aR_b);
    const double ww = 0.5 * wL * wR * w_b;
    out.p(kSinkRho, 2, jL * (ww - aL * aL_b));
    out.p(kSinkRho, 3, -jR * (ww + aR * aR_b));
}

}  // namespace xf
