// xf_face64.hpp -- one face of the convective flux in FP64 (the steps and the
// eigenvectors are those at the top of xf_face.hpp; the mixed path's FP32
// faces keep the forms there).
//
// What bounds it: in the sweeps that wait least for memory vector instructions
// issue on two thirds of the SIMDs' cycles (z, which only stores, 67 %; y, which adds
// to the sum, 57 %; four fifths with the plain forms), so the face is written for its
// instruction count.  Every form below is equal to the plain one in exact arithmetic:
//   * the split values g+- = (wF +- alpha wU)/2 are taken times two (times
//     four in the acoustic fields, where w = DF/2 -+ c XF/(2 c^2) halves once
//     more) and eps with them; the fluxes leave the face times kFluxScale;
//   * the reconstructions work on first differences: candidates relative to
//     the centre cell, and smoothness indicators as sums of two squares with
//     shared terms, 12 beta / 16 = (d0 - 11/8 d1)^2 + 39/64 d1^2,
//     (d1 - 5/8 d2)^2 + 39/64 d2^2 and (d3 - 11/8 d2)^2 + 39/64 d2^2
//     (30 operations per WENO5 side where the plain form takes 45);
//   * g+- of a species is r (u_n +- a0) - Y (DF +- a0 DU): the brackets are
//     formed once per face, as differences for the second;
//   * sum_s chi_s rho_s = Gamma (q^2/2 rho - sum_s e_s rho_s) + T~ sum_s R_s
//     rho_s, so the species thermo is evaluated once for the Roe state and
//     the six cells together, and n.F_m - u_n F_rho = u_n (n.m - u~_n rho) + p.
// Vector instructions per nine-species face in a y/z tile: 3198 in the plain
// forms, 2420 with those above, 2128 with the constants and the uniform
// polynomial coefficients in scalar registers (in_sgpr, fma_uniform) and the
// exchange's lane index formed once.  z sweep at 256^3, nine species: 1.95 ->
// 1.60 -> 1.52 ms.
#pragma once

#include "xf_face.hpp"

namespace xf {

// Fluxes of face_flux_f64 are this multiple of the true ones.
constexpr double kFluxScale = 2.0;

// 1 / sqrt(x) of a positive normal number: the hardware estimate and two
// Newton steps y <- y + y (1 - x y^2) / 2.
XF_HD double rsqrt_nr(double x) {
#ifdef __HIP_DEVICE_COMPILE__
    double y = __builtin_amdgcn_rsq(x);
#else
    double y = 1.0 / sqrt(x);
#endif
    double e = fma(-x * y, y, 1.0);
    y = fma(0.5 * y, e, y);
    e = fma(-x * y, y, 1.0);
    return fma(0.5 * y, e, y);
}

// A constant held in scalar registers: left to itself the compiler takes most
// FP64 constants as literals, which only the two-operand multiply-add accepts,
// and then copies the addend first wherever it is needed again.
XF_HD double in_sgpr(double v) {
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+s"(v));
#endif
    return v;
}
// a * b + c with c uniform, as one instruction (the compiler copies a uniform
// addend into the destination's registers first)
XF_HD double fma_uniform(double a, double b, double c) {
#ifdef __HIP_DEVICE_COMPILE__
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
#else
    return fma(a, b, c);
#endif
}
// e_s(T) and C_v,s(T) of a species the whole wave works on
XF_HD double e_uniform(const ThermoK<double> &th, int s, double T) {
    double v = fma(T, th.e[s][5], th.e[s][4]);
#pragma unroll
    for (int k = 3; k >= 0; --k) v = fma_uniform(v, T, th.e[s][k]);
    return v;
}
XF_HD double cv_uniform(const ThermoK<double> &th, int s, double T) {
    double v = fma(T, th.cv[s][4], th.cv[s][3]);
#pragma unroll
    for (int k = 2; k >= 0; --k) v = fma_uniform(v, T, th.cv[s][k]);
    return v;
}

// Constants of the WENO5 weights.
struct WenoK {
    double a, b, h, c3, c5, c6, c12, sixth;
    XF_HD WenoK()
        : a(in_sgpr(-1.375)), b(in_sgpr(-0.625)), h(in_sgpr(0.609375)), c3(in_sgpr(3.0)), c5(in_sgpr(5.0)),
          c6(in_sgpr(6.0)), c12(in_sgpr(12.0)), sixth(in_sgpr(1.0 / 6.0)) {}
};

// Differences per side, the cells they span, and the fluxes' guard: products
// of the weights' denominators past kWideProduct (never reached by fluxes at
// SI scales) are taken after both sides are scaled by powers of two.
template <int REC>
constexpr int recon_diffs() { return REC == kReconWeno7 ? 6 : REC == kReconCu6 ? 5 : 4; }
constexpr double kWideProduct = 1e280;

// WENO5-JS from the first differences d0..d3 of the five point values (centre
// between d1 and d2): the value is centre + N / (6 D).  eps is 1e-6 * 12/16
// times the square of the values' scale.
XF_HD void weno5_diff(const WenoK &K, const double *d, double eps, double &N, double &D) {
    const double h1 = fma(K.h * d[1], d[1], eps), h2 = fma(K.h * d[2], d[2], eps);
    const double z0 = fma(K.a, d[1], d[0]), z1 = fma(K.b, d[2], d[1]), z2 = fma(K.a, d[2], d[3]);
    const double s0 = fma(z0, z0, h1), s1 = fma(z1, z1, h2), s2 = fma(z2, z2, h2);
    const double p0 = s1 * s2, p1 = s0 * s2, p2 = s0 * s1;
    const double w0 = p0 * p0, w1 = p1 * p1, w2 = p2 * p2;
    // candidates minus the centre, times 6 and the linear weights 1, 6, 3
    const double m = K.c12 * d[2];
    const double q0 = fma(K.c5, d[1], -2.0 * d[0]), q1 = fma(K.c6, d[1], m), q2 = fma(-K.c3, d[3], m);
    N = fma(w2, q2, fma(w1, q1, w0 * q0));
    D = fma(K.c3, w2, fma(K.c6, w1, w0));
}

// WENO-CU6 from d0..d4 (forms of weno_cu6; the indicators times 12/16):
// centre + N / (6 D).
XF_HD void cu6_diff(const double *d, double eps, double &N, double &D) {
    const double h1 = 0.609375 * d[1] * d[1], h2 = 0.609375 * d[2] * d[2];
    const double z0 = fma(-1.375, d[1], d[0]), z1 = fma(-0.625, d[2], d[1]), z2 = fma(-1.375, d[2], d[3]);
    const double b0 = fma(z0, z0, h1), b1 = fma(z1, z1, h2), b2 = fma(z2, z2, h2);
    const double y0 = fma(0.4518745009732172, d[4],
                          fma(-2.2318538224071762, d[3],
                              fma(4.137755308541131, d[2], fma(-3.3800293620919937, d[1], d[0]))));
    const double y1 = fma(-0.2835945203123665, d[4], fma(1.2398246217680282, d[3], fma(-1.8788632502196132, d[2], d[1])));
    const double y2 = fma(0.22441845180562248, d[4], fma(-0.8641384480158466, d[3], d[2]));
    const double y3 = fma(-0.3841978250666033, d[4], d[3]);
    const double b6 = fma(0.75 * 2.2468501984126985 * y0, y0,
                          fma(0.75 * 3.6320275079835525 * y1, y1,
                              fma(0.75 * 4.213886137822353 * y2, y2,
                                  fma(0.75 * 1.0316113515772065 * y3, y3, 0.75 * 0.03897812227306876 * d[4] * d[4]))));
    const double tau = fma(-1.0 / 6.0, fma(4.0, b1, b0 + b2), b6);
    const double e0 = b0 + eps, e1 = b1 + eps, e2 = b2 + eps, e3 = b6 + eps;
    const double p01 = e0 * e1, p23 = e2 * e3;
    // weights times 20 prod e; linear weights 1, 9, 9, 1
    const double w0 = fma(20.0, e0, tau) * (e1 * p23), w1 = fma(20.0, e1, tau) * (e0 * p23);
    const double w2 = fma(20.0, e2, tau) * (p01 * e3), w3 = fma(20.0, e3, tau) * (p01 * e2);
    // candidates minus the centre, times 6; the middle two with their 9
    const double m = 6.0 * d[2];
    const double q0 = fma(5.0, d[1], -2.0 * d[0]), q1 = fma(9.0, d[1], 3.0 * m), q2 = fma(-9.0, d[3], 6.0 * m);
    const double q3 = fma(2.0, d[4], fma(-5.0, d[3], m));
    N = fma(w3, q3, fma(w2, q2, fma(w1, q1, w0 * q0)));
    D = fma(9.0, w1 + w2, w0 + w3);
}

// WENO7-JS from d0..d5 (forms of weno7_parts; weights after scaling the four
// (eps + beta) by one power of two): the value minus the centre.
XF_HD double weno7_diff(const double *d, double eps) {
    double e[4];
    {
        const double z0 = fma(927.0 / 547.0, d[2], fma(-1394.0 / 547.0, d[1], d[0])), z1 = fma(-3167.0 / 2126.0, d[2], d[1]);
        e[0] = fma(547.0 / 240.0 * z0, z0, fma(1063.0 / 1641.0 * z1, z1, fma(10153.0 / 12756.0 * d[2], d[2], eps)));
    }
    {
        const double z0 = fma(247.0 / 267.0, d[3], fma(-554.0 / 267.0, d[2], d[1])), z1 = fma(-1345.0 / 2126.0, d[3], d[2]);
        e[1] = fma(89.0 / 80.0 * z0, z0, fma(1063.0 / 801.0 * z1, z1, fma(10153.0 / 12756.0 * d[3], d[3], eps)));
    }
    {
        const double z0 = fma(247.0 / 547.0, d[4], fma(-714.0 / 547.0, d[3], d[2])), z1 = fma(-3167.0 / 7330.0, d[4], d[3]);
        e[2] = fma(547.0 / 240.0 * z0, z0, fma(3665.0 / 1641.0 * z1, z1, fma(10153.0 / 43980.0 * d[4], d[4], eps)));
    }
    {
        const double z0 = fma(927.0 / 2107.0, d[5], fma(-2594.0 / 2107.0, d[4], d[3])), z1 = fma(-13313.0 / 27098.0, d[5], d[4]);
        e[3] = fma(2107.0 / 240.0 * z0, z0, fma(13549.0 / 6321.0 * z1, z1, fma(10153.0 / 162588.0 * d[5], d[5], eps)));
    }
    int ex;
    frexp(fmax(fmax(e[0], e[1]), fmax(e[2], e[3])), &ex);
    const double f0 = ldexp(e[0], -ex), f1 = ldexp(e[1], -ex), f2 = ldexp(e[2], -ex), f3 = ldexp(e[3], -ex);
    const double s0 = f0 * f0, s1 = f1 * f1, s2 = f2 * f2, s3 = f3 * f3;
    const double p01 = s0 * s1, p23 = s2 * s3;
    const double w0 = s1 * p23, w1 = s0 * p23, w2 = p01 * s3, w3 = p01 * s2;
    // candidates minus the centre, times 12 and the linear weights 1, 12, 18, 4
    const double q0 = fma(13.0, d[2], fma(-10.0, d[1], 3.0 * d[0])), q1 = 12.0 * fma(3.0, d[3], fma(4.0, d[2], -d[1]));
    const double q2 = 18.0 * (fma(6.0, d[3], d[2]) - d[4]), q3 = 4.0 * fma(9.0, d[3], fma(-4.0, d[4], d[5]));
    const double N = fma(w3, q3, fma(w2, q2, fma(w1, q1, w0 * q0)));
    const double D = fma(4.0, w3, fma(18.0, w2, fma(12.0, w1, w0)));
    return N / (12.0 * D);
}

// Both sides of one characteristic field, from the centre values cp, cm (g+
// of cell i, g- of cell i+1) and the differences p (along g+) and m (along
// the mirrored g-); SCALE that of the values.  One reciprocal for the two.
template <int REC, int SCALE>
XF_HD double recon_sum(const WenoK &K, double cp, const double *p, double cm, const double *m) {
    if constexpr (REC == kReconWeno7) {
        constexpr double eps = 1e-6 * (SCALE * SCALE);
        return (cp + cm) + (weno7_diff(p, eps) + weno7_diff(m, eps));
    } else {
        constexpr double eps = 0.75e-6 * (SCALE * SCALE);
        double Np, Dp, Nm, Dm;
        if constexpr (REC == kReconCu6) {
            cu6_diff(p, eps, Np, Dp);
            cu6_diff(m, eps, Nm, Dm);
        } else {
            weno5_diff(K, p, eps, Np, Dp);
            weno5_diff(K, m, eps, Nm, Dm);
        }
        double P = Dp * Dm;
        if (!(P < kWideProduct)) {
            int ep, em;
            frexp(Dp, &ep);
            frexp(Dm, &em);
            Np = ldexp(Np, -ep);
            Dp = ldexp(Dp, -ep);
            Nm = ldexp(Nm, -em);
            Dm = ldexp(Dm, -em);
            P = Dp * Dm;
        }
        return fma(fma(Nm, Dp, Np * Dm) * rcp_nr(P), K.sixth, cp + cm);
    }
}

// The numerical flux at one face, every component handed to out(q, v) times
// kFluxScale as soon as it is final (species first, then momentum and
// energy): out.start() asks for what component 0 needs from memory,
// out.next<SLOT>(q) for component q a whole species ahead of out.put<SLOT>(q,
// v), SLOT = q mod 2, out.rest() for the last three.  Other parameters as
// face_flux_to of xf_face.hpp.  The species loops run as loops, the last one
// two species at a time (so that a load held for the next species stays in
// its registers: moving it would wait for it); fully unrolled, the
// per-species values would need twice the registers.
template <int NS, int DIR, int SPD, int REC, class St, class Out>
XF_HD void face_flux_f64(const St &st, const ThermoK<double> &th, Out &&out, unsigned &flags, const Dissip &ds) {
    constexpr int RAD = stencil_radius(REC);
    constexpr int W = 2 * RAD;       // stencil cells
    constexpr int CL = RAD - 1;      // slot of cell i (left of the face)
    constexpr int CR = RAD;          // slot of cell i+1
    constexpr int ND = recon_diffs<REC>();
    constexpr int IM = NS;
    constexpr int IE = NS + 3;
    constexpr int IN = NS + Axes<DIR>::n;
    constexpr int I1 = NS + Axes<DIR>::t1;
    constexpr int I2 = NS + Axes<DIR>::t2;

    const WenoK K;
    // ---- Roe weights, averaged velocity, enthalpy and temperature ---------
    // sqrt(rho_L) / (sqrt(rho_L) + sqrt(rho_R)) from the cells' 1 / rho
    const double iL = st.p(3, CL), iR = st.p(3, CR);
    const double qL = iL * rsqrt_nr(iL), qR = iR * rsqrt_nr(iR);
    const double wL = qR * rcp_nr(qL + qR), wR = 1.0 - wL;
    const double aL = wL * iL, aR = wR * iR;   // weights on conservative values
    double ut[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) ut[k] = aL * st.u(IM + k, CL) + aR * st.u(IM + k, CR);
    const double Ht = aL * (st.u(IE, CL) + st.p(1, CL)) + aR * (st.u(IE, CR) + st.p(1, CR));
    const double Tt = wL * st.p(0, CL) + wR * st.p(0, CR);

    // ---- sum_s rho_s, sum_s e_s rho_s and sum_s R_s rho_s of every cell ----
    double rh[W], Se[W], SR[W], cvL = 0.0, cvR = 0.0;
#pragma unroll
    for (int m = 0; m < W; ++m) rh[m] = Se[m] = SR[m] = 0.0;
#pragma unroll 1
    for (int s = 0; s < NS; ++s) {
        const double es = e_uniform(th, s, Tt), cs = cv_uniform(th, s, Tt), Rs = th.Rs[s];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            const double r = st.u(s, m);
            rh[m] += r;
            Se[m] = fma(es, r, Se[m]);
            SR[m] = fma(Rs, r, SR[m]);
            if (m == CL) cvL = fma(cs, r, cvL);
            if (m == CR) cvR = fma(cs, r, cvR);
        }
    }
    // ---- Roe state: Gamma = R / C_v, c^2 = sum_s Y_s chi_s + Gamma (H - q^2)
    const double Rb = fma(aL, SR[CL], aR * SR[CR]), cvb = fma(aL, cvL, aR * cvR);
    const double Gam = Rb * rcp_nr(cvb), KT = Tt * (cvb * rcp_nr(Rb));   // KT = T~ / Gamma
    const double q2 = ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2];
    const double S1 = fma(aL, rh[CL], aR * rh[CR]), Sb = fma(aL, Se[CL], aR * Se[CR]);
    const double hq = 0.5 * q2;
    const double c2 = Gam * (Ht - q2) + Gam * (hq * S1 - Sb) + Tt * Rb;
    if (!(c2 > 0.0)) flags |= XF_FLAG_C2;
    const double ic = rsqrt_nr(c2);       // 1 / c
    const double ct = c2 * ic, ic2 = ic * ic;
    const double utn = ut[Axes<DIR>::n], ut1 = ut[Axes<DIR>::t1], ut2 = ut[Axes<DIR>::t2];

    XF_FENCE();
    // ---- per-cell scalars: u_n, DU = dp(U) / c^2, DF = dp(F) / c^2, speeds
    double un[W], DU[W], DF[W];
    double aM = 0.0, a0 = 0.0, aP = 0.0;
    {
        const double Gi = Gam * ic2, Ti = Tt * ic2;
#pragma unroll
        for (int m = 0; m < W; ++m) {
            const double pm = st.p(1, m), cm = st.p(2, m);
            const double unm = st.u(IN, m) * st.p(3, m);
            double t = fma(-ut[0], st.u(IM, m), st.u(IE, m));
            t = fma(-ut[1], st.u(IM + 1, m), t);
            t = fma(-ut[2], st.u(IM + 2, m), t);
            t += fma(hq, rh[m], -Se[m]);
            un[m] = unm;
            DU[m] = fma(Gi, t, Ti * SR[m]);
            DF[m] = fma(unm, DU[m], (Gi * pm) * (unm - utn));
            if constexpr (SPD == kViscLlf) {
                aM = fmax(aM, fabs(unm - cm));
                a0 = fmax(a0, fabs(unm));
                aP = fmax(aP, fabs(unm + cm));
            } else {
                (void)cm;
            }
        }
    }
    if constexpr (SPD == kViscRoe) {
        aM = fabs(utn - ct);
        a0 = fabs(utn);
        aP = fabs(utn + ct);
    } else if constexpr (SPD == kViscGlf) {
        aM = ds.glf[0];
        a0 = ds.glf[1];
        aP = ds.glf[2];
    } else if constexpr (SPD == kViscFrozen) {
        aM = ds.alpha[ds.fidx];
        a0 = ds.alpha[ds.astride + ds.fidx];
        aP = ds.alpha[2 * ds.astride + ds.fidx];
    }

    XF_FENCE();
    // one field from its split values: wF + a wU of slots 0..ND, and
    // wF - a wU of the mirrored slots W-1..W-1-ND
    auto field = [&](auto scale, const double *wU, const double *wF, double a) {
        double p[ND], m[ND];
        double g = fma(a, wU[0], wF[0]), cp = g;
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const double gn = fma(a, wU[k + 1], wF[k + 1]);
            p[k] = gn - g;
            g = gn;
            if (k + 1 == CL) cp = g;
        }
        g = fma(-a, wU[W - 1], wF[W - 1]);
        double cm = g;
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const double gn = fma(-a, wU[W - 2 - k], wF[W - 2 - k]);
            m[k] = gn - g;
            g = gn;
            if (k + 1 == CL) cm = g;
        }
        return recon_sum<REC, decltype(scale)::value>(K, cp, p, cm, m);
    };
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;

    // ---- acoustic pair (times four): w = DU -+ X / c ------------------------
    double hm, hp;
    {
        double wU[W], wF[W];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            const double XU = fma(-utn, rh[m], st.u(IN, m)), XF = fma(un[m], XU, st.p(1, m));
            wU[m] = fma(-ic, XU, DU[m]);
            wF[m] = fma(-ic, XF, DF[m]);
        }
        hm = field(Four{}, wU, wF, aM);
        // D + X / c as 2 D - (D - X / c): X need not be held
#pragma unroll
        for (int m = 0; m < W; ++m) {
            wU[m] = fma(2.0, DU[m], -wU[m]);
            wF[m] = fma(2.0, DF[m], -wF[m]);
        }
        hp = field(Four{}, wU, wF, aP);
    }
    const double Asum = 0.5 * (hm + hp), Dif = 0.5 * (hp - hm);

    XF_FENCE();
    // ---- tangential pair (times two) ----------------------------------------
    double h1, h2;
    {
        double wU[W], wF[W];
#pragma unroll
        for (int m = 0; m < W; ++m) {
            wU[m] = fma(-ut1, rh[m], st.u(I1, m));
            wF[m] = un[m] * wU[m];
        }
        h1 = field(Two{}, wU, wF, a0);
#pragma unroll
        for (int m = 0; m < W; ++m) {
            wU[m] = fma(-ut2, rh[m], st.u(I2, m));
            wF[m] = un[m] * wU[m];
        }
        h2 = field(Two{}, wU, wF, a0);
    }

    // ---- species fields (times two), back-projected as they come -------------
    // g+ = r lp - Y DP with lp = u_n + a0, DP = DF + a0 DU; g- mirrored
    double lp[ND + 1], lm[ND + 1], dP[ND], dM[ND], DPc, DMc;
    {
        double a = fma(a0, DU[0], DF[0]), b = fma(-a0, DU[W - 1], DF[W - 1]);
        DPc = a;
        DMc = b;
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const double an = fma(a0, DU[k + 1], DF[k + 1]), bn = fma(-a0, DU[W - 2 - k], DF[W - 2 - k]);
            dP[k] = an - a;
            dM[k] = bn - b;
            a = an;
            b = bn;
            if (k + 1 == CL) {
                DPc = a;
                DMc = b;
            }
        }
#pragma unroll
        for (int k = 0; k <= ND; ++k) {
            lp[k] = un[k] + a0;
            lm[k] = un[W - 1 - k] - a0;
        }
    }
    double gsum = 0.0, gE = 0.0;
    out.start();
    auto species = [&](int s, auto slot) {
        constexpr int SLOT = decltype(slot)::value;
        XF_FENCE();
        out.template next<1 - SLOT>(s + 1);
        double r[W];
#pragma unroll
        for (int m = 0; m < W; ++m) r[m] = st.u(s, m);
        const double Ys = aL * r[CL] + aR * r[CR];
        // (q^2 - chi_s / Gamma) - q^2 / 2
        const double ts = fma(-KT, th.Rs[s], e_uniform(th, s, Tt));
        double p[ND], m[ND], cp = 0.0, cm = 0.0;
        double tp = r[0] * lp[0], tm = r[W - 1] * lm[0];
#pragma unroll
        for (int k = 0; k < ND; ++k) {
            const double np = r[k + 1] * lp[k + 1], nm = r[W - 2 - k] * lm[k + 1];
            p[k] = fma(-Ys, dP[k], np - tp);
            m[k] = fma(-Ys, dM[k], nm - tm);
            tp = np;
            tm = nm;
            if (k + 1 == CL) {
                cp = fma(-Ys, DPc, tp);
                cm = fma(-Ys, DMc, tm);
            }
        }
        const double hs = recon_sum<REC, 2>(K, cp, p, cm, m);
        out.template put<SLOT>(s, Ys * Asum + hs);
        gsum += hs;
        gE = fma(ts, hs, gE);
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    // the count is hidden from the compiler: a loop of one turn (two and three
    // species) would be taken apart and its pieces held in registers
    int ns = NS > 1 ? NS : 0;
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(ns));
#endif
    if constexpr (NS > 1)
#pragma unroll 1
    for (int s = 0; s + 1 < ns; s += 2) {
        species(s, Even{});
        species(s + 1, Odd{});
    }
    if constexpr (NS % 2) species(NS - 1, Even{});

    // ---- momentum and energy of F^ = R h ------------------------------------
    out.rest();
    double Fm[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) Fm[k] = ut[k] * (Asum + gsum);
    Fm[Axes<DIR>::n] += ct * Dif;
    Fm[Axes<DIR>::t1] += h1;
    Fm[Axes<DIR>::t2] += h2;
    out.template put<NS % 2>(IM + 0, Fm[0]);
    out.template put<2>(IM + 1, Fm[1]);
    out.template put<3>(IM + 2, Fm[2]);
    out.template put<4>(IE, Ht * Asum + utn * ct * Dif + ut1 * h1 + ut2 * h2 + (hq * gsum + gE));
}

// The face of a sweep in its arithmetic type, and the factor that turns its
// fluxes into the true ones.
template <int NS, typename R, int DIR, int SPD, int REC, class St, class Out>
__device__ __forceinline__ void sweep_face(const St &st, const ThermoK<R> &th, Out &&out, unsigned &flags,
                                           const Dissip &ds) {
    if constexpr (sizeof(R) == 8)
        face_flux_f64<NS, DIR, SPD, REC>(st, th, out, flags, ds);
    else
        face_flux_to<NS, R, DIR, SPD, REC>(st, th, out, flags, ds);
}
template <typename R>
constexpr R flux_unit() { return sizeof(R) == 8 ? R(1.0 / kFluxScale) : R(1); }

}  // namespace xf
