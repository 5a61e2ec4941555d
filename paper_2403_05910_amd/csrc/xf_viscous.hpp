// xf_viscous.hpp -- viscous and diffusive fluxes F_v of Eq. 2 (Eq. 3-6) with
// the fitted transport of Eq. 29, the mixing rule of Eq. 22 and the
// effective diffusion coefficients of Eq. 26; fourth order, FP64.
//
// Per cell (k_transport): mole fractions, mu_s, kappa_s and 1/D_st from the
// fits, mu_bar and kappa_bar by Eq. 22, D_sm by Eq. 26 (mole fractions
// floored at X_t + 1e-12 inside its sums, which keeps a pure species
// finite), and the velocity.  Per face (k_visc_x, k_visc_tile): the point
// value of F_v = (-J_s, tau . n, tau . u . n - q_c - q_d) from the four cells
// i-1..i+2 across the face: face values (-f0 + 9 f1 + 9 f2 - f3)/16, normal
// derivatives (f0 - 27 f1 + 27 f2 - f3)/(24 dx), tangential derivatives
// interpolated from the cell-centred (1, -8, 8, -1)/(12 dy) differences;
// J_s = -rho (D_sm dY_s - Y_s sum_j D_jm dY_j) (Eq. 6 with the correction
// that makes the fluxes sum to zero).  The residual of cell i is the
// difference of the numerical fluxes F^_{i+1/2} = (-F_{i-1/2} + 26 F_{i+1/2}
// - F_{i+3/2})/24, i.e. the staggered fourth-order difference of the point
// fluxes (a plain difference of point fluxes is second order).
#pragma once

#include "xf_reaction.hpp"

namespace xf {

// ---------------------------------------------------------------------------
// transport pass
// ---------------------------------------------------------------------------
// What bounds it: vector instructions (54 exponentials, 2 N^2 mixing terms
// and 3 N divisions per cell at nine species).  The exponentials are the
// reaction kernel's (rx_exp), with their constants in scalar registers; a_s of
// a fit f is taken through its root, sqrt(a_s) = exp(f / 2), which the mixing
// rule needs anyway; divisions are by reciprocals of positive normal numbers.
// With libm's exp, sqrt and IEEE divisions (3837 vector instructions a wave,
// now 2918) this pass and the velocity gradient took 488 us at nine
// species and 2.9 M cells, now 400 us.
template <int NS>
__global__ __launch_bounds__(256) void k_transport(const double *__restrict__ U, const double *__restrict__ P,
                                                   double *__restrict__ Q, Geo g,
                                                   const TransportK *__restrict__ tkp) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= g.cells) return;
    const cptr<TransportK> tk = (cptr<TransportK>)tkp;
    const long long C = g.cells;
    const double rinv = P[3 * C + idx], T = P[idx], p = P[C + idx];
    const cptr<double> ec = exp_table();
    double X[NS];
    double nsum = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        X[s] = U[s * C + idx] * rinv * tk->iW[s];
        nsum += X[s];
    }
    const double inv = 1.0 / nsum;
    double Wbar = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        X[s] *= inv;
        Wbar += X[s] * tk->W[s];
    }
    const double lt = log(T);
    auto fit = [&](cptr<double> a) {
        return fma_sc(fma_sc(fma(a[3], lt, a[2]), lt, a[1]), lt, a[0]);
    };
    // Eq. 22 for one property: sum_s X_s a_s / sum_t X_t Phi_st with
    // Phi_st = wa_st (1 + sqrt(a_s / a_t) wb_st)^2
    auto mix = [&](cptr<double> coef) {
        double sa[NS], isa[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            sa[s] = rx_exp(0.5 * fit(coef + 4 * s), ec);
            isa[s] = rcp_nr(sa[s]);
        }
        double out = 0.0;
        // one row of the pair tables at a time (unrolled, all 2 NS^2
        // table values are loaded up front and spill the scalar registers)
#pragma unroll 1
        for (int s = 0; s < NS; ++s) {
            double den = 0.0;
#pragma unroll
            for (int t = 0; t < NS; ++t) {
                const double f = fma(sa[s] * isa[t], tk->wb[s][t], 1.0);
                den = fma(X[t] * tk->wa[s][t], f * f, den);
            }
            out = fma(X[s] * (sa[s] * sa[s]), rcp_nr(den), out);
        }
        return out;
    };
    Q[idx] = mix((cptr<double>)&tk->mu[0][0]);
    Q[C + idx] = mix((cptr<double>)&tk->kappa[0][0]);
    Q[2 * C + idx] = U[NS * C + idx] * rinv;
    Q[3 * C + idx] = U[(NS + 1) * C + idx] * rinv;
    Q[4 * C + idx] = U[(NS + 2) * C + idx] * rinv;
    // Eq. 26: D_sm = sum_{t != s} X_t W_t / (Wbar sum_{t != s} X_t / D_st),
    // 1 / D_st = exp(-fit) p / p_ref
    double num[NS], den[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) num[s] = den[s] = 0.0;
    const double pr = p * tk->ip_ref;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int t = s + 1; t < NS; ++t) {
            const double iD = rx_exp(-fit((cptr<double>)&tk->D[s][t][0]), ec) * pr;
            const double Xs = X[s] + 1e-12, Xt = X[t] + 1e-12;
            num[s] = fma(Xt, tk->W[t], num[s]);
            den[s] = fma(Xt, iD, den[s]);
            num[t] = fma(Xs, tk->W[s], num[t]);
            den[t] = fma(Xs, iD, den[t]);
        }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) Q[(5 + s) * C + idx] = NS > 1 ? num[s] / (Wbar * den[s]) : 0.0;
}

// ---------------------------------------------------------------------------
// point value of F_v at one face
// ---------------------------------------------------------------------------
XF_HD double fv_face(double a0, double a1, double a2, double a3) {
    return (-a0 + 9.0 * a1 + 9.0 * a2 - a3) * 0.0625;
}
XF_HD double fv_normal(double a0, double a1, double a2, double a3, double i24h) {
    return (a0 - 27.0 * a1 + 27.0 * a2 - a3) * i24h;
}

// One block's cells along the sweep axis, thread t one cell, neighbours along
// the axis W threads apart: the cells' fields go to LDS, threads with a face
// (between the cells at t + W and t + 2 W) form its point flux from the four
// cells t..t + 3 W, and threads with fin add their own cell's residual from
// the point fluxes of t - 3 W..t.  cell: the thread's cell (in the padded
// grid also where it neither owns a face nor finishes).
//
// What bounds it: memory.  A face needs 4 (2 NS + 11) values; read from global
// memory face by face, those loads went out in groups as registers allowed and
// the kernels waited on them (x 384, y 509, z 522 us a pass at nine species and
// 2.9 M cells, against 295 us for the bytes).  Staged, each cell's fields are
// loaded once by its own thread, most of them before the first wait, and the species'
// enthalpies and mass fractions are formed once a cell instead of four times:
// x 295, y 320, z 310 us.  The diffusion coefficients, needed last, are asked for
// after the first fields have gone to LDS: all at once spill (y 366 us).
template <int NS>
struct ViscStage {
    static constexpr int kFields = NS + 10 > 2 * NS + 1 ? NS + 10 : 2 * NS + 1;   // and >= NS + 4 fluxes
};

template <int NS, int DIR, int NT, int W>
__device__ __forceinline__ void visc_block(const double *__restrict__ U, const double *__restrict__ P,
                                           const double *__restrict__ Q, const double *__restrict__ G,
                                           double *__restrict__ rhs, const Geo &g, const ThermoK<double> &th,
                                           int terms, double id, double (*S)[NT], int t, long long cell, bool face,
                                           bool fin) {
    constexpr int NV = NS + 4;
    const long long C = g.cells;
    constexpr int T1 = Axes<DIR>::t1, T2 = Axes<DIR>::t2;
    const bool a1 = (T1 == 0 ? g.nx : T1 == 1 ? g.ny : g.nz) > 1;
    const bool a2 = (T2 == 0 ? g.nx : T2 == 1 ? g.ny : g.nz) > 1;
    const bool stress = terms & kViscousStress, heat = terms & kViscousHeat, diff = terms & kViscousDiffusion;
    const double i24h = id / 24.0;
    auto fc = [&](int f) { return fv_face(S[f][t], S[f][t + W], S[f][t + 2 * W], S[f][t + 3 * W]); };
    auto nd = [&](int f) { return fv_normal(S[f][t], S[f][t + W], S[f][t + 2 * W], S[f][t + 3 * W], i24h); };
    const double T = P[cell];
    double A[9] = {}, y[NS], D[NS], rho = 0.0;
    if (stress) {
        A[0] = Q[cell];
#pragma unroll
        for (int k = 0; k < 3; ++k) A[1 + k] = Q[(2 + k) * C + cell];
        // tangential derivatives: d u_DIR / d x_t and d u_t / d x_t
        if (a1) A[4] = G[(3 * T1 + DIR) * C + cell], A[5] = G[(3 * T1 + T1) * C + cell];
        if (a2) A[6] = G[(3 * T2 + DIR) * C + cell], A[7] = G[(3 * T2 + T2) * C + cell];
    }
    if (heat) A[8] = Q[C + cell];
    if (diff) {
        const double rinv = P[3 * C + cell];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            y[s] = U[s * C + cell];
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            rho += y[s];
            y[s] *= rinv;
        }
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) S[q][t] = A[q];
    S[9][t] = T;
    if (diff) {
#pragma unroll
        for (int s = 0; s < NS; ++s) S[10 + s][t] = e_species(th, s, T) + th.Rs[s] * T;
        XF_FENCE();
#pragma unroll
        for (int s = 0; s < NS; ++s) D[s] = Q[(5 + s) * C + cell];
    }
    __syncthreads();
    double F[NV], hf[NS];
#pragma unroll
    for (int q = 0; q < NV; ++q) F[q] = 0.0;
    if (face && stress) {
        const double mu = fc(0);
        double uf[3], Gf[3][3] = {};            // Gf[a][b] = d u_b / d x_a, the entries used
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            uf[k] = fc(1 + k);
            Gf[DIR][k] = nd(1 + k);
        }
        Gf[T1][DIR] = a1 ? fc(4) : 0.0;
        Gf[T1][T1] = a1 ? fc(5) : 0.0;
        Gf[T2][DIR] = a2 ? fc(6) : 0.0;
        Gf[T2][T2] = a2 ? fc(7) : 0.0;
        const double div = Gf[0][0] + Gf[1][1] + Gf[2][2];
        double work = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double tau = mu * (Gf[k][DIR] + Gf[DIR][k]);
            if (k == DIR) tau = tau - 2.0 / 3.0 * mu * div;
            F[NS + k] = tau;
            work = work + tau * uf[k];
        }
        F[NS + 3] = work;
    }
    if (face && heat) F[NS + 3] = F[NS + 3] + fc(8) * nd(9);     // - q_c = kappa dT/dx
    if (diff) {
        if (face) {
#pragma unroll
            for (int s = 0; s < NS; ++s) hf[s] = fc(10 + s);
        }
        __syncthreads();
        S[0][t] = rho;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            S[1 + s][t] = y[s];
            S[1 + NS + s][t] = D[s];
        }
        __syncthreads();
        if (face) {
            const double rf = fc(0);
            double Yf[NS], Dd[NS];
            double corr = 0.0;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                Yf[s] = fc(1 + s);
                Dd[s] = fc(1 + NS + s) * nd(1 + s);
                corr = corr + Dd[s];
            }
            double e = F[NS + 3];
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const double J = -rf * (Dd[s] - Yf[s] * corr);
                F[s] = -J;
                e = e - hf[s] * J;              // - q_d
            }
            F[NS + 3] = e;
        }
    }
    double r[NV];
    if (fin) {
#pragma unroll
        for (int q = 0; q < NV; ++q) r[q] = rhs[q * C + cell];
    }
    __syncthreads();
    if (face) {
#pragma unroll
        for (int q = 0; q < NV; ++q) S[q][t] = F[q];
    }
    __syncthreads();
    if (fin) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double hl = (-S[q][t - 3 * W] + 26.0 * S[q][t - 2 * W] - S[q][t - W]) * (1.0 / 24.0);
            const double hr = (-S[q][t - 2 * W] + 26.0 * S[q][t - W] - S[q][t]) * (1.0 / 24.0);
            rhs[q * C + cell] = r[q] + (hr - hl) * id;
        }
    }
}

// ---------------------------------------------------------------------------
// x direction: cells -3..nx+2 of every interior row, linearised (nx + 6 per
// row); a block of 256 threads takes 256 consecutive cells and blocks overlap
// by six, so each cell's four point faces meet in one block.  The block count
// is a multiple of the XCD count and each XCD takes one contiguous range of
// cells (neighbouring blocks share their edge cells in one L2).
// ---------------------------------------------------------------------------
constexpr int kViscXBlock = 256;

template <int NS>
__global__ __launch_bounds__(kViscXBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_visc_x(
    const double *__restrict__ U, const double *__restrict__ P, const double *__restrict__ Q,
    const double *__restrict__ G, double *__restrict__ rhs, Geo g, ThermoK<double> th, int terms) {
    __shared__ double S[ViscStage<NS>::kFields][kViscXBlock];
    unsigned lb, u1, u2;
    xcd_block(lb, u1, u2);
    const int t = threadIdx.x;
    const long long n = ((long long)g.nx + 6) * g.ny * g.nz;
    const long long f0 = (long long)lb * (kViscXBlock - 6);
    if (f0 >= n) return;   // blocks that round the grid up to a multiple of 8
    const long long f = f0 + t;
    int kk, j, k;                                // cell kk - 3 of row (j, k)
    split3(g, f < n ? f : n - 1, g.nx + 6, g.ny, g.dvf, g.dny, kk, j, k);
    const long long cell = (long long)(g.gz + k) * g.sz + (long long)(g.gy + j) * g.sy + g.gx + kk - 3;
    const bool face = f < n && kk <= g.nx + 2 && t < kViscXBlock - 3;
    visc_block<NS, 0, kViscXBlock, 1>(U, P, Q, G, rhs, g, th, terms, g.idx, S, t, cell, face,
                                      face && kk >= 3 && t >= 3);
}

// ---------------------------------------------------------------------------
// y/z directions: tiles of kViscTX x-columns by kViscTS consecutive cells
// along the sweep axis; tiles overlap by six cells.  Lanes run along x
// (coalesced loads).
// ---------------------------------------------------------------------------
constexpr int kViscTX = 16, kViscTS = 32;

template <int NS, int DIR>
__global__ __launch_bounds__(kViscTX *kViscTS) __attribute__((amdgpu_waves_per_eu(4))) void k_visc_tile(
    const double *__restrict__ U, const double *__restrict__ P, const double *__restrict__ Q,
    const double *__restrict__ G, double *__restrict__ rhs, Geo g, ThermoK<double> th, int terms) {
    __shared__ double S[ViscStage<NS>::kFields][kViscTX * kViscTS];
    unsigned bx, by, bz;
    xcd_block(bx, by, bz);
    const int tx = threadIdx.x, ts = threadIdx.y;
    const int x = bx * kViscTX + tx;
    const int kk = by * (kViscTS - 6) + ts;       // cell kk - 3 of the column
    const int nsw = DIR == 1 ? g.ny : g.nz;
    const long long col =
        (long long)(g.gx + min(x, g.nx - 1)) +
        (DIR == 1 ? (long long)(g.gz + bz) * g.sz : (long long)(g.gy + bz) * g.sy);
    const long long cell =
        col + (long long)((DIR == 1 ? g.gy : g.gz) + min(kk, nsw + 5) - 3) * (DIR == 1 ? g.sy : g.sz);
    const bool face = x < g.nx && kk <= nsw + 2 && ts < kViscTS - 3;
    visc_block<NS, DIR, kViscTX * kViscTS, kViscTX>(U, P, Q, G, rhs, g, th, terms, DIR == 1 ? g.idy : g.idz, S,
                                                    ts * kViscTX + tx, cell, face, face && ts >= 3);
}

}  // namespace xf
