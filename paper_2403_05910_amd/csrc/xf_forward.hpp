// xf_forward.hpp -- forward kernels of the convective right-hand side.
//
//   k_prims       primitive recovery with the Newton temperature (Eq. 7, 21);
//                 the CFL maximum (Eq. 17) and the GLF speeds
//   k_sweep_x     x-direction flux difference, one face per thread
//   k_sweep_tile  y/z-direction flux difference, tiles of one face per thread
#pragma once

#include "xf_face64.hpp"

namespace xf {

// ---------------------------------------------------------------------------
// primitive variables and Newton temperature (always FP64)
// ---------------------------------------------------------------------------
// The mixture's internal energy and C_v at fixed Y as polynomials in T:
// e(T) = sum_k E_k T^k (k = 0..5), C_v(T) = sum_k C_k T^k (k = 0..4), the
// species tables weighted by Y once per solve, so that a Newton iteration
// costs two Horner evaluations instead of one per species.
struct MixPoly {
    double E[6], C[5];
    __device__ __forceinline__ double e(double T) const {
        return ((((E[5] * T + E[4]) * T + E[3]) * T + E[2]) * T + E[1]) * T + E[0];
    }
    __device__ __forceinline__ double cv(double T) const {
        return (((C[4] * T + C[3]) * T + C[2]) * T + C[1]) * T + C[0];
    }
};

// Newton on e(T) = e (Eq. 21) with the mixture polynomials m:
// T <- T + (e - e(T)) / C_v(T) from the start T clamped into the bracket
// [T_lo, T_hi] where there is one; every evaluation narrows the bracket
// (e(T) > e: hi = T, else lo = T) and a step that leaves the closed bracket
// is replaced by bisection.  Stop when |dT| <= 1e-11 |T|, then one more
// Newton update.  Returns false if not converged in 50 iterations.  The
// primitive pass starts from the cold start e / C_v(T_ref); the reaction
// step from the cell's previous temperature (the root does not depend on
// the start).
__device__ __forceinline__ bool newton_poly(bool bracket, double T_lo, double T_hi, const MixPoly &m, double e,
                                            double &T) {
    double lo = T_lo, hi = T_hi;
    if (bracket) T = T < lo ? lo : (T > hi ? hi : T);
    for (int it = 0; it < kNewtonMaxIt; ++it) {
        const double f = m.e(T) - e;
        double Tn = T - f / m.cv(T);
        if (bracket) {
            if (f > 0.0)
                hi = fmin(hi, T);
            else
                lo = fmax(lo, T);
            if (Tn < lo || Tn > hi) Tn = 0.5 * (lo + hi);
        }
        const bool conv = fabs(Tn - T) <= kNewtonTol * fabs(T);
        T = Tn;
        if (conv) {
            T = T - (m.e(T) - e) / m.cv(T);
            return true;
        }
    }
    return false;
}

// The fold of the species tables with Y (the table at hand, by value or
// in kernel arguments).
template <int NS>
__device__ __forceinline__ void mix_poly_of(const ThermoK<double> &th, const double *Y, MixPoly &m) {
#pragma unroll
    for (int k = 0; k < 6; ++k) m.E[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 5; ++k) m.C[k] = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int k = 0; k < 6; ++k) m.E[k] += Y[s] * th.e[s][k];
#pragma unroll
        for (int k = 0; k < 5; ++k) m.C[k] += Y[s] * th.cv[s][k];
    }
}

// The primitive variables of one cell from its conserved values u(f)
// (f = 0..N+3): T by Newton (Eq. 21) on the mixture polynomials,
// p = rho Rbar T, c^2 = (1 + Rbar / C_v) Rbar T, 1/rho; returns the cell's
// status flags.
template <int NS, class Get>
__device__ __forceinline__ unsigned cell_prims(const Get &u, const ThermoK<double> &th, double &T, double &p,
                                               double &c, double &rinv) {
    double Y[NS];
    double rho = 0.0;
    bool finite = true;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        Y[s] = u(s);
        rho += Y[s];
        finite = finite && isfinite(Y[s]);
    }
    rinv = 1.0 / rho;
    unsigned flags = 0;
    bool yneg = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        Y[s] *= rinv;
        yneg = yneg || (Y[s] < -1e-12);
    }
    const double mx = u(NS), my = u(NS + 1), mz = u(NS + 2);
    const double E = u(NS + 3);
    finite = finite && isfinite(mx) && isfinite(my) && isfinite(mz) && isfinite(E);
    const double uu = mx * rinv, v = my * rinv, w = mz * rinv;
    const double e = E * rinv - 0.5 * (uu * uu + v * v + w * w);
    // Newton on the mixture's folded polynomials from the cold start
    // e / C_v(T_ref)
    MixPoly m;
    mix_poly_of<NS>(th, Y, m);
    T = e / m.cv(th.T_ref);
    const bool conv = newton_poly(th.bracket, th.T_lo, th.T_hi, m, e, T);
    double Rb = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) Rb += Y[s] * th.Rs[s];
    const double cv = m.cv(T);
    p = rho * Rb * T;
    c = sqrt((1.0 + Rb / cv) * Rb * T);
    if (rho <= 0.0) flags |= XF_FLAG_RHO;
    if (yneg) flags |= XF_FLAG_Y;
    if (p <= 0.0 || T <= 0.0) flags |= XF_FLAG_P;
    if (th.bracket && (T < th.T_lo || T > th.T_hi)) flags |= XF_FLAG_TRANGE;
    if (!conv) flags |= XF_FLAG_NEWTON;
    if (!finite || !isfinite(T) || !isfinite(c)) flags |= XF_FLAG_NAN;
    return flags;
}

// P[0..3][cell] = (T, p, c, 1/rho) for every cell with at most one
// coordinate in a ghost layer (the cells axis-aligned stencils read).
// Uf, Pf (optional): FP32 copies of U and of (T, p, c, 1/rho) for the
// mixed-precision sweeps, written for the same cells; P may be null when
// only they are needed.
// DT: the last block also divides; GLF: the pass takes the GLF speeds.  With
// run-time switches instead, the passes that do neither got slower: with DT, a
// CU6 GLF right-hand side of 0.7 M cells took 271 us instead of 268; with GLF,
// the pass alone 13.7 us instead of 13.1 (64^3, nine species) and 43.5 instead of
// 42.0 (128^3, five).  The GLF instance still tests its pointer: without the test
// its code is scheduled otherwise, and the right-hand side above took 0.5 to 0.8 %
// longer.
template <int NS, bool DT, bool GLF>
__global__ __launch_bounds__(256) void k_prims(const double *U, double *__restrict__ P, Geo g,
                                               ThermoK<double> th, unsigned *status, float *__restrict__ Uf,
                                               float *__restrict__ Pf, int all_cells, double *Ug,
                                               unsigned long long *mx, unsigned long long *glf, double cfl, double *dt) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    // GLF: the direction's speeds |u_d - c|, |u_d|, |u_d + c| of a cell its
    // stencils read (interior in the other axes)
    double gv[9] = {};
    double sv = 0.0;   // with cfl: the cell's rate sum_d (|u_d| + c) / dx_d of Eq. 17 (interior cells)
    if (idx < g.cells) {
        int x, y, z;
        split3(g, idx, g.px, g.py, g.dpx, g.dpy, x, y, z);
        const int ng = (x < g.gx || x >= g.gx + g.nx) + (y < g.gy || y >= g.gy + g.ny) +
                       (z < g.gz || z >= g.gz + g.nz);
        // edge and corner ghosts lie outside every stencil
        if (ng <= 1 || all_cells) {
            const long long C = g.cells;
            // with Ug (= U): a ghost takes its boundary source's state, written
            // to the ghost as the ghost fill would.  Each ghost coordinate maps
            // to its source on its own axis (the axis-by-axis fill gives an edge
            // or corner ghost the state of the interior cell all its
            // coordinates map to); sources are interior cells, which this pass
            // does not write.
            long long src = idx;
            if (Ug && ng > 0) {
                const int sx = ghost_map(x, g.nx, g.gx, g.bc[0], g.bc[1]), sy = ghost_map(y, g.ny, g.gy, g.bc[2], g.bc[3]),
                          sz = ghost_map(z, g.nz, g.gz, g.bc[4], g.bc[5]);
                src = sx + (long long)g.px * (sy + (long long)g.py * sz);
            }
            double u[NS + 4];
#pragma unroll
            for (int f = 0; f < NS + 4; ++f) u[f] = U[f * C + src];
            if (src != idx) {
#pragma unroll
                for (int f = 0; f < NS + 4; ++f) Ug[f * C + idx] = u[f];
            }
            // the FP32 copies go out before the Newton solve, from the loaded
            // values (read again after it, the state was partly evicted from
            // the L2 and fetched twice: 2.43 against 1.92 GB per launch at
            // 256^3, nine species)
            if (Uf) {
#pragma unroll
                for (int f = 0; f < NS + 4; ++f) Uf[f * C + idx] = (float)u[f];
            }
            double T, p, c, rinv;
            const unsigned flags = cell_prims<NS>([&](int f) { return u[f]; }, th, T, p, c, rinv);
            if (P) {
                P[idx] = T;
                P[C + idx] = p;
                P[2 * C + idx] = c;
                P[3 * C + idx] = rinv;
            }
            if (Uf) {
                Pf[idx] = (float)T;
                Pf[C + idx] = (float)p;
                Pf[2 * C + idx] = (float)c;
                Pf[3 * C + idx] = (float)rinv;
            }
            if (mx && ng == 0) {
                double v = 0.0;
                if (g.nx > 1) v += (fabs(u[NS] * rinv) + c) * g.idx;
                if (g.ny > 1) v += (fabs(u[NS + 1] * rinv) + c) * g.idy;
                if (g.nz > 1) v += (fabs(u[NS + 2] * rinv) + c) * g.idz;
                if (v > sv) sv = v;   // NaN never wins (it is flagged)
            }
            if (GLF && glf) {
                const bool in[3] = {x >= g.gx && x < g.gx + g.nx, y >= g.gy && y < g.gy + g.ny,
                                    z >= g.gz && z < g.gz + g.nz};
                const bool active[3] = {g.nx > 1, g.ny > 1, g.nz > 1};
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double un = u[NS + d] * rinv;
                    if (active[d] && in[(d + 1) % 3] && in[(d + 2) % 3]) {   // fmax: NaN never wins
                        gv[3 * d] = fmax(0.0, fabs(un - c));
                        gv[3 * d + 1] = fmax(0.0, fabs(un));
                        gv[3 * d + 2] = fmax(0.0, fabs(un + c));
                    }
                }
            }
            if (flags) atomicOr(status, flags);
        }
    }
    if (GLF && glf) {
        // block maxima, then one 64-bit atomicMax each (see below).  A pass of
        // its own per direction read the state again, 27 us each at 0.7 M
        // cells where the primitives themselves take 21
#pragma unroll
        for (int k = 0; k < 9; ++k) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) gv[k] = fmax(gv[k], __shfl_xor(gv[k], off, 64));
        }
        __shared__ double gmax[9][4];
        if ((threadIdx.x & 63) == 0) {
#pragma unroll
            for (int k = 0; k < 9; ++k) gmax[k][threadIdx.x >> 6] = gv[k];
        }
        __syncthreads();
        if (threadIdx.x < 9) {
            const double *w = gmax[threadIdx.x];
            const unsigned long long bits =
                (unsigned long long)__double_as_longlong(fmax(fmax(w[0], w[1]), fmax(w[2], w[3])));
            if (bits > __atomic_load_n(glf + threadIdx.x, __ATOMIC_RELAXED)) atomicMax(glf + threadIdx.x, bits);
        }
    }
    if (mx) {
        // block max, then one 64-bit atomicMax (positive doubles order like
        // their bit patterns), skipped when the running max is already larger
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sv = fmax(sv, __shfl_xor(sv, off, 64));
        __shared__ double wmax[4];
        if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = sv;
        __syncthreads();
        if (threadIdx.x == 0) {
            const double m = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
            const unsigned long long bits = (unsigned long long)__double_as_longlong(m);
            if (bits > __atomic_load_n(mx, __ATOMIC_RELAXED)) atomicMax(mx, bits);
            if constexpr (DT) {
                __threadfence();
                if (atomicAdd(mx + kCflDone, 1ull) == gridDim.x - 1) {
                    __threadfence();
                    *dt = cfl / __longlong_as_double((long long)atomicMax(mx, 0ull));
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Occupancy per kernel flavour, from the compiler's resource report and
// timings at 256^3, nine species: the exchanging FP64 WENO5 instances fit three
// waves per SIMD (168 registers) without spill, with their species loops rolled
// two species at a time; the positivity-blend instances stay at two (at three the
// FP64 blended step went from 37.5 to 47.7 ms, taken with an earlier face), CU6
// too (28 to 120 bytes of spill at three), the FP64 WENO7 instances at one (at
// two they spilled 324-460 bytes per lane).
// Waves per SIMD asked of a face-per-thread sweep (X: the x sweep).
template <typename R, int REC, bool X, bool PP>
constexpr int sweep_waves() {
    if (sizeof(R) == 4) return X ? 4 : (!PP && REC == kReconWeno5) ? 5 : 1;
    if (REC == kReconWeno7) return 1;
    if (!X && !PP && REC == kReconWeno5) return 3;     // the exchanging FP64 tiles (CU6 spills at three)
    return (X && !PP && REC == kReconWeno5) ? 3 : 2;
}

// lam = D dt / dx_d of the positivity blend (D active dimensions).
template <typename R>
__device__ __forceinline__ R pp_lambda(const Geo &g, const StageArgs &sa, double idx) {
    const double h = sa.dt_dev ? *sa.dt_dev : sa.dt;
    const int D = (g.nx > 1) + (g.ny > 1) + (g.nz > 1);
    return R(D * h * idx);
}

// Where a sweep's flux differences go.  kStore: to rhs; kAdd: added to what
// an earlier direction left in rhs; kFinish: the last sweep of an RK3 stage
// finishes it, Uout = a U0 + b (Uin + h L) with L the sum of the directions.
// FP64 sweeps accumulate L in rhs and take Uin from the staged stencil; the
// mixed ones keep one FP32 buffer per direction and read Uin in FP64.  The
// separate stage kernel this replaced moved 10.4 GB per stage at 256^3, nine
// species (1.85 ms), most of it read again from what the sweeps had just
// touched.  What bounds the finish is the latency of its loads: load() runs a
// component ahead of put() in the exchanging sweeps, and for all components
// at once where the block's fluxes wait in LDS.  The exchanging sweeps take
// the mode as a template argument and load without a branch (an address that
// is not needed is replaced by one that is, its value multiplied by zero):
// with run-time switches around each component the z sweep, which only
// stores, took 1.85 ms instead of 1.57.  kByArgs: read from the arguments.
constexpr int kByArgs = -1, kStore = 0, kAdd = 1, kFinish = 2;
template <typename R, int MODE>
struct CellOut {
    // what one cell and field needs from memory
    struct Held {
        double L = 0.0, U0 = 0.0;              // FP64: the directions summed so far
        double Uin = 0.0, Lv = 0.0;            // mixed
        float Ly = 0.0f, Lz = 0.0f;
    };
    R *rhs;
    const StageArgs &sa;
    const double *pL, *p0;                     // FP64 kFinish: where L and U0 are read
    double h, fL;                              // fL: 1 when L is read, 0 when this sweep is the only one
    int accumulate;
    __device__ __forceinline__ CellOut(R *r, const StageArgs &s, int acc)
        : rhs(r), sa(s), h(!s.Uout ? 0.0 : s.dt_dev ? *s.dt_dev : s.dt), accumulate(acc) {
        if constexpr (sizeof(R) == 8 && MODE == kFinish) {
            pL = acc ? rhs : s.Uin;
            p0 = s.a != 0.0 ? s.U0 : pL;
            fL = acc ? 1.0 : 0.0;
        }
    }
    __device__ __forceinline__ bool finish() const { return MODE == kByArgs ? sa.Uout != nullptr : MODE == kFinish; }
    __device__ __forceinline__ bool add() const { return MODE == kByArgs ? accumulate != 0 : MODE == kAdd; }
    __device__ __forceinline__ void load(long long o, Held &v) const {
        if constexpr (sizeof(R) == 8 && MODE == kFinish) {
            v.L = pL[o];
            v.U0 = p0[o];
            return;
        }
        if constexpr (sizeof(R) == 8) {
            if (add()) v.L = rhs[o];
        } else if (finish()) {
            v.Uin = sa.Uin[o];
            if (sa.Ly32) v.Ly = sa.Ly32[o];
            if (sa.Lz32) v.Lz = sa.Lz32[o];
            if (sa.Lv) v.Lv = sa.Lv[o];
        }
        if (finish() && sa.a != 0.0) v.U0 = sa.U0[o];
    }
    // d: the flux difference of this sweep; Uin: the stage input (FP64 sweeps)
    __device__ __forceinline__ void put(long long o, double d, double Uin, const Held &v) const {
        if constexpr (sizeof(R) == 8 && MODE == kFinish) {
            sa.Uout[o] = sa.a * v.U0 + sa.b * (Uin + h * (fL * v.L + d));
            return;
        }
        if constexpr (sizeof(R) == 8) {
            if (add()) d = v.L + d;
        } else if (finish()) {
            if (sa.Ly32) d += (double)v.Ly;
            if (sa.Lz32) d += (double)v.Lz;
            if (sa.Lv) d += v.Lv;
            Uin = v.Uin;
        }
        if (finish()) {
            const double w = Uin + h * d;
            sa.Uout[o] = sa.a == 0.0 ? sa.b * w : sa.a * v.U0 + sa.b * w;
        } else {
            rhs[o] = R(d);
        }
    }
    // all NV fields of one cell, the loads ahead of their uses: all of them at
    // once, or in the mixed finish, whose values take eight registers a
    // field, five fields at a time
    template <int NV, class D, class U>
    __device__ __forceinline__ void put_all(long long cells, long long cell, D &&d, U &&uin) const {
        constexpr int B = sizeof(R) == 8 ? NV : 5;
#pragma unroll
        for (int b = 0; b < NV; b += B) {
            Held v[B];
#pragma unroll
            for (int k = 0; k < B && b + k < NV; ++k) load((b + k) * cells + cell, v[k]);
#pragma unroll
            for (int k = 0; k < B && b + k < NV; ++k)
                put((b + k) * cells + cell, d(b + k), uin(b + k), v[k]);
        }
    }
};

// Hands the flux components of an exchanging sweep on: the component of this
// face goes to its own lane's cell (the one below the face) together with the
// neighbouring face's, taken STEP lanes down; faces in a wave's first and
// last row leave theirs for the cell between two waves (first, last).
template <int IM, int STEP, class CO, typename R, class First, class Last, class Uin>
struct ExchangeOut {
    const CO &co;
    long long cells, cell;
    R id;
    bool own, top;                   // the cell below is this wave's; the face is in its last row
    First first;
    Last last;
    Uin uin;
    typename CO::Held held[5];
    int from = 4 * (int)((threadIdx.x + blockDim.x * threadIdx.y - STEP) & 63);   // byte index of that lane
    __device__ __forceinline__ R lanes_down(R v) const {
        if constexpr (sizeof(R) == 8) {
            const int lo = __builtin_amdgcn_ds_bpermute(from, __double2loint(v));
            const int hi = __builtin_amdgcn_ds_bpermute(from, __double2hiint(v));
            return __hiloint2double(hi, lo);
        } else {
            return __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(v)));
        }
    }
    // every lane loads (a cell that is not its own lies in the padded array
    // too), so that no branch parts the loads from the work ahead of their use
    __device__ __forceinline__ void start() { co.load(cell, held[0]); }
    template <int SLOT>
    __device__ __forceinline__ void next(int q) {
        co.load(q * cells + cell, held[SLOT]);
    }
    __device__ __forceinline__ void rest() {
#pragma unroll
        for (int k = 1; k < 4; ++k) co.load((IM + k) * cells + cell, held[1 + k]);
    }
    template <int SLOT>
    __device__ __forceinline__ void put(int q, R v) {
        const R vb = lanes_down(v);            // the face below, valid wherever this face is
        if (own) {
            // the FP32 face asks for nothing ahead (its sweeps only store,
            // but for the y or z sweep that finishes a stage without an x axis)
            if constexpr (sizeof(R) == 4) co.load(q * cells + cell, held[SLOT]);
            co.put(q * cells + cell, double((vb - v) * id), uin(q), held[SLOT]);
        } else {
            first(q, v);
        }
        if (top) last(q, v);
    }
};

// Keeps a face's whole flux vector (in LDS).
template <class Put>
struct StoreOut {
    Put f;
    __device__ __forceinline__ void start() {}
    template <int SLOT>
    __device__ __forceinline__ void next(int) {}
    __device__ __forceinline__ void rest() {}
    template <int SLOT, typename R>
    __device__ __forceinline__ void put(int q, R v) {
        f(q, v);
    }
};
template <class Put>
__device__ __forceinline__ StoreOut<Put> store_out(Put p) {
    return StoreOut<Put>{p};
}

// ---------------------------------------------------------------------------
// x sweep: faces linearised over interior rows (face i of row r = the face
// between interior cells i-1 and i, i = 0..nx).  A block of 256 threads takes
// fpb <= 256 consecutive faces and blocks overlap by one face, so every cell
// whose two faces lie in a block gets (F^_{i-1/2} - F^_{i+1/2}) / dx there.
// The block first copies U and the primitives of its stencil cells to LDS,
// row segment by row segment: the faces of one row need their own cells plus
// 2 RAD - 1 more, so a block touching nseg rows stages fpb + nseg (2 RAD - 1)
// cells.  Unstaged, the six overlapping stencil loads of each field went to
// the caches, and at three blocks per CU the working set outgrew the L2:
// 4.0 GB fetched per launch at 256^3, nine species, against 2.33 GB of
// stencil inputs.  fpb is 256 whenever a row holds at least 255 faces; for
// shorter rows the launch lowers it until the staged cells fit x_stage_cells.
// The FP64 WENO5 instances without the blend hand each flux component to
// the cell below as soon as it is final, taking the neighbouring face's
// value from the next lane down; the first lane of each wave takes it
// through LDS.  The others keep the block's fluxes in LDS (the blend limits
// whole flux vectors).  In an RK3 step it also finishes the stage (sa.Uout),
// which at 256^3 and nine species makes it memory bound: 7.5 GB in FP64, 1.81 ms,
// where a copy of that size takes 1.72.
// ---------------------------------------------------------------------------
constexpr int kXBlock = 256;

template <int RAD>
constexpr int x_stage_cells() { return kXBlock + 2 * (2 * RAD - 1); }

// Faces per x-sweep block for rows of nfx faces: the largest count whose
// worst-case staging (a window of fpb faces spans at most
// ceil((fpb - 1) / nfx) + 1 rows) fits x_stage_cells.
template <int RAD>
inline int x_faces_per_block(long long nfx) {
    constexpr int gap = 2 * RAD - 1;
    int fpb = kXBlock;
    while (fpb > 2 && fpb + ((fpb - 1 + nfx - 1) / nfx + 1) * gap > x_stage_cells<RAD>()) --fpb;
    return fpb;
}

// Exchanging x sweeps: FP64 WENO5 (three waves per SIMD).  The CU6 and
// WENO7 faces (two and one waves per SIMD) took 3.09 ms per x sweep
// exchanging against 2.62 and 2.65 ms with the fluxes in LDS (256^3, nine
// species, with an earlier face).
template <typename R, int REC, bool PP>
constexpr bool x_exchange() { return sizeof(R) == 8 && REC == kReconWeno5 && !PP; }

// Copies U and the primitives of a block's stencil cells into LDS, SZ cells
// field by field; at(e, cell) tells whether staged cell e exists and gives
// its padded index.  A block has a few more cells than threads, so some
// threads take a second one; all loads go out before the first is waited for
// (one cell at a time, the second waited out a memory latency of its own
// while most of the block idled).
template <int NV, int THREADS, int SZ, typename S, class At>
__device__ __forceinline__ void stage_cells(const S *__restrict__ U, const S *__restrict__ P, long long cells, S *to,
                                            int t, const At &at) {
    static_assert(SZ <= 2 * THREADS, "two cells a thread");
    S a[NV + 4], b[NV + 4];
    long long ca, cb;
    const bool ha = at(t, ca), hb = t + THREADS < SZ && at(t + THREADS, cb);
    auto load = [&](S *v, long long cell) {
#pragma unroll
        for (int q = 0; q < NV; ++q) v[q] = U[q * cells + cell];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[NV + q] = P[q * cells + cell];
    };
    auto store = [&](const S *v, int e) {
#pragma unroll
        for (int q = 0; q < NV + 4; ++q) to[q * SZ + e] = v[q];
    };
    if (ha) load(a, ca);
    if (hb) load(b, cb);
    if (ha) store(a, t);
    if (hb) store(b, t + THREADS);
}

template <int NS, typename R, typename S, bool PP, int SPD, int REC, int MODE>
__global__ __launch_bounds__(kXBlock) __attribute__((amdgpu_waves_per_eu(sweep_waves<R, REC, true, PP>()))) void k_sweep_x(
    const S *__restrict__ U, const S *__restrict__ P, R *__restrict__ rhs, Geo g, ThermoK<R> th, int accumulate,
    StageArgs sa, unsigned *status, Dissip ds, int fpb, FastDiv dw) {
    constexpr int NV = NS + 4;
    constexpr int RAD = stencil_radius(REC);
    constexpr int GAP = 2 * RAD - 1;
    constexpr int XC = x_stage_cells<RAD>();
    constexpr bool EXCH = x_exchange<R, REC, PP>();
    constexpr int NW = kXBlock / 64;
    __shared__ R sF[EXCH ? 1 : NV][EXCH ? 1 : kXBlock];
    __shared__ R sEdge[2][EXCH ? NW : 1][EXCH ? NV : 1];
    __shared__ S xf_xstage[(NV + 4) * XC];
    const unsigned lb = xcd_linear(blockIdx.x, gridDim.x);
    const int t = threadIdx.x;
    const long long nfx = (long long)g.nx + 1;
    const long long nfaces = nfx * g.ny * g.nz;
    const long long f0 = (long long)lb * (fpb - 1);
    if (f0 >= nfaces) return;   // blocks that round the grid up to a multiple of 8
    const long long flast = min(f0 + fpb - 1, nfaces - 1);
    // the block's first face: face i0 of row row0 = (j0, k0); its faces lie
    // in rows row0 .. row0 + nseg - 1 (segment sg = row row0 + sg), so the
    // per-cell and per-face indexing below needs 32-bit divisions only
    int i0, j0, k0;
    split3(g, f0, g.nx + 1, g.ny, g.dnf, g.dny, i0, j0, k0);
    const int nfx32 = g.nx + 1;
    auto row_base = [&](int sg) {
        int j = j0 + sg, k = k0;
        if (j >= g.ny) {   // (j < ny + 257)
            const int n = (int)g.dny.of((unsigned)j);
            k += n;
            j -= n * g.ny;
        }
        return (g.gz + k) * g.sz + (long long)(g.gy + j) * g.sy + g.gx;
    };
    {
        // staged cell e: segment sg = (e + i0) / W, W = nfx + GAP, x index
        // e + i0 - sg W - RAD of that row (segment 0 starts at face i0, the
        // others at face 0)
        const int nseg = (int)g.dnf.of((unsigned)(flast - f0) + i0) + 1;
        const int ncell = (int)(flast - f0 + 1) + nseg * GAP;
        const int W = nfx32 + GAP;
        auto at = [&](int e, long long &cell) {
            const int sg = (int)dw.of((unsigned)(e + i0));
            cell = row_base(sg) + (e + i0 - sg * W - RAD);
            return e < ncell;
        };
        stage_cells<NV, kXBlock, XC>(U, P, g.cells, xf_xstage, t, at);
    }
    __syncthreads();
    const long long f = f0 + t;
    const bool valid = t < fpb && f < nfaces;
    const int lane = t & 63, w = t >> 6;
    unsigned flags = 0;
    const R id = R(g.idx) * flux_unit<R>();
    const CellOut<R, MODE> co(rhs, sa, accumulate);
    const auto *stage = (const __attribute__((address_space(3))) S *)xf_xstage;
    int e0 = 0;               // staged index of the face's stencil cell 0
    long long cell = 0;       // the cell below the face
    bool inner = false;       // and whether it is an interior one
    if (valid) {
        const int sg = (int)g.dnf.of((unsigned)(t + i0)), i = t + i0 - sg * nfx32;
        cell = row_base(sg) + i - 1;
        inner = i > 0;
        // stencil cell m of face i (cell i - RAD + m of its row) is staged at
        // t + sg GAP + m
        e0 = t + sg * GAP;
        StencilLds<NV, S> st{stage, e0, 1, XC};
        if constexpr (SPD == kViscFrozen) ds.fidx = f;   // x faces: i + (nx + 1) (j + ny k)
        if constexpr (EXCH) {
            auto first = [&](int q, R v) {
                if (lane == 0) sEdge[1][w][q] = v;
            };
            auto last = [&](int q, R v) { sEdge[0][w][q] = v; };
            auto uin = [&](int q) { return (double)st.u(q, RAD - 1); };
            // face f - 1 is lane t - 1
            ExchangeOut<NS, 1, decltype(co), R, decltype(first), decltype(last), decltype(uin)> out{
                co, g.cells, cell, id, lane > 0 && inner, lane == 63, first, last, uin};
            sweep_face<NS, R, 0, SPD, REC>(st, th, out, flags, ds);
        } else {
            auto out = store_out([&](int q, R v) { sF[q][t] = v; });
            sweep_face<NS, R, 0, SPD, REC>(st, th, out, flags, ds);
            if constexpr (PP) {
                R Fq[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) Fq[q] = sF[q][t] * flux_unit<R>();
                pp_limit<NS, R, 0, RAD>(st, pp_lambda<R>(g, sa, g.idx), Fq);
#pragma unroll
                for (int q = 0; q < NV; ++q) sF[q][t] = Fq[q] * (R(1) / flux_unit<R>());
            }
        }
    }
    __syncthreads();
    // EXCH: only the cell between the last face of wave w - 1 and the first of
    // w is left
    const bool left = EXCH ? lane == 0 && w > 0 : t > 0;
    if (left && inner)
        co.template put_all<NV>(
            g.cells, cell,
            [&](int q) {
                if constexpr (EXCH)
                    return double((sEdge[0][w - 1][q] - sEdge[1][w][q]) * id);
                else
                    return double((sF[q][t - 1] - sF[q][t]) * id);
            },
            [&](int q) { return (double)stage[q * XC + e0 + RAD - 1]; });
    if (flags) atomicOr(status, flags);
}

// ---------------------------------------------------------------------------
// Tiled y/z sweep: one face per thread, like the x sweep.  A block is a tile
// of TileShape::x x-columns by TileShape::s consecutive faces along the
// sweep axis (in one plane of the third axis); tiles overlap by one face
// along the sweep axis, so each finishes s - 1 cells per column.  Lanes run
// along x, so the staging loads of a wave read whole row segments.  Tiles
// that are neighbours along x or the sweep axis share stencil rows and are
// numbered to run on the same XCD.
// ---------------------------------------------------------------------------
// Tile shape per instance.  Every tile stages its stencils in LDS: the block
// copies U and the primitives of its (s + 2 RAD - 1) x x stencil cells once,
// in whole rows, and every face reads its stencil from there (a face's
// stencil is six rows apart in memory, so unstaged each wave issues twice
// the loads of the x sweep, one per row and field).  The WENO5 tiles
// without the blend are 8 x 32 and exchange their fluxes across lanes
// instead of holding them in LDS (FP64: 46.9 KB per block, three blocks,
// three waves per SIMD, in 146 registers; FP32: 23.5 KB, five waves in 95
// registers); the other instances are 16 x 16 with the fluxes in LDS (FP64:
// 72 KB, two waves; the CU6 and WENO7 faces need more than the 168
// registers of three waves; FP32: 36 KB, four waves).  Measured at 256^3,
// nine species, y/z, the shapes with an earlier face: FP64 WENO5 2.92/3.01 ms
// unstaged, 2.10/2.19 staged at 16 x 16, 1.92/1.97 exchanging at 8 x 32 (CU6 and
// WENO7 ran 5 % slower at 8 x 32 than at 16 x 16); FP32 1.43/1.49 unstaged at
// 32 x 8, 1.15/1.16 staged at 16 x 16, 1.12/1.11 exchanging at 8 x 32.  With the
// present faces, in an RK3 step: FP64 1.79 (y, adding to the sum) and 1.52 (z),
// FP32 1.08/1.09.
template <typename R, int REC, bool PP>
struct TileShape {
    static constexpr bool exchange = REC == kReconWeno5 && !PP;
    static constexpr int x = exchange ? 8 : 16, s = exchange ? 32 : 16;
};

template <int NS, typename R, int DIR, typename S, bool PP, int SPD, int REC, int MODE>
__global__ __launch_bounds__((TileShape<R, REC, PP>::x * TileShape<R, REC, PP>::s)) __attribute__((amdgpu_waves_per_eu(sweep_waves<R, REC, false, PP>()))) void
k_sweep_tile(const S *__restrict__ U, const S *__restrict__ P, R *__restrict__ rhs, Geo g, ThermoK<R> th,
             int accumulate, StageArgs sa, unsigned *status, Dissip ds, FastDiv dgx, FastDiv dgy) {
    constexpr int NV = NS + 4;
    using Shape = TileShape<R, REC, PP>;
    constexpr int kTileX = Shape::x, kTileS = Shape::s;
    constexpr int RAD = stencil_radius(REC);
    constexpr int kRows = kTileS + 2 * RAD - 1;        // stencil rows of the tile's faces
    constexpr int TSZ = kRows * kTileX;                // staged cells
    // EXCH: each flux component goes to the cell below as soon as it is
    // final, the neighbouring face's value taken across lanes (the face
    // below is kTileX lanes down in the same wave); only the first and last
    // face rows of each wave pass theirs through LDS, for the cell between
    // two waves.  Otherwise (the blend, which limits the whole flux vector at
    // once, and the FP32 sweep that finishes a stage, whose face asks for nothing
    // ahead: each component then waited out the latency of its own loads) the
    // fluxes wait in LDS for the block.  A mixed step of nine species without an x
    // axis, exchanging and not: 300 cells 121 and 111 us, 1200 x 1000 4.14 and 3.97
    // ms (five species 91 and 83 us, 2.94 and 2.68 ms).
    constexpr bool EXCH = Shape::exchange && !(sizeof(R) == 4 && MODE == kFinish);
    constexpr int RPW = 64 / kTileX;                   // face rows per wave
    constexpr int NWV = kTileS / RPW;                  // waves per block
    __shared__ R sF[EXCH ? 1 : NV][EXCH ? 1 : kTileS][EXCH ? 1 : kTileX];
    __shared__ R sEdge[2][EXCH ? NWV : 1][EXCH ? NV : 1][EXCH ? kTileX : 1];
    __shared__ S xf_ftile[(NV + 4) * TSZ];
    unsigned bx, by, bz;
    xcd_block(dgx, dgy, bx, by, bz);
    const int tx = threadIdx.x, ts = threadIdx.y;
    const int x = bx * kTileX + tx;
    const int j0 = by * (kTileS - 1);                 // the tile's first face
    const int j = j0 + ts;                            // face j: between cells j-1 and j of the sweep axis
    const int nsw = (DIR == 1) ? g.ny : g.nz;
    const bool valid = x < g.nx && j <= nsw;
    const long long step = (DIR == 1) ? g.sy : g.sz;
    const int gs = (DIR == 1) ? g.gy : g.gz;
    const long long plane = (DIR == 1) ? (long long)(g.gz + bz) * g.sz : (long long)(g.gy + bz) * g.sy;
    const long long col = (long long)(g.gx + x) + plane;
    unsigned flags = 0;
    {
        // tile row r = padded sweep row gs + j0 - RAD + r, for the tile's x
        // columns; rows past the padded extent and columns past the interior
        // are never read
        const int npad = nsw + 2 * gs;
        auto at = [&](int e, long long &cell) {
            const int cx = bx * kTileX + (e % kTileX), row = gs + j0 - RAD + e / kTileX;
            cell = plane + g.gx + cx + (long long)row * step;
            return e < TSZ && cx < g.nx && row < npad;
        };
        stage_cells<NV, kTileX * kTileS, TSZ>(U, P, g.cells, xf_ftile, ts * kTileX + tx, at);
    }
    __syncthreads();
    const R id = R((DIR == 1) ? g.idy : g.idz) * flux_unit<R>();
    const CellOut<R, MODE> co(rhs, sa, accumulate);
    const long long below = col + (long long)(gs + j - 1) * step;   // the cell below the face
    const auto *stage = (const __attribute__((address_space(3))) S *)xf_ftile;
    const int r = ts % RPW, w = ts / RPW;
    if (valid) {
        if constexpr (SPD == kViscFrozen)   // y faces: i + nx (j + (ny + 1) k); z faces: i + nx (j + ny k)
            ds.fidx = DIR == 1 ? x + (long long)g.nx * (j + (long long)(g.ny + 1) * bz)
                               : x + (long long)g.nx * (bz + (long long)g.ny * j);
        // stencil cell m of face j is tile row j - j0 + m
        const StencilLds<NV, S> st{stage, ts * kTileX + tx, kTileX, TSZ};
        if constexpr (EXCH) {
            auto first = [&](int q, R v) { sEdge[1][w][q][tx] = v; };
            auto last = [&](int q, R v) { sEdge[0][w][q][tx] = v; };
            auto uin = [&](int q) { return (double)st.u(q, RAD - 1); };
            ExchangeOut<NS, kTileX, decltype(co), R, decltype(first), decltype(last), decltype(uin)> out{
                co, g.cells, below, id, r > 0, r == RPW - 1, first, last, uin};
            sweep_face<NS, R, DIR, SPD, REC>(st, th, out, flags, ds);
        } else {
            auto out = store_out([&](int q, R v) { sF[q][ts][tx] = v; });
            sweep_face<NS, R, DIR, SPD, REC>(st, th, out, flags, ds);
            if constexpr (PP) {
                R Fq[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) Fq[q] = sF[q][ts][tx] * flux_unit<R>();
                pp_limit<NS, R, DIR, RAD>(st, pp_lambda<R>(g, sa, DIR == 1 ? g.idy : g.idz), Fq);
#pragma unroll
                for (int q = 0; q < NV; ++q) sF[q][ts][tx] = Fq[q] * (R(1) / flux_unit<R>());
            }
        }
    }
    __syncthreads();
    // EXCH: only the cell between the last face row of wave w - 1 and the
    // first of w is left
    const bool left = EXCH ? r == 0 && w > 0 : ts > 0;
    if (valid && left)
        co.template put_all<NV>(
            g.cells, below,
            [&](int q) {
                if constexpr (EXCH)
                    return double((sEdge[0][w - 1][q][tx] - sEdge[1][w][q][tx]) * id);
                else
                    return double((sF[q][ts - 1][tx] - sF[q][ts][tx]) * id);
            },
            [&](int q) { return (double)stage[q * TSZ + (ts + RAD - 1) * kTileX + tx]; });
    if (flags) atomicOr(status, flags);
}

}  // namespace xf
