// xf_few32.hpp -- FP32 sweeps of contexts with one or two species.
//
// With so few species the compiler takes the species loops of the FP32 face
// apart and pairs its multiply-adds across them, differently with every
// change of the code around the face; another pairing is another rounding,
// and the state moves in the eighth digit.  These contexts keep the sweeps and the
// separate stage kernel whose results they have always had.  From three
// species on the loops stay loops, the face rounds alike in every kernel, and
// the sweeps of xf_forward.hpp serve both precisions (1.12 -> 1.07 ms per y/z
// sweep and 2.22 -> 1.61 ms for the finishing x sweep at 256^3, nine species).
#pragma once

#include "xf_forward.hpp"

namespace xf {

// Contexts served here.
template <int NS, typename R>
constexpr bool few32() { return sizeof(R) == 4 && NS <= 2; }

// SSP-RK3 stage of Eq. 16 on the interior cells: Uout = a U0 + b (Uin + h L),
// L = ((Lx + Ly) + Lz) + Lv; a block takes one interior row of one field.
template <int NS>
__global__ __launch_bounds__(256) void k_few32_stage(double *Uout, const double *U0, const double *Uin, const float *Lx,
                                                     const float *Ly, const float *Lz, const double *Lv, Geo g, double a,
                                                   double b, double dt, const double *dt_dev) {
    const int row = blockIdx.x;
    const int j = row % g.ny, k = row / g.ny;
    const long long base = (long long)blockIdx.y * g.cells + (long long)(g.gz + k) * g.sz +
                           (long long)(g.gy + j) * g.sy + g.gx;
    const double h = dt_dev ? *dt_dev : dt;
    for (int i = threadIdx.x; i < g.nx; i += blockDim.x) {
        const long long o = base + i;
        double L = 0.0;
        if (Lx) L = (double)Lx[o];
        if (Ly) L = L + (double)Ly[o];
        if (Lz) L = L + (double)Lz[o];
        if (Lv) L = L + Lv[o];
        const double v = Uin[o] + h * L;
        Uout[o] = a == 0.0 ? b * v : a * U0[o] + b * v;
    }
}

// x sweep (as k_sweep_x, the fluxes in LDS): one thread per face.
template <int NS, bool PP, int SPD, int REC>
__global__ __launch_bounds__(kXBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_few32_x(
    const float *__restrict__ U, const float *__restrict__ P, float *__restrict__ rhs, Geo g, ThermoK<float> th,
    StageArgs sa, unsigned *status, Dissip ds, int fpb) {
    using R = float;
    using S = float;
    constexpr int NV = NS + 4;
    constexpr int RAD = stencil_radius(REC);
    constexpr int GAP = 2 * RAD - 1;
    constexpr int XC = x_stage_cells<RAD>();
    __shared__ R sF[NV][kXBlock];
    __shared__ S xf_xstage[(NV + 4) * XC];
    unsigned lb, u1, u2;
    xcd_block(lb, u1, u2);
    const int t = threadIdx.x;
    const long long nfx = (long long)g.nx + 1;
    const long long nfaces = nfx * g.ny * g.nz;
    const long long f0 = (long long)lb * (fpb - 1);
    if (f0 >= nfaces) return;   // blocks that round the grid up to a multiple of 8
    const long long flast = min(f0 + fpb - 1, nfaces - 1);
    // the block's first face: face i0 of row row0 = (j0, k0); its faces lie
    // in rows row0 .. row0 + nseg - 1 (segment sg = row row0 + sg), so the
    // per-cell and per-face indexing below needs 32-bit divisions only
    const long long row0 = f0 / nfx;
    const int i0 = (int)(f0 - row0 * nfx);
    const int j0 = (int)(row0 % g.ny);
    const long long k0 = row0 / g.ny;
    const int nfx32 = g.nx + 1;
    auto row_base = [&](int sg) {
        int j = j0 + sg;
        long long k = k0;
        if (j >= g.ny) {
            k += j / g.ny;
            j %= g.ny;
        }
        return (g.gz + k) * g.sz + (long long)(g.gy + j) * g.sy + g.gx;
    };
    {
        // staged cell e: segment sg = (e + i0) / W, W = nfx + GAP, x index
        // e + i0 - sg W - RAD of that row (segment 0 starts at face i0, the
        // others at face 0)
        const int nseg = (int)(flast / nfx - row0) + 1;
        const int ncell = (int)(flast - f0 + 1) + nseg * GAP;
        const int W = nfx32 + GAP;
        for (int e = t; e < ncell; e += kXBlock) {
            const int sg = (e + i0) / W;
            const int cx = e + i0 - sg * W - RAD;
            const long long cell = row_base(sg) + cx;
#pragma unroll
            for (int q = 0; q < NV; ++q) xf_xstage[q * XC + e] = U[q * g.cells + cell];
#pragma unroll
            for (int q = 0; q < 4; ++q) xf_xstage[(NV + q) * XC + e] = P[q * g.cells + cell];
        }
    }
    __syncthreads();
    const long long f = f0 + t;
    const bool valid = t < fpb && f < nfaces;
    int i = 0;
    unsigned flags = 0;
    long long rowbase = 0;
    const R id = R(g.idx);
    // the result of interior cell `cell` from its flux difference L (x part); a
    // stage with the blend or viscous fluxes is left to k_few32_stage
    auto emit = [&](int q, long long cell, double L) {
        const long long o = q * g.cells + cell;
        if (!PP && sa.Uout) {
            const double h = sa.dt_dev ? *sa.dt_dev : sa.dt;
            if (sa.Ly32) L = L + (double)sa.Ly32[o];
            if (sa.Lz32) L = L + (double)sa.Lz32[o];
            const double v = sa.Uin[o] + h * L;
            sa.Uout[o] = sa.a == 0.0 ? sa.b * v : sa.a * sa.U0[o] + sa.b * v;
        } else {
            rhs[o] = R(L);
        }
    };
    if (valid) {
        const int sg = (t + i0) / nfx32;
        i = t + i0 - sg * nfx32;
        rowbase = row_base(sg);
        // stencil cell m of face i (cell i - RAD + m of its row) is staged at
        // t + sg GAP + m
        StencilLds<NV, S> st{(const __attribute__((address_space(3))) S *)xf_xstage, t + sg * GAP, 1, XC};
        if constexpr (SPD == kViscFrozen) ds.fidx = f;   // x faces: i + (nx + 1) (j + ny k)
        auto out = store_out([&](int q, R v) { sF[q][t] = v; });
        face_flux_to<NS, R, 0, SPD, REC>(st, th, out, flags, ds);
        if constexpr (PP) {
            R Fq[NV];
#pragma unroll
            for (int q = 0; q < NV; ++q) Fq[q] = sF[q][t];
            pp_limit<NS, R, 0, RAD>(st, pp_lambda<R>(g, sa, g.idx), Fq);
#pragma unroll
            for (int q = 0; q < NV; ++q) sF[q][t] = Fq[q];
        }
    }
    __syncthreads();
    if (valid && t > 0 && i > 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) emit(q, rowbase + i - 1, double((sF[q][t - 1] - sF[q][t]) * id));
    }
    if (flags) atomicOr(status, flags);
}

// y/z sweep (as k_sweep_tile).
template <int NS, int DIR, bool PP, int SPD, int REC>
__global__ __launch_bounds__((TileShape<float, REC, PP>::x * TileShape<float, REC, PP>::s)) __attribute__((amdgpu_waves_per_eu(1))) void
k_few32_tile(const float *__restrict__ U, const float *__restrict__ P, float *__restrict__ rhs, Geo g, ThermoK<float> th,
             StageArgs sa, unsigned *status, Dissip ds) {
    using R = float;
    using S = float;
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
    // two waves.  Otherwise (the blend, which limits the whole flux vector
    // at once) the fluxes wait in LDS for the block.
    constexpr bool EXCH = Shape::exchange;
    constexpr int RPW = 64 / kTileX;                   // face rows per wave
    constexpr int NWV = kTileS / RPW;                  // waves per block
    __shared__ R sF[EXCH ? 1 : NV][EXCH ? 1 : kTileS][EXCH ? 1 : kTileX];
    __shared__ R sEdge[2][EXCH ? NWV : 1][EXCH ? NV : 1][EXCH ? kTileX : 1];
    __shared__ S xf_ftile[(NV + 4) * TSZ];
    unsigned bx, by, bz;
    xcd_block(bx, by, bz);
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
        for (int e = ts * kTileX + tx; e < TSZ; e += kTileX * kTileS) {
            const int r = e / kTileX, cx = bx * kTileX + (e % kTileX);
            const int row = gs + j0 - RAD + r;
            if (cx >= g.nx || row >= npad) continue;
            const long long cell = plane + g.gx + cx + (long long)row * step;
#pragma unroll
            for (int q = 0; q < NV; ++q) xf_ftile[q * TSZ + e] = U[q * g.cells + cell];
#pragma unroll
            for (int k = 0; k < 4; ++k) xf_ftile[(NV + k) * TSZ + e] = P[k * g.cells + cell];
        }
        __syncthreads();
    }
    if (valid) {
        if constexpr (SPD == kViscFrozen)   // y faces: i + nx (j + (ny + 1) k); z faces: i + nx (j + ny k)
            ds.fidx = DIR == 1 ? x + (long long)g.nx * (j + (long long)(g.ny + 1) * bz)
                               : x + (long long)g.nx * (bz + (long long)g.ny * j);
        auto face = [&](const auto &st) {
            if constexpr (EXCH) {
                const R id = R((DIR == 1) ? g.idy : g.idz);
                const int r = ts % RPW, w = ts / RPW;
                const long long below = col + (long long)(gs + j - 1) * step;
                auto out = store_out([&](int q, R v) {
                        // face j - 1 of this column, valid wherever face j is
                        const R vb = __shfl_up(v, kTileX);
                        if (r > 0) rhs[q * g.cells + below] = (vb - v) * id;
                        if (r == RPW - 1) sEdge[0][w][q][tx] = v;
                        if (r == 0) sEdge[1][w][q][tx] = v;
                });
                face_flux_to<NS, R, DIR, SPD, REC>(st, th, out, flags, ds);
                return;
            }
            auto out = store_out([&](int q, R v) { sF[q][ts][tx] = v; });
            face_flux_to<NS, R, DIR, SPD, REC>(st, th, out, flags, ds);
            if constexpr (PP) {
                R Fq[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) Fq[q] = sF[q][ts][tx];
                pp_limit<NS, R, DIR, RAD>(st, pp_lambda<R>(g, sa, DIR == 1 ? g.idy : g.idz), Fq);
#pragma unroll
                for (int q = 0; q < NV; ++q) sF[q][ts][tx] = Fq[q];
            }
        };
        // stencil cell m of face j is tile row j - j0 + m
        face(StencilLds<NV, S>{(const __attribute__((address_space(3))) S *)xf_ftile, ts * kTileX + tx, kTileX, TSZ});
    }
    __syncthreads();
    if constexpr (EXCH) {
        // the cell between the last face row of wave w - 1 and the first of w
        const int r = ts % RPW, w = ts / RPW;
        if (valid && r == 0 && w > 0) {
            const R id = R((DIR == 1) ? g.idy : g.idz);
            const long long cell = col + (long long)(gs + j - 1) * step;
#pragma unroll
            for (int q = 0; q < NV; ++q)
                rhs[q * g.cells + cell] = (sEdge[0][w - 1][q][tx] - sEdge[1][w][q][tx]) * id;
        }
    } else if (valid && ts > 0) {
        const R id = R((DIR == 1) ? g.idy : g.idz);
        const long long cell = col + (long long)(gs + j - 1) * step;
#pragma unroll
        for (int q = 0; q < NV; ++q)
            rhs[q * g.cells + cell] = (sF[q][ts - 1][tx] - sF[q][ts][tx]) * id;
    }
    if (flags) atomicOr(status, flags);
}

}  // namespace xf
