// xf_misc.hip -- species-independent kernels: boundary ghosts and their
// adjoint, ghost zeroing, SSP-RK3 stage combinations (Eq. 16) and their
// adjoint, CFL finish, copies.
#include <algorithm>

#include "xf_common.hpp"

namespace xf {
namespace {

unsigned blocks_for(long long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

// The ghost cells of the padded grid, enumerated: the z layers with whole
// planes, then the y layers of the interior z, then the x layers of interior
// rows (a row's ghosts in consecutive lanes).
__host__ __device__ __forceinline__ long long ghost_count(const Geo &g) {
    return 2ll * g.gz * g.px * g.py + 2ll * g.gy * g.px * g.nz + 2ll * g.gx * g.ny * g.nz;
}

__device__ __forceinline__ void ghost_cell(const Geo &g, long long q, int &x, int &y, int &z) {
    const long long plane = (long long)g.px * g.py, nz = 2ll * g.gz * plane;
    if (q < nz) {
        const int k = (int)(q / plane);
        const long long r = q - k * plane;
        z = k < g.gz ? k : g.nz + k;
        y = (int)(r / g.px);
        x = (int)(r - (long long)y * g.px);
        return;
    }
    q -= nz;
    const long long slab = (long long)g.px * g.nz, ny = 2ll * g.gy * slab;
    if (q < ny) {
        const int k = (int)(q / slab);
        const long long r = q - k * slab;
        const int j = (int)(r / g.px);
        y = k < g.gy ? k : g.ny + k;
        z = g.gz + j;
        x = (int)(r - (long long)j * g.px);
        return;
    }
    q -= ny;
    const int w = 2 * g.gx;
    const long long r = q / w;
    const int k = (int)(q - r * w), j = (int)(r / g.ny);
    x = k < g.gx ? k : g.nx + k;
    z = g.gz + j;
    y = g.gy + (int)(r - (long long)j * g.ny);
}

// One thread per ghost cell and kFillFields fields.  What bounds the small
// grids is the launch and one chain of loads, so the three axes go in one
// launch: each ghost coordinate maps to its source on its own axis, which is
// what axis-by-axis copies over the full extent of the others give (an edge
// or corner ghost takes the interior cell all its coordinates map to).
// Against a launch per axis: 155 -> 76 us at 256^3, nine species, and 22 ->
// 8 us at 64^3, five species.
constexpr int kFillFields = 4;

__global__ __launch_bounds__(256) void k_fill(double *U, Geo g, int nv) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ghost_count(g)) return;
    int x, y, z;
    ghost_cell(g, q, x, y, z);
    const long long src = ghost_map(x, g.nx, g.gx, g.bc[0], g.bc[1]) +
                          g.sy * ghost_map(y, g.ny, g.gy, g.bc[2], g.bc[3]) +
                          g.sz * ghost_map(z, g.nz, g.gz, g.bc[4], g.bc[5]);
    const long long dst = x + g.sy * y + g.sz * z;
    const int f0 = blockIdx.y * kFillFields;
    double *u = U + f0 * g.cells;
    double v[kFillFields];
#pragma unroll
    for (int f = 0; f < kFillFields; ++f)
        if (f0 + f < nv) v[f] = u[f * g.cells + src];
#pragma unroll
    for (int f = 0; f < kFillFields; ++f)
        if (f0 + f < nv) u[f * g.cells + dst] = v[f];
}

// Zeroes the ghosts of A.
__global__ __launch_bounds__(256) void k_zero_ghosts(double *A, Geo g, int nv) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ghost_count(g)) return;
    int x, y, z;
    ghost_cell(g, q, x, y, z);
    const long long dst = x + g.sy * y + g.sz * z;
    const int f0 = blockIdx.y * kFillFields;
#pragma unroll
    for (int f = 0; f < kFillFields; ++f)
        if (f0 + f < nv) A[(f0 + f) * g.cells + dst] = 0.0;
}

// Adjoint of the fill, as a gather: the interior cells that any ghost copies
// (along each axis the ng cells next to either end) add up their ghost images
// and zero them; every ghost has one source, so the threads are independent.
struct Shell {
    int lo, hi, n;   // cells [0, lo) and [hi, n) of an axis; the others are [lo, hi)
    __host__ __device__ Shell(int n_, int ng) : lo(ng < n_ ? ng : n_), hi(n_ - ng > lo ? n_ - ng : lo), n(n_) {}
    __host__ __device__ int count() const { return lo + n - hi; }
    __host__ __device__ int inner() const { return hi - lo; }
    __host__ __device__ int cell(int k) const { return k < lo ? k : hi + (k - lo); }
};

// What one launch folds: per axis its cells from padded index org on, and the
// ghost layers folded onto them (0: none along this axis).
struct Fold {
    int n[3], ng[3], org[3];
};

__host__ __device__ __forceinline__ long long shell_count(const Fold &g) {
    const Shell x(g.n[0], g.ng[0]), y(g.n[1], g.ng[1]), z(g.n[2], g.ng[2]);
    return (long long)z.count() * g.n[0] * g.n[1] + (long long)z.inner() * ((long long)y.count() * g.n[0] +
           (long long)y.inner() * x.count());
}

// The padded positions along one axis that hold interior cell c or a copy of
// it, as offsets from it: lo, lo + step, ..., count of them (periodic: a period
// apart; outflow: the end cell and the layers outside it).
struct Images {
    int lo, step, count;
    __device__ Images(int c, int n, int ng, int bc) : lo(0), step(1), count(1) {
        if (ng == 0) return;
        const bool below = c >= n - ng, above = c < ng;   // copies below and above it
        if (bc == XF_BC_PERIODIC) {   // periodic sides come in pairs
            lo = below ? -n : 0;
            step = n;
            count = 1 + below + above;
        } else if (c == 0 || c == n - 1) {
            lo = c == 0 ? -ng : 0;
            count = 1 + ng;
        }
    }
};

// One thread per cell with copies and kFillFields fields.  On small grids the
// time is that of the thread with the most copies, one chain of loads: next to an
// outflow side a cell holds all NG layers, NG + 1 values, the square of that at an
// edge and the cube at a corner.  So NG + 1 values (a row of copies; all a face
// cell holds) are asked for at once, without a branch between the loads, the next
// one's address takes additions only, and the launch below folds z apart where
// two axes have outflow sides.  64^3, five species, three layers: periodic 8.3 us,
// outflow 15.6 (the loads one by one, each behind a zero store: 12.0 and 43.4;
// an axis per launch 23.9 and 22.4); 256^3, nine species, outflow: 143 (225, 335).
template <int NG>
__global__ __launch_bounds__(256) void k_fill_vjp(double *Ub, Geo g, Fold fo, int nv) {
    long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= shell_count(fo)) return;
    const Shell sx(fo.n[0], fo.ng[0]), sy(fo.n[1], fo.ng[1]), sz(fo.n[2], fo.ng[2]);
    const int nx = fo.n[0];
    int i, j, k;
    const long long plane = (long long)nx * fo.n[1];
    if (q < sz.count() * plane) {
        const int m = (int)(q / plane);
        const long long r = q - m * plane;
        k = sz.cell(m);
        j = (int)(r / nx);
        i = (int)(r - (long long)j * nx);
    } else {
        q -= sz.count() * plane;
        const long long slab = (long long)sy.count() * nx + (long long)sy.inner() * sx.count();
        const int m = (int)(q / slab);
        long long r = q - m * slab;
        k = sz.lo + m;
        if (r < (long long)sy.count() * nx) {
            const int e = (int)(r / nx);
            j = sy.cell(e);
            i = (int)(r - (long long)e * nx);
        } else {
            r -= (long long)sy.count() * nx;
            const int e = (int)(r / sx.count());
            j = sy.lo + e;
            i = sx.cell((int)(r - (long long)e * sx.count()));
        }
    }
    const Images X(i, nx, fo.ng[0], g.bc[0]), Y(j, fo.n[1], fo.ng[1], g.bc[2]), Z(k, fo.n[2], fo.ng[2], g.bc[4]);
    const int n = X.count * Y.count * Z.count;
    if (n == 1) return;
    const int f0 = blockIdx.y * kFillFields, last = min(kFillFields, nv - f0) - 1;
    double *u = Ub + f0 * g.cells + (fo.org[0] + i) + g.sy * (fo.org[1] + j) + g.sz * (fo.org[2] + k);
    // the image at hand, x fastest: its numbers in x and y and its offset
    const long long o0 = X.lo + g.sy * Y.lo + g.sz * Z.lo;
    const long long dx = X.step, dy = g.sy * Y.step - dx * X.count, dz = g.sz * Z.step - g.sy * Y.step * Y.count;
    int a = 0, b = 0;
    long long o = o0;
    auto next = [&] {
        const bool wx = ++a == X.count;
        a = wx ? 0 : a;
        b += wx;
        const bool wy = b == Y.count;
        b = wy ? 0 : b;
        o += dx + (wx ? dy : 0) + (wy ? dz : 0);
    };
    double v[kFillFields] = {};
    for (int m = 0; m < n; m += NG + 1) {
        // past the last image the cell itself is read, past the last field the
        // last one; neither is added
        double w[NG + 1][kFillFields];
#pragma unroll
        for (int t = 0; t <= NG; ++t) {
            const double *p = u + (m + t < n ? o : 0);
#pragma unroll
            for (int f = 0; f < kFillFields; ++f) w[t][f] = p[min(f, last) * g.cells];
            next();
        }
#pragma unroll
        for (int t = 0; t <= NG; ++t)
#pragma unroll
            for (int f = 0; f < kFillFields; ++f) v[f] += m + t < n ? w[t][f] : 0.0;
    }
    a = b = 0;
    o = o0;
    for (int m = 0; m < n; ++m, next()) {
#pragma unroll
        for (int f = 0; f < kFillFields; ++f)
            if (f <= last) u[f * g.cells + o] = o == 0 ? v[f] : 0.0;
    }
}

// rhs = ((Lz + Ly) + Lx) on the interior cells from FP32 per-direction
// differences (the order in which the FP64 sweeps accumulate).
__global__ __launch_bounds__(256) void k_sum_dirs(double *rhs, const float *Lx, const float *Ly, const float *Lz,
                                                  Geo g, int nv) {
    const long long nint = (long long)g.nx * g.ny * g.nz;
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nint * nv) return;
    const long long f = q / nint, r = q - f * nint;
    int i, j, k;
    split3(g, r, g.nx, g.ny, g.dnx, g.dny, i, j, k);
    const long long o = f * g.cells + (long long)(g.gz + k) * g.sz + (long long)(g.gy + j) * g.sy + (g.gx + i);
    double L = 0.0;
    bool first = true;
    if (Lz) {
        L = (double)Lz[o];
        first = false;
    }
    if (Ly) {
        L = first ? (double)Ly[o] : L + (double)Ly[o];
        first = false;
    }
    if (Lx) L = first ? (double)Lx[o] : L + (double)Lx[o];
    rhs[o] = L;
}

// Adjoint of one stage given the stage cotangent lam (of the stage output)
// and mu = J(V)^T lam (the rhs-VJP at that stage's input V):
//   stage 3 (U = 1/3 V0 + 2/3 (V2 + dt L(V2))): lam0 = lam/3;      lam = 2/3 (lam + dt mu)
//   stage 2 (U = 3/4 V0 + 1/4 (V1 + dt L(V1))): lam0 += 3/4 lam;   lam = 1/4 (lam + dt mu)
//   stage 1 (U = V0 + dt L(V0)):                lam0 += lam + dt mu
__global__ __launch_bounds__(256) void k_rk3_stage_vjp(double *lam, double *lam0, const double *mu, long long n,
                                                       int stage, double dt, const double *dt_dev) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double h = dt_dev ? *dt_dev : dt;
    const double l = lam[q];
    if (stage == 3) {
        lam0[q] = l / 3.0;
        lam[q] = 2.0 / 3.0 * (l + h * mu[q]);
    } else if (stage == 2) {
        lam0[q] += 0.75 * l;
        lam[q] = 0.25 * (l + h * mu[q]);
    } else {
        lam0[q] += l + h * mu[q];
    }
}

__global__ void k_reset_u64(unsigned long long *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

__global__ void k_cfl_finish(const unsigned long long *mx, double cfl, double *dt) {
    *dt = cfl / __longlong_as_double((long long)*mx);
}

__global__ __launch_bounds__(256) void k_copy(long long n, const double *src, double *dst) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) dst[q] = src[q];
}

// Cell-centred velocity gradient G[3 a + b] = d u_b / d x_a by the
// fourth-order difference (u_{-2} - 8 u_{-1} + 8 u_{+1} - u_{+2}) / (12 dx_a)
// at every cell two or more layers inside the padded extent along an active
// axis a (the velocity u_b is Q[2 + b] of the transport pass); the other
// entries are left as they are (no face stencil reads them).
__global__ __launch_bounds__(256) void k_vel_grad(const double *__restrict__ Q, double *__restrict__ G, Geo g) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= g.cells) return;
    const long long C = g.cells;
    int co[3];
    split3(g, idx, g.px, g.py, g.dpx, g.dpy, co[0], co[1], co[2]);
    const int n[3] = {g.nx, g.ny, g.nz}, p[3] = {g.px, g.py, g.pz};
    const long long st[3] = {1, g.sy, g.sz};
    const double ih[3] = {g.idx, g.idy, g.idz};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (n[a] <= 1 || co[a] < 2 || co[a] >= p[a] - 2) continue;
        const long long s = st[a];
        const double f = ih[a] * (1.0 / 12.0);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const double *u = Q + (2 + b) * C + idx;
            G[(3 * a + b) * C + idx] = (u[-2 * s] - 8.0 * u[-s] + 8.0 * u[s] - u[2 * s]) * f;
        }
    }
}

__global__ __launch_bounds__(256) void k_zero(long long n, double *dst) {
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < n) dst[q] = 0.0;
}

}  // namespace

unsigned field_groups(int nv) { return (unsigned)((nv + kFillFields - 1) / kFillFields); }

hipError_t launch_fill_ghosts(const LaunchCtx &c, int nv, double *U, hipStream_t s) {
    hipLaunchKernelGGL(k_fill, dim3(blocks_for(ghost_count(c.g), 256), field_groups(nv)), dim3(256), 0, s, U, c.g,
                       nv);
    return hipGetLastError();
}

hipError_t launch_fill_ghosts_vjp(const LaunchCtx &c, int nv, double *Ub, hipStream_t s) {
    const Geo &g = c.g;
    const int n[3] = {g.nx, g.ny, g.nz}, ng[3] = {g.gx, g.gy, g.gz}, p[3] = {g.px, g.py, g.pz};
    // folds the axes of a bit set, onto the padded extent of those left for a
    // later launch
    auto fold = [&](int axes, int later) {
        Fold f;
        for (int d = 0; d < 3; ++d) {
            const bool whole = later >> d & 1;
            f.n[d] = whole ? p[d] : n[d];
            f.ng[d] = axes >> d & 1 ? ng[d] : 0;
            f.org[d] = whole ? 0 : ng[d];
        }
        const dim3 grid(blocks_for(shell_count(f), 256), field_groups(nv));
        if (std::max(std::max(ng[0], ng[1]), ng[2]) <= 3)
            hipLaunchKernelGGL(k_fill_vjp<3>, grid, dim3(256), 0, s, Ub, g, f, nv);
        else
            hipLaunchKernelGGL(k_fill_vjp<4>, grid, dim3(256), 0, s, Ub, g, f, nv);
        return hipGetLastError();
    };
    // two or three axes with outflow sides: z first, in a launch of its own (one
    // launch for all: 64^3 with two, three layers 16.2 against 10.9 us, four layers
    // 23.2 against 12.4)
    int outflow = 0;
    for (int d = 0; d < 3; ++d) outflow += ng[d] > 0 && g.bc[2 * d] != XF_BC_PERIODIC;
    if (outflow < 2 || ng[2] == 0 || ng[0] * ng[1] == 0) return fold(7, 0);
    const hipError_t e = fold(4, 3);
    return e == hipSuccess ? fold(3, 0) : e;
}

hipError_t launch_zero_ghosts(const LaunchCtx &c, int nv, double *A, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_ghosts, dim3(blocks_for(ghost_count(c.g), 256), field_groups(nv)), dim3(256), 0, s, A, c.g,
                       nv);
    return hipGetLastError();
}

hipError_t launch_rk3_stage_vjp(const LaunchCtx &c, int nv, int stage, double *lam, double *lam0, double *mu,
                                const double *dt_dev, double dt, hipStream_t s) {
    const long long n = c.g.cells * nv;
    hipLaunchKernelGGL(k_rk3_stage_vjp, dim3(blocks_for(n, 256)), dim3(256), 0, s, lam, lam0, mu, n, stage, dt,
                       dt_dev);
    return hipGetLastError();
}

hipError_t launch_sum_dirs(const LaunchCtx &c, int nv, double *rhs, const float *const L[3], hipStream_t s) {
    const long long n = (long long)c.g.nx * c.g.ny * c.g.nz * nv;
    hipLaunchKernelGGL(k_sum_dirs, dim3(blocks_for(n, 256)), dim3(256), 0, s, rhs, L[0], L[1], L[2], c.g, nv);
    return hipGetLastError();
}

hipError_t launch_vel_grad(const LaunchCtx &c, const double *Q, double *G, hipStream_t s) {
    hipLaunchKernelGGL(k_vel_grad, dim3(blocks_for(c.g.cells, 256)), dim3(256), 0, s, Q, G, c.g);
    return hipGetLastError();
}

hipError_t launch_reset_u64(unsigned long long *p, int n, hipStream_t s) {
    if (n < 1 || n > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_reset_u64, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_cfl_finish(const unsigned long long *mx, double cfl, double *dt_dev, hipStream_t s) {
    hipLaunchKernelGGL(k_cfl_finish, dim3(1), dim3(1), 0, s, mx, cfl, dt_dev);
    return hipGetLastError();
}

hipError_t launch_copy(long long n, const double *src, double *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_copy, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, src, dst);
    return hipGetLastError();
}

hipError_t launch_zero(long long n, double *dst, hipStream_t s) {
    hipLaunchKernelGGL(k_zero, dim3(blocks_for(n, 256)), dim3(256), 0, s, n, dst);
    return hipGetLastError();
}

}  // namespace xf
