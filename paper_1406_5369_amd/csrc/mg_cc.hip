// Cell-centred grids with a homogeneous Neumann boundary (Table 1: cell-
// centred discretisation, Neumann boundary condition, constant interpolation;
// the boundary of the complex-diffusion application of Section 4).
//
// n = 2^L cells per axis, h = 1/n, one FP64 value per cell (no ghost cells),
// x fastest.  Zero flux through the boundary: a neighbour outside the domain
// takes the cell's own value, so
//   (A u)_p = c (2d u_p - s),  s = ((uW+uE)+(uS+uN))[+(uB+uT)] with ghosts,
// relaxation u + wd[m] r with wd[m] = omega h^2 / (2d - m) (m = faces of the
// cell on the boundary: omega over the true diagonal), restriction by the
// average of the 2^d children, constant interpolation, a single-cell
// coarsest level (zero correction).  The operator is singular: the solve
// projects f onto mean zero and keeps the iterate at mean zero, with sums in
// a fixed order (each x-row left to right, the rows of a plane, the planes).
//
// A solve runs the same driver as the node-based path.  3D red-black sweeps
// are those of mg_smooth3d_rb.inl; here are the 2D ones (an LDS tile per
// workgroup, both colours), the Jacobi sweeps, the transfers, the fixed-order
// sums and the coarse tail.  The cycle's result is not projected in a pass of
// its own: the next cycle's first sweep subtracts the mean as it loads u, and
// sums the residual norm; u itself is projected once, after the last cycle.
#include <algorithm>
#include <cstring>

#include "mg_cc.h"
#include "mg_kern.h"

namespace mg {
namespace {

template <int DIM>
__device__ __forceinline__ double cc_apply(const MG_GLOBAL double* u, int n, double c, int i, int j, int k,
                                           size_t p) {
    const double uC = u[p];
    const double uW = i > 0 ? u[p - 1] : uC, uE = i < n - 1 ? u[p + 1] : uC;
    const double uS = j > 0 ? u[p - n] : uC, uN = j < n - 1 ? u[p + n] : uC;
    if constexpr (DIM == 2) {
        return c * (4.0 * uC - ((uW + uE) + (uS + uN)));
    } else {
        const size_t sz = (size_t)n * n;
        const double uB = k > 0 ? u[p - sz] : uC, uT = k < n - 1 ? u[p + sz] : uC;
        return c * (6.0 * uC - (((uW + uE) + (uS + uN)) + (uB + uT)));
    }
}

template <int DIM>
__device__ __forceinline__ void cc_ijk(size_t p, int n, int& i, int& j, int& k) {
    i = (int)(p % (size_t)n);
    const size_t q = p / (size_t)n;
    j = (int)(q % (size_t)n);
    k = DIM == 2 ? 0 : (int)(q / (size_t)n);
}

// RBGS colour (in place; a colour reads only the other colour) or Jacobi
// (out of place) relaxation of every cell of one level.
template <int DIM, bool JAC>
__global__ __launch_bounds__(NT) void k_cc_relax(const double* uin_, double* uout_,
                                                 const double* __restrict__ f_, CCConst L, int colour) {
    const MG_GLOBAL double* uin = gp(uin_);
    MG_GLOBAL double* uout = gp(uout_);
    const MG_GLOBAL double* __restrict__ f = gp(f_);
    const int n = L.n;
    const size_t N = DIM == 2 ? (size_t)n * n : (size_t)n * n * n;
    const size_t p = (size_t)blockIdx.x * NT + threadIdx.x;
    if (p >= N) return;
    int i, j, k;
    cc_ijk<DIM>(p, n, i, j, k);
    if (!JAC && ((i + j + k) & 1) != colour) return;
    int m = (i == 0) + (i == n - 1) + (j == 0) + (j == n - 1);
    if (DIM == 3) m += (k == 0) + (k == n - 1);
    const double r = f[p] - cc_apply<DIM>(uin, n, L.c, i, j, k, p);
    uout[p] = uin[p] + L.wd[m] * r;
}

// fc = average of the residuals of the 2^d children of each coarse cell
template <int DIM>
__device__ __forceinline__ void cc_restrict_cell(const MG_GLOBAL double* __restrict__ u,
                                                 const MG_GLOBAL double* __restrict__ f,
                                                 MG_GLOBAL double* __restrict__ fc, int n, double c) {
    const int nc = n / 2;
    const size_t Nc = DIM == 2 ? (size_t)nc * nc : (size_t)nc * nc * nc;
    const size_t q = (size_t)blockIdx.x * NT + threadIdx.x;
    if (q >= Nc) return;
    int I, J, K;
    cc_ijk<DIM>(q, nc, I, J, K);
    auto res = [&](int i, int j, int k) {
        const size_t p = ((size_t)k * n + j) * n + i;
        return f[p] - cc_apply<DIM>(u, n, c, i, j, k, p);
    };
    const int i = 2 * I, j = 2 * J, k = 2 * K;
    const double q0 = (res(i, j, k) + res(i + 1, j, k)) + (res(i, j + 1, k) + res(i + 1, j + 1, k));
    double v;
    if constexpr (DIM == 2) {
        v = 0.25 * q0;
    } else {
        const double q1 = (res(i, j, k + 1) + res(i + 1, j, k + 1)) + (res(i, j + 1, k + 1) + res(i + 1, j + 1, k + 1));
        v = 0.125 * (q0 + q1);
    }
    fc[q] = v;
}
template <int DIM>
__global__ __launch_bounds__(NT) void k_cc_restrict(const double* __restrict__ u, const double* __restrict__ f,
                                                    double* __restrict__ fc, CCConst L) {
    cc_restrict_cell<DIM>(gp(u), gp(f), gp(fc), L.n, L.c);
}

// u += e(parent) (constant interpolation)
template <int DIM>
__device__ __forceinline__ void cc_prolong_cell(MG_GLOBAL double* __restrict__ u,
                                                const MG_GLOBAL double* __restrict__ ec, int n) {
    const size_t N = DIM == 2 ? (size_t)n * n : (size_t)n * n * n;
    const size_t p = (size_t)blockIdx.x * NT + threadIdx.x;
    if (p >= N) return;
    int i, j, k;
    cc_ijk<DIM>(p, n, i, j, k);
    const int nc = n / 2;
    const size_t q = ((size_t)(k / 2) * nc + j / 2) * nc + i / 2;
    u[p] = u[p] + ec[q];
}
template <int DIM>
__global__ __launch_bounds__(NT) void k_cc_prolong(double* __restrict__ u, const double* __restrict__ ec, int n) {
    cc_prolong_cell<DIM>(gp(u), gp(ec), n);
}

// Sums in the fixed order: out[t] = (sum over x of row t, left to right) *
// scale^-1 (scale 0: the sum), rows of n values.  A workgroup takes as many
// rows as fit in LDS, loads them whole (coalesced, every load in flight), and
// one thread per row adds them up.  What bounds it is the chain of n dependent
// additions; one thread per row reading device memory took 18.4 us for the
// rows of 128^3 cells, 13.1 us for its planes.
constexpr int kRowLds = 4352;  // doubles: 32 rows of 128 (+ 1 each), 4 of 1024
__host__ __device__ inline int cc_rows_per_block(int n) {
    const int r = 4096 / n;
    return r < 1 ? 1 : (r > 32 ? 32 : r);
}
__global__ __launch_bounds__(NT) void k_cc_rows(const double* __restrict__ v_, const GridDesc* __restrict__ desc,
                                                int n, int nrows, double scale, double* __restrict__ out) {
    __shared__ double L[kRowLds];
    if (desc && desc->done && *gp(desc->done)) return;
    const int per = cc_rows_per_block(n), r0 = blockIdx.x * per, cnt = min(per, nrows - r0);
    const MG_GLOBAL double* __restrict__ v = gp(v_ ? v_ : (const double*)desc->u) + (size_t)r0 * n;
    double s = 0.0;
    for (int c0 = 0; c0 < n; c0 += 4096) {  // whole rows up to 4096 values, longer ones in parts
        const int w = min(n - c0, 4096);
        if (c0) __syncthreads();
        if (w == n) {
#pragma unroll 8
            for (int q = threadIdx.x; q < cnt * n; q += NT) L[q + q / n] = v[q];
        } else {
#pragma unroll 8
            for (int q = threadIdx.x; q < w; q += NT) L[q] = v[c0 + q];
        }
        __syncthreads();
        if ((int)threadIdx.x < cnt) {
            const double* row = L + threadIdx.x * (n + 1);
#pragma unroll 8
            for (int i = 0; i < w; ++i) s += row[i];
        }
    }
    if ((int)threadIdx.x < cnt) gp(out)[r0 + threadIdx.x] = scale != 0.0 ? s / scale : s;
}
__global__ __launch_bounds__(NT) void k_cc_sub(double* __restrict__ v_, const GridDesc* __restrict__ desc, size_t N,
                                               const double* __restrict__ mean) {
    if (desc && desc->done && *gp(desc->done)) return;
    const size_t p = (size_t)blockIdx.x * NT + threadIdx.x;
    if (p >= N) return;
    MG_GLOBAL double* v = gp(v_ ? v_ : (double*)desc->u);
    v[p] = v[p] - *gp(mean);
}

// per-block partial sums of r^2 (the residual norm; any summation order)
template <int DIM>
__global__ __launch_bounds__(NT) void k_cc_norm(const GridDesc* __restrict__ desc, const double* __restrict__ u_,
                                                const double* __restrict__ f_, double* __restrict__ part) {
    __shared__ double red4[4];
    const GridDesc& d = *desc;
    const MG_GLOBAL double* __restrict__ u = gp(u_ ? u_ : (const double*)d.u);
    const MG_GLOBAL double* __restrict__ f = gp(f_ ? f_ : (const double*)d.f);
    const int n = d.n;
    const size_t N = DIM == 2 ? (size_t)n * n : (size_t)n * n * n;
    const size_t p = (size_t)blockIdx.x * NT + threadIdx.x;
    double acc = 0.0;
    if (p < N) {
        int i, j, k;
        cc_ijk<DIM>(p, n, i, j, k);
        const double r = f[p] - cc_apply<DIM>(u, n, d.c, i, j, k, p);
        acc = r * r;
    }
    const double s = block_sum(acc, red4);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// ---------------------------------------------------------------------------
// Sweeps, restriction and correction of a level given by its descriptor.
// ---------------------------------------------------------------------------

// The incoming iterate at cell (i, j[, k]) of a sweep: u, zero, u + the
// parent's correction, or u - mean.
template <int DIM, int FL>
struct CCIn {
    const MG_GLOBAL double* __restrict__ u;
    const MG_GLOBAL double* __restrict__ ec;
    int n;
    double mean;
    __device__ __forceinline__ CCIn(const GridDesc& d, int sel)
        : u(gp((const double*)((sel & 1) ? d.t : d.u))), ec(gp((const double*)d.uc)), n(d.n), mean(0.0) {
        if constexpr ((FL & SWEEP_NORM) != 0) mean = *gp(d.mean);
    }
    __device__ __forceinline__ double operator()(int i, int j, int k) const {
        if constexpr ((FL & SWEEP_ZERO_GUESS) != 0) return 0.0;
        const size_t p = ((size_t)k * n + j) * n + i;
        double v = u[p];
        if constexpr ((FL & SWEEP_PROLONG) != 0) {
            const int nc = n >> 1;
            v = v + ec[((size_t)(k >> 1) * nc + (j >> 1)) * nc + (i >> 1)];
        }
        if constexpr ((FL & SWEEP_NORM) != 0) v = v - mean;
        return v;
    }
};

// 2D red-black sweep: one 64 x BY LDS box per workgroup; the first colour on
// the tile plus one ring, the second on the tile, written to the partner.
template <int BY, int FL>
__global__ __launch_bounds__(NT) void k_cc_sweep2d(const GridDesc* __restrict__ descs, int sel) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    constexpr bool NRM = (FL & SWEEP_NORM) != 0;
    constexpr int H = 2, TX = BX - 2 * H, TY = BY - 2 * H, RPT = BY / 4;
    __shared__ double U[BY][BX];
    const int n = d.n, ntx = (n + TX - 1) / TX;
    const int tile = sweep_tile(sel, blockIdx.x, gridDim.x);
    const int x0 = (tile % ntx) * TX, y0 = (tile / ntx) * TY;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int gx = x0 - H + lane, cfirst = (sel & SEL_BLACK_FIRST) ? 1 : 0;
    const CCIn<2, FL> in(d, sel);
    const MG_GLOBAL double* __restrict__ f = gp((const double*)d.f);
    MG_GLOBAL double* __restrict__ uout = gp((double*)((sel & 1) ? d.u : d.t));
    const double c = d.c;
    const bool colg = gx >= 0 && gx < n;
    const int mx = (gx == 0) + (gx == n - 1);
    double fr[RPT];
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
        const int ly = w + 4 * m, gy = y0 - H + ly;
        const int xc = min(max(gx, 0), n - 1), yc = min(max(gy, 0), n - 1);
        U[ly][lane] = in(xc, yc, 0);
        fr[m] = f[(size_t)yc * n + xc];
    }
    __syncthreads();
    auto res = [&](int ly, int gy, double fv) {
        const double uC = U[ly][lane];
        const double uW = gx > 0 ? U[ly][lane - 1] : uC, uE = gx < n - 1 ? U[ly][lane + 1] : uC;
        const double uS = gy > 0 ? U[ly - 1][lane] : uC, uN = gy < n - 1 ? U[ly + 1][lane] : uC;
        return fv - c * (4.0 * uC - ((uW + uE) + (uS + uN)));
    };
    auto in_tile = [&](int ly, int gy) {
        return colg && gy < n && lane >= H && lane <= BX - 1 - H && ly >= H && ly <= BY - 1 - H;
    };
    double acc = 0.0;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        double v[RPT];
        const int q = 1 + half;  // rings left out
#pragma unroll
        for (int m = 0; m < RPT; ++m) {
            const int ly = w + 4 * m, gy = y0 - H + ly;
            const bool on = colg && gy >= 0 && gy < n && lane >= q && lane <= BX - 1 - q && ly >= q && ly <= BY - 1 - q;
            v[m] = U[ly][lane];
            if (on) {
                const bool mine = ((gx + gy) & 1) == (cfirst ^ half);
                if (mine || (NRM && half == 0)) {
                    const double r = res(ly, gy, fr[m]);
                    if constexpr (NRM) {
                        if (half == 0 && in_tile(ly, gy)) acc += r * r;
                    }
                    if (mine) v[m] = v[m] + d.sc[mx + (gy == 0) + (gy == n - 1)] * r;
                }
            }
        }
        if (half == 0) {
            __syncthreads();
#pragma unroll
            for (int m = 0; m < RPT; ++m) U[w + 4 * m][lane] = v[m];
            __syncthreads();
        } else {
#pragma unroll
            for (int m = 0; m < RPT; ++m) {
                const int ly = w + 4 * m, gy = y0 - H + ly;
                if (in_tile(ly, gy)) uout[(size_t)gy * n + gx] = v[m];
            }
        }
    }
    if constexpr (NRM) {
        __shared__ double red4[4];
        const double tot = block_sum(acc, red4);
        if (threadIdx.x == 0) gp(d.npart)[blockIdx.x] = tot;
    }
}

// Jacobi sweep, one cell per thread (a colour choice would idle no lane).
template <int DIM, int FL>
__global__ __launch_bounds__(NT) void k_cc_jacobi(const GridDesc* __restrict__ descs, int sel) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    constexpr bool NRM = (FL & SWEEP_NORM) != 0;
    const int n = d.n;
    const size_t N = DIM == 2 ? (size_t)n * n : (size_t)n * n * n;
    const size_t p = (size_t)blockIdx.x * NT + threadIdx.x;
    double acc = 0.0;
    if (p < N) {
        int i, j, k;
        cc_ijk<DIM>(p, n, i, j, k);
        const CCIn<DIM, FL> in(d, sel);
        const double uC = in(i, j, k);
        int m = (i == 0) + (i == n - 1) + (j == 0) + (j == n - 1);
        double s = ((i > 0 ? in(i - 1, j, k) : uC) + (i < n - 1 ? in(i + 1, j, k) : uC)) +
                   ((j > 0 ? in(i, j - 1, k) : uC) + (j < n - 1 ? in(i, j + 1, k) : uC));
        if constexpr (DIM == 3) {
            m += (k == 0) + (k == n - 1);
            s = s + ((k > 0 ? in(i, j, k - 1) : uC) + (k < n - 1 ? in(i, j, k + 1) : uC));
        }
        const double r = gp((const double*)d.f)[p] - d.c * ((DIM == 2 ? 4.0 : 6.0) * uC - s);
        if constexpr (NRM) acc = r * r;
        gp((double*)((sel & 1) ? d.u : d.t))[p] = uC + d.sc[m] * r;
    }
    if constexpr (NRM) {
        __shared__ double red4[4];
        const double tot = block_sum(acc, red4);
        if (threadIdx.x == 0) gp(d.npart)[blockIdx.x] = tot;
    }
}

template <int DIM>
__global__ __launch_bounds__(NT) void k_cc_restrict_d(const GridDesc* __restrict__ descs, int sel) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    cc_restrict_cell<DIM>(gp((const double*)(sel ? d.t : d.u)), gp((const double*)d.f), gp((double*)d.fc), d.n, d.c);
}
template <int DIM>
__global__ __launch_bounds__(NT) void k_cc_prolong_d(const GridDesc* __restrict__ descs, int sel) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    cc_prolong_cell<DIM>(gp((double*)(sel ? d.t : d.u)), gp((const double*)d.uc), d.n);
}

// ---------------------------------------------------------------------------
// Coarse tail: every level from 2^C cells per axis (C up to 6 in 2D, 4 in 3D)
// down to one cell in one launch, one workgroup, all fields in LDS (as k_tail
// of the node-based path, whose comment says what bounds it).  16^3 cells and
// below: 22.8 us a V(2,2) visit.  There is no
// boundary layer, so a half-sweep's items are exactly the colour's cells.  The
// single cell's operator is zero, so is its correction.
// ---------------------------------------------------------------------------
constexpr int CTN = 1024;
__host__ __device__ constexpr int ct_cells(int dim, int C) { return 1 << (dim * C); }
__host__ __device__ constexpr int ct_off(int dim, int C) {
    int s = 0;
    for (int c = 0; c < C; ++c) s += ct_cells(dim, c);
    return s;
}
__host__ __device__ constexpr int ct_wave_level(int dim) { return dim == 2 ? 4 : 2; }

struct CTail {
    double *U, *F, *W;  // iterates and right-hand sides of all levels, residual of the level at hand
    const double* wd;   // level C: wd[m] at 4 C + m
    double c[7];
    int nu1, nu2, post_first;
};

template <bool WAVE>
__device__ __forceinline__ void ct_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// The thread's number, opaque to the compiler: a step's cell coordinates are
// then formed in the step (kept from step to step for every level they spill).
__device__ __forceinline__ int ct_tid() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

template <int DIM, bool JAC, int C>
struct CTLevel {
    static constexpr int M = 1 << C, OFF = ct_off(DIM, C), CELLS = ct_cells(DIM, C);
    static constexpr bool WAVE = C <= ct_wave_level(DIM);
    static constexpr int NTH = WAVE ? 64 : CTN;

    static __device__ __forceinline__ int at(int i, int j, int k) { return ((k << C) + j) * M + i; }
    // Residual at cell (i, j, k) whose own value is uC (a neighbour outside the
    // domain takes it too); m: its boundary faces.  Loads are unconditional
    // (from the cell itself where there is no neighbour), so they all issue.
    static __device__ __forceinline__ double res(const CTail& x, const double* u, int i, int j, int k, double uC, int& m) {
        const int p = at(i, j, k);
        const bool w = i > 0, e = i < M - 1, so = j > 0, n = j < M - 1;
        const double vW = u[w ? p - 1 : p], vE = u[e ? p + 1 : p], vS = u[so ? p - M : p], vN = u[n ? p + M : p];
        const double uW = w ? vW : uC, uE = e ? vE : uC, uS = so ? vS : uC, uN = n ? vN : uC;
        m = (int)!w + (int)!e + (int)!so + (int)!n;
        double s = (uW + uE) + (uS + uN);
        if constexpr (DIM == 3) {
            const bool bo = k > 0, to = k < M - 1;
            const double vB = u[bo ? p - M * M : p], vT = u[to ? p + M * M : p];
            m += (int)!bo + (int)!to;
            s = s + ((bo ? vB : uC) + (to ? vT : uC));
        }
        return x.F[OFF + p] - x.c[C] * ((DIM == 2 ? 4.0 : 6.0) * uC - s);
    }
    static __device__ __forceinline__ int faces(int i, int j, int k) {
        const int m = (i == 0) + (i == M - 1) + (j == 0) + (j == M - 1);
        return DIM == 2 ? m : m + (k == 0) + (k == M - 1);
    }
    static __device__ __forceinline__ double weight(const CTail& x, int m) { return x.wd[4 * C + m]; }

    static __device__ __forceinline__ void half(const CTail& x, int colour, bool zero, bool first) {
        const int tid = ct_tid();
        constexpr int IT = CELLS / 2, R = (IT + NTH - 1) / NTH;
        double* u = x.U + OFF;
        double v[R];
        int p[R];
        if (IT >= NTH || tid < IT) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = r * NTH + tid;
                const int j = (q >> (C - 1)) & (M - 1), k = DIM == 3 ? q >> (2 * C - 1) : 0;
                const int i = 2 * (q & (M / 2 - 1)) + ((j + k + colour) & 1);
                p[r] = at(i, j, k);
                if (zero && first) {
                    v[r] = 0.0 + weight(x, faces(i, j, k)) * x.F[OFF + p[r]];
                } else {
                    // the stored value of a zero iterate may be a previous visit's
                    const double uC = zero ? 0.0 : u[p[r]];
                    int m;
                    const double rr = res(x, u, i, j, k, uC, m);
                    v[r] = uC + weight(x, m) * rr;
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r) u[p[r]] = v[r];
        }
        ct_sync<WAVE>();
    }
    static __device__ __forceinline__ void jacobi(const CTail& x, bool zero) {
        const int tid = ct_tid();
        constexpr int R = (CELLS + NTH - 1) / NTH;
        double* u = x.U + OFF;
        double v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + tid;
            if (CELLS >= NTH || q < CELLS) {
                const int i = q & (M - 1), j = (q >> C) & (M - 1), k = DIM == 3 ? q >> (2 * C) : 0;
                if (zero) {
                    v[r] = 0.0 + weight(x, faces(i, j, k)) * x.F[OFF + q];
                } else {
                    int m;
                    const double rr = res(x, u, i, j, k, u[q], m);
                    v[r] = u[q] + weight(x, m) * rr;
                }
            }
        }
        ct_sync<WAVE>();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + tid;
            if (CELLS >= NTH || q < CELLS) u[q] = v[r];
        }
        ct_sync<WAVE>();
    }
    static __device__ __forceinline__ void sweep(const CTail& x, bool zero, int first) {
        if constexpr (JAC) {
            jacobi(x, zero);
        } else {
            half(x, first, zero, true);
            half(x, first ^ 1, zero, false);
        }
    }
    static __device__ __forceinline__ void restrict_avg(const CTail& x) {
        const int tid = ct_tid();
        constexpr int MC = M / 2, IT = ct_cells(DIM, C - 1), R = (CELLS + NTH - 1) / NTH;
        const double* u = x.U + OFF;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + tid;
            if (CELLS >= NTH || q < CELLS) {
                const int i = q & (M - 1), j = (q >> C) & (M - 1), k = DIM == 3 ? q >> (2 * C) : 0;
                int m;
                x.W[q] = res(x, u, i, j, k, u[q], m);
            }
        }
        ct_sync<WAVE>();
        for (int q = tid; q < IT; q += NTH) {
            const int i = 2 * (q & (MC - 1)), j = 2 * ((q >> (C - 1)) & (MC - 1));
            const int k = DIM == 3 ? 2 * (q >> (2 * (C - 1))) : 0;
            const double* w = x.W + at(i, j, k);
            const double q0 = (w[0] + w[1]) + (w[M] + w[M + 1]);
            double v;
            if constexpr (DIM == 2) {
                v = 0.25 * q0;
            } else {
                const double* z = w + M * M;
                const double q1 = (z[0] + z[1]) + (z[M] + z[M + 1]);
                v = 0.125 * (q0 + q1);
            }
            x.F[ct_off(DIM, C - 1) + q] = v;
        }
        ct_sync<WAVE>();
    }
    static __device__ __forceinline__ void correct(const CTail& x) {
        const int tid = ct_tid();
        constexpr int MC = M / 2, IT = ct_cells(DIM, C - 1);
        double* u = x.U + OFF;
        for (int q = tid; q < IT; q += NTH) {
            const int i = 2 * (q & (MC - 1)), j = 2 * ((q >> (C - 1)) & (MC - 1));
            const int k = DIM == 3 ? 2 * (q >> (2 * (C - 1))) : 0;
            const double e = x.U[ct_off(DIM, C - 1) + q];
            constexpr int K = DIM == 2 ? 4 : 8;
            double v[K];
#pragma unroll
            for (int o = 0; o < K; ++o) v[o] = u[at(i + (o & 1), j + ((o >> 1) & 1), k + (o >> 2))] + e;
#pragma unroll
            for (int o = 0; o < K; ++o) u[at(i + (o & 1), j + ((o >> 1) & 1), k + (o >> 2))] = v[o];
        }
        ct_sync<WAVE>();
    }
    // Algorithm 1 from this level: kind 0 V, 1 W, 2 F; zero: its iterate counts as zero.
    static __device__ __forceinline__ void cycle(const CTail& x, int kind, bool zero) {
        if constexpr (C == 0) {
            if (threadIdx.x == 0) x.U[OFF] = 0.0;
            ct_sync<WAVE>();
        } else {
            if (zero && x.nu1 == 0) {
                for (int q = (int)threadIdx.x; q < CELLS; q += NTH) x.U[OFF + q] = 0.0;
                ct_sync<WAVE>();
            }
            for (int s = 0; s < x.nu1; ++s) sweep(x, zero && s == 0, 0);
            if constexpr (C > 1) restrict_avg(x);  // one cell's right-hand side is not read
            using Next = CTLevel<DIM, JAC, C - 1>;
            const int calls = (kind == 0 || C == 1) ? 1 : 2;
            if constexpr (Next::WAVE && !WAVE) {
                if (threadIdx.x < 64)
                    for (int r = 0; r < calls; ++r) Next::cycle(x, kind == 2 && r ? 0 : kind, r == 0);
                __syncthreads();
            } else {
                for (int r = 0; r < calls; ++r) Next::cycle(x, kind == 2 && r ? 0 : kind, r == 0);
            }
            correct(x);
            for (int s = 0; s < x.nu2; ++s) sweep(x, false, x.post_first);
        }
    }
    static __device__ __forceinline__ void top(const CTail& x, int nl, int kind, bool zero) {
        if (nl == C + 1) {
            if constexpr (WAVE) {
                if (threadIdx.x < 64) cycle(x, kind, zero);
                __syncthreads();
            } else {
                cycle(x, kind, zero);
            }
        } else if constexpr (C > 0) {
            CTLevel<DIM, JAC, C - 1>::top(x, nl, kind, zero);
        }
    }
};

template <int DIM, bool JAC>
__global__ __launch_bounds__(CTN) void k_cc_tail(const TailDesc* __restrict__ descs, int nu1, int nu2, int post_first,
                                                 int kind, int zero) {
    constexpr int CM = DIM == 2 ? 6 : 4, TOT = ct_off(DIM, CM + 1);
    __shared__ double Us[TOT], Fs[TOT], Ws[ct_cells(DIM, CM)], wd[4 * (CM + 1)];
    const TailDesc& td = descs[blockIdx.x];
    const int* done = td.lv[0].done;
    if (done && *gp(done)) return;
    const int nl = td.nlev, t = (int)threadIdx.x;
    if (t < 4 * nl) wd[t] = td.lv[nl - 1 - t / 4].sc[t % 4];
    CTail x{Us, Fs, Ws, wd, {}, nu1, nu2, post_first};
#pragma unroll
    for (int c = 0; c <= CM; ++c) x.c[c] = c < nl ? td.lv[c < nl ? nl - 1 - c : 0].c : 0.0;
    const int np0 = 1 << (DIM * (nl - 1));
    int off0 = 0;
#pragma unroll
    for (int c = 0; c < CM; ++c) off0 += c < nl - 1 ? ct_cells(DIM, c) : 0;
    const MG_GLOBAL double* __restrict__ f0 = gp((const double*)td.lv[0].f);
    MG_GLOBAL double* u0 = gp((double*)td.lv[0].u);
#pragma unroll 4
    for (int p = t; p < np0; p += CTN) {
        Fs[off0 + p] = f0[p];
        Us[off0 + p] = zero ? 0.0 : u0[p];
    }
    __syncthreads();
    CTLevel<DIM, JAC, CM>::top(x, nl, kind, zero != 0);
    for (int p = t; p < np0; p += CTN) u0[p] = Us[off0 + p];
}

inline unsigned blocks_for(size_t N) { return (unsigned)((N + NT - 1) / NT); }

}  // namespace

size_t cc_cells(int dim, int n) { return dim == 2 ? (size_t)n * n : (size_t)n * n * n; }

CCConst cc_const(int dim, int n, double omega) {
    CCConst L;
    L.n = n;
    const double h = 1.0 / (double)n;
    L.c = 1.0 / (h * h);
    for (int m = 0; m < 4; ++m) L.wd[m] = (omega * (h * h)) / (double)(2 * dim - m);
    return L;
}

hipError_t cc_relax(int dim, bool jacobi, const double* uin, double* uout, const double* f, CCConst L, int colour,
                    hipStream_t s) {
    const unsigned b = blocks_for(cc_cells(dim, L.n));
    if (dim == 2) {
        if (jacobi) k_cc_relax<2, true><<<b, NT, 0, s>>>(uin, uout, f, L, colour);
        else k_cc_relax<2, false><<<b, NT, 0, s>>>(uin, uout, f, L, colour);
    } else {
        if (jacobi) k_cc_relax<3, true><<<b, NT, 0, s>>>(uin, uout, f, L, colour);
        else k_cc_relax<3, false><<<b, NT, 0, s>>>(uin, uout, f, L, colour);
    }
    return hipGetLastError();
}

hipError_t cc_restrict(int dim, const double* u, const double* f, double* fc, CCConst L, hipStream_t s) {
    const unsigned b = blocks_for(cc_cells(dim, L.n / 2));
    if (dim == 2) k_cc_restrict<2><<<b, NT, 0, s>>>(u, f, fc, L);
    else k_cc_restrict<3><<<b, NT, 0, s>>>(u, f, fc, L);
    return hipGetLastError();
}

hipError_t cc_prolong(int dim, double* u, const double* ec, int n, hipStream_t s) {
    const unsigned b = blocks_for(cc_cells(dim, n));
    if (dim == 2) k_cc_prolong<2><<<b, NT, 0, s>>>(u, ec, n);
    else k_cc_prolong<3><<<b, NT, 0, s>>>(u, ec, n);
    return hipGetLastError();
}

hipError_t cc_mean(int dim, int n, const double* v, const GridDesc* d, double* work, double* mean, hipStream_t s) {
    const double N = (double)cc_cells(dim, n);
    const int nrows = dim == 2 ? n : n * n, per = cc_rows_per_block(n);
    k_cc_rows<<<cdiv(nrows, per), NT, 0, s>>>(v, d, n, nrows, 0.0, work);
    double* last = work;
    if (dim == 3) {
        k_cc_rows<<<cdiv(n, per), NT, 0, s>>>(work, d, n, n, 0.0, work + nrows);
        last = work + nrows;
    }
    k_cc_rows<<<1, NT, 0, s>>>(last, d, n, 1, N, mean);
    return hipGetLastError();
}

hipError_t cc_remove_mean(int dim, int n, double* v, double* work, double* mean, hipStream_t s) {
    hipError_t e = cc_mean(dim, n, v, nullptr, work, mean, s);
    if (e != hipSuccess) return e;
    return cc_subtract(dim, n, v, nullptr, mean, s);
}

hipError_t cc_subtract(int dim, int n, double* v, const GridDesc* d, const double* mean, hipStream_t s) {
    const size_t N = cc_cells(dim, n);
    k_cc_sub<<<blocks_for(N), NT, 0, s>>>(v, d, N, mean);
    return hipGetLastError();
}

int cc_norm_parts(int dim, int n) { return (int)blocks_for(cc_cells(dim, n)); }

hipError_t cc_norm(int dim, const GridDesc* d, int n, const double* u, const double* f, double* part, double* norm,
                   hipStream_t s, const StopTest* stop) {
    const int nparts = cc_norm_parts(dim, n);
    if (dim == 2) k_cc_norm<2><<<nparts, NT, 0, s>>>(d, u, f, part);
    else k_cc_norm<3><<<nparts, NT, 0, s>>>(d, u, f, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_norm_finalize(part, nparts, nparts, 0, 1, norm, s, stop);
}

namespace {
template <int FL>
hipError_t cc_smooth_fl(int dim, int sm, const GridDesc* d, int arg, TileCfg cfg, dim3 grid, hipStream_t s) {
    if (sm == SM_JACOBI) {
        if (dim == 2) k_cc_jacobi<2, FL><<<grid, NT, 0, s>>>(d, arg);
        else k_cc_jacobi<3, FL><<<grid, NT, 0, s>>>(d, arg);
        return hipGetLastError();
    }
    if (cfg.by == 8) k_cc_sweep2d<8, FL><<<grid, NT, 0, s>>>(d, arg);
    else k_cc_sweep2d<16, FL><<<grid, NT, 0, s>>>(d, arg);
    return hipGetLastError();
}
}  // namespace

hipError_t cc_launch_smooth(int dim, int sm, const GridDesc* d, int ninst, int n, int sel, int flags, TileCfg cfg,
                            hipStream_t s) {
    if (n < 2 || ninst <= 0 || (dim == 2 && sm == SM_RBGS && cfg.by != 8 && cfg.by != 16)) return hipErrorInvalidValue;
    const dim3 grid(smooth_tiles(dim, sm, n, cfg, OP_CC), ninst);
    if (dim == 3 && sm == SM_RBGS) {
        const hipError_t e = launch_smooth3d<double>(sm, OP_CC, d, sel, flags, cfg, grid, s);
        return e != hipSuccess ? e : hipGetLastError();
    }
    const int arg = sweep_arg(sel, cfg);
    switch (flags) {
        case 0: return cc_smooth_fl<0>(dim, sm, d, arg, cfg, grid, s);
        case SWEEP_ZERO_GUESS: return cc_smooth_fl<SWEEP_ZERO_GUESS>(dim, sm, d, arg, cfg, grid, s);
        case SWEEP_PROLONG: return cc_smooth_fl<SWEEP_PROLONG>(dim, sm, d, arg, cfg, grid, s);
        case SWEEP_NORM: return cc_smooth_fl<SWEEP_NORM>(dim, sm, d, arg, cfg, grid, s);
        default: return hipErrorInvalidValue;
    }
}
hipError_t cc_launch_restrict(int dim, const GridDesc* d, int ninst, int n, int sel, hipStream_t s) {
    const dim3 grid(blocks_for(cc_cells(dim, n / 2)), ninst);
    if (dim == 2) k_cc_restrict_d<2><<<grid, NT, 0, s>>>(d, sel);
    else k_cc_restrict_d<3><<<grid, NT, 0, s>>>(d, sel);
    return hipGetLastError();
}
hipError_t cc_launch_prolong(int dim, const GridDesc* d, int ninst, int n, int sel, hipStream_t s) {
    const dim3 grid(blocks_for(cc_cells(dim, n)), ninst);
    if (dim == 2) k_cc_prolong_d<2><<<grid, NT, 0, s>>>(d, sel);
    else k_cc_prolong_d<3><<<grid, NT, 0, s>>>(d, sel);
    return hipGetLastError();
}
int cc_tail_max_edge(int dim) { return dim == 2 ? 64 : 16; }
hipError_t cc_launch_tail(int dim, int sm, const TailDesc* d, int ninst, int nu1, int nu2, int post_first, int kind,
                          bool zero, hipStream_t s) {
    const int z = zero ? 1 : 0;
    if (dim == 2) {
        if (sm == SM_JACOBI) k_cc_tail<2, true><<<ninst, CTN, 0, s>>>(d, nu1, nu2, post_first, kind, z);
        else k_cc_tail<2, false><<<ninst, CTN, 0, s>>>(d, nu1, nu2, post_first, kind, z);
    } else {
        if (sm == SM_JACOBI) k_cc_tail<3, true><<<ninst, CTN, 0, s>>>(d, nu1, nu2, post_first, kind, z);
        else k_cc_tail<3, false><<<ninst, CTN, 0, s>>>(d, nu1, nu2, post_first, kind, z);
    }
    return hipGetLastError();
}

size_t cc_work_doubles(int dim, int n) { return (dim == 2 ? (size_t)n : (size_t)n * n) + (size_t)n; }

}  // namespace mg
