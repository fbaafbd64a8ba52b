// Coarse tail of a multigrid cycle in one launch: every level from a small grid
// down to the coarsest, one workgroup per instance, all fields in LDS.
//
// Below a few thousand nodes a level is far too small to fill the chip, and
// the six launches a level costs per cycle (two pre-sweeps, residual and
// restriction, correction, two post-sweeps) are pure launch latency.  Here the
// whole recursion of Algorithm 1 below the tail's finest level (one, or with
// W- and F-cycles two recursive calls per level) runs inside one workgroup.
// The per-point arithmetic is the same as in the level kernels (same helpers,
// same operation order), so results are bitwise those of the level-by-level
// path:
//   * a zero coarse iterate (Algorithm 1's first call) or the level's iterate
//     (a W- or F-cycle's second call), then nu1 sweeps;
//   * RBGS relaxes all red nodes, then all black nodes, in place (a colour's
//     updates read only the other colour); Jacobi out of place (through
//     registers);
//   * r = f - A u on inner nodes, full weighting onto the coarse inner nodes;
//   * the coarsest grid (n = 3) is solved exactly, u = f / diag;
//   * u += P u_coarse on inner nodes, then nu2 sweeps;
//   * the tail's finest iterate is written back to its level's u.
//
// What bounds it: the chain of dependent steps (11 per level and V(2,2)
// visit), each an LDS round trip, the relaxation's dependent arithmetic and a
// barrier.  So every step is kept short: the level's edge 2^C + 1 is a
// template parameter (node coordinates are shifts and masks of the thread
// number, LDS offsets immediates), a half-sweep enumerates one colour only (no
// idle lanes), a thread issues all of its loads before its first store, the
// correction is formed per coarse cell (the 2^d nodes of a cell share their
// coarse values and no lane diverges), face coefficients are formed once per
// launch, and levels of at most 128 nodes per colour run in the first
// wavefront alone, where a step ends without a workgroup barrier.  Measured, a
// V(2,2) visit of the 33 x 33 FP64 levels and below takes 11.3 us (18.2 with
// run-time geometry and both colours enumerated), of 65 x 65 and below 21.6 us
// (against 18.2 us and six launches of 4.6 us); a 1025 x 1025 FP64 W-cycle
// solve takes 10.6 ms (61.6 ms with every level's steps launched apart).  One
// copy of the code with run-time geometry was slower again (27.6 us): the
// address arithmetic costs more than the cold instruction cache.
#include "mg_cc.h"
#include "mg_kern.h"

namespace mg {
namespace {

constexpr int TNT = 1024;  // threads per tail workgroup

// Level C has 2^C + 1 nodes per axis.  Levels lie in LDS from the coarsest up,
// so a level's place does not depend on the tail's finest level.
__host__ __device__ constexpr int tail_nodes(int dim, int C) {
    const int n = (1 << C) + 1;
    return dim == 2 ? n * n : n * n * n;
}
__host__ __device__ constexpr int tail_off(int dim, int C) {
    int s = 0;
    for (int c = 1; c < C; ++c) s += tail_nodes(dim, c);
    return s;
}
// Levels up to this C run in the first wavefront (at most 128 nodes per colour).
__host__ __device__ constexpr int tail_wave_level(int dim) { return dim == 2 ? 4 : 2; }

// The tail's constants and LDS arrays.
template <typename T, int CM>
struct TailCtx {
    T* U;          // iterates of all levels
    T* F;          // right-hand sides of all levels
    T* W;          // residual of the level at hand
    T* K[3];       // face coefficients (+x, +y, +z face of every node) of all levels
    T c[CM + 1], wd[CM + 1], om;
    T s[7];        // constant stencil
    int nu1, nu2, post_first;
};

// The end of a step: a workgroup barrier, or, where one wavefront runs the
// level (its LDS accesses execute in order), a compiler fence only.
template <bool WAVE>
__device__ __forceinline__ void tail_sync() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}

// One level: geometry and the steps of a cycle on it.
template <typename ST, typename T, int DIM, int OP, int C, int CM>
struct TailLevel {
    static constexpr int M = 1 << C, n = M + 1, sy = n, sz = n * n;
    static constexpr int OFF = tail_off(DIM, C);
    static constexpr bool WAVE = C <= tail_wave_level(DIM);
    static constexpr int NTH = WAVE ? 64 : TNT;
    static constexpr int CELLS = DIM == 2 ? M * M : M * M * M;
    using Ctx = TailCtx<T, CM>;

    // Residual at node p whose own value is uC.
    static __device__ __forceinline__ T res(const Ctx& x, const T* u, int p, T uC, T& ds) {
        const T f = x.F[OFF + p];
        if constexpr (OP == OP_VAR) {
            const T* kx = x.K[0] + OFF;
            const T* ky = x.K[1] + OFF;
            if constexpr (DIM == 2) {
                return res_var2f(uC, u[p - 1], u[p + 1], u[p - sy], u[p + sy], kx[p - 1], kx[p], ky[p - sy], ky[p],
                                 f, x.c[C], ds);
            } else {
                const T* kz = x.K[2] + OFF;
                return res_var3f(uC, u[p - 1], u[p + 1], u[p - sy], u[p + sy], u[p - sz], u[p + sz], kx[p - 1],
                                 kx[p], ky[p - sy], ky[p], kz[p - sz], kz[p], f, x.c[C], ds);
            }
        } else {
            ds = T(0);
            if constexpr (DIM == 2)
                return res_const2<OP>(uC, u[p - 1], u[p + 1], u[p - sy], u[p + sy], f, x.c[C], x.s);
            else
                return res_const3<OP>(uC, u[p - 1], u[p + 1], u[p - sy], u[p + sy], u[p - sz], u[p + sz], f, x.c[C],
                                      x.s);
        }
    }
    static __device__ __forceinline__ T dsum(const Ctx& x, int p) {
        const T* kx = x.K[0] + OFF;
        const T* ky = x.K[1] + OFF;
        const T xy = (kx[p - 1] + kx[p]) + (ky[p - sy] + ky[p]);
        if constexpr (DIM == 2) {
            return xy;
        } else {
            const T* kz = x.K[2] + OFF;
            return xy + (kz[p - sz] + kz[p]);
        }
    }
    static __device__ __forceinline__ T relaxed(const Ctx& x, T uC, T r, T ds) {
        return stored<ST>(relax<T, OP == OP_VAR>(uC, r, ds, x.c[C], x.wd[C], x.om));
    }
    // The update of a node whose neighbours and own value are zero reads
    // neither: its residual is f.
    static __device__ __forceinline__ T relaxed_zero(const Ctx& x, int p) {
        T ds = T(0);
        if constexpr (OP == OP_VAR) ds = dsum(x, p);
        return relaxed(x, T(0), x.F[OFF + p], ds);
    }
    // Node of item q of one colour ((i + j [+ k]) & 1 == colour), M/2 per row;
    // false where the item falls on the far boundary (p is then an inner node).
    static __device__ __forceinline__ bool colour_node(int q, int colour, int& p) {
        const int j = 1 + ((q >> (C - 1)) & (M - 1));
        const int k = DIM == 3 ? 1 + (q >> (2 * C - 1)) : 0;
        const int i = 1 + 2 * (q & (M / 2 - 1)) + ((1 + j + k + colour) & 1);
        const bool in = i < M && j < M && k < M;
        p = in ? (k * n + j) * n + i : (DIM == 2 ? n + 1 : (n + 1) * n + 1);
        return in;
    }
    static __device__ __forceinline__ bool node(int q, int& p) {
        const int i = 1 + (q & (M - 1)), j = 1 + ((q >> C) & (M - 1));
        const int k = DIM == 3 ? 1 + (q >> (2 * C)) : 0;
        const bool in = i < M && j < M && k < M;
        p = in ? (k * n + j) * n + i : (DIM == 2 ? n + 1 : (n + 1) * n + 1);
        return in;
    }

    // A half-sweep: every node of one colour.  zero: the iterate is zero
    // (first: so is the other colour, else the other colour has been relaxed).
    static __device__ __forceinline__ void half(const Ctx& x, int colour, bool zero, bool first) {
        constexpr int IT = CELLS / 2, R = (IT + NTH - 1) / NTH;
        T* u = x.U + OFF;
        T v[R];
        int p[R];
        bool in[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + (int)threadIdx.x;
            in[r] = colour_node(q < IT ? q : IT - 1, colour, p[r]) && q < IT;
        }
        if (IT >= NTH || (int)threadIdx.x < ((IT + 63) & ~63)) {
            if (zero && first) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = relaxed_zero(x, p[r]);
            } else {
                // the stored value of a zero iterate may be a previous visit's
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const T uC = zero ? T(0) : u[p[r]];
                    T ds;
                    const T rr = res(x, u, p[r], uC, ds);
                    v[r] = relaxed(x, uC, rr, ds);
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (in[r]) u[p[r]] = v[r];
        }
        tail_sync<WAVE>();
    }

    static __device__ __forceinline__ void jacobi(const Ctx& x, bool zero) {
        constexpr int R = (CELLS + NTH - 1) / NTH;
        T* u = x.U + OFF;
        T v[R];
        int p[R];
        bool in[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + (int)threadIdx.x;
            in[r] = node(q < CELLS ? q : CELLS - 1, p[r]) && q < CELLS;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (zero) {
                v[r] = relaxed_zero(x, p[r]);
            } else {
                T ds;
                const T rr = res(x, u, p[r], u[p[r]], ds);
                v[r] = relaxed(x, u[p[r]], rr, ds);
            }
        }
        tail_sync<WAVE>();
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (in[r]) u[p[r]] = v[r];
        tail_sync<WAVE>();
    }

    template <int SM>
    static __device__ __forceinline__ void sweep(const Ctx& x, bool zero, int first) {
        if constexpr (SM == SM_RBGS) {
            half(x, first, zero, true);
            half(x, first ^ 1, zero, false);
        } else {
            jacobi(x, zero);
        }
    }

    static __device__ __forceinline__ void residual(const Ctx& x) {
        constexpr int R = (CELLS + NTH - 1) / NTH;
        const T* u = x.U + OFF;
        T v[R];
        int p[R];
        bool in[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = r * NTH + (int)threadIdx.x;
            in[r] = node(q < CELLS ? q : CELLS - 1, p[r]) && q < CELLS;
            T ds;
            v[r] = res(x, u, p[r], u[p[r]], ds);
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (in[r]) x.W[p[r]] = v[r];
        tail_sync<WAVE>();
    }

    // Full weighting of the residual in W onto level C - 1's right-hand side;
    // same operation order as the restriction kernel.
    static __device__ __forceinline__ void restrict_fw(const Ctx& x) {
        constexpr int MC = M / 2, nc = MC + 1, IT = DIM == 2 ? MC * MC : MC * MC * MC;
        T* fc = x.F + tail_off(DIM, C - 1);
        for (int q = (int)threadIdx.x; q < IT; q += NTH) {
            const int I = 1 + (q & (MC - 1)), J = 1 + ((q >> (C - 1)) & (MC - 1));
            const int K = DIM == 3 ? 1 + (q >> (2 * (C - 1))) : 0;
            if (I >= MC || J >= MC || K >= MC) continue;
            const T* R = x.W + ((2 * K) * n + 2 * J) * n + 2 * I;
            T v;
            if constexpr (DIM == 2) {
                const T edges = (R[-1] + R[1]) + (R[-sy] + R[sy]);
                const T corners = (R[-sy - 1] + R[-sy + 1]) + (R[sy - 1] + R[sy + 1]);
                v = (T(0.25) * R[0] + T(0.125) * edges) + T(0.0625) * corners;
            } else {
                const T* Rb = R - sz;
                const T* Ra = R + sz;
                const T faces = ((R[-1] + R[1]) + (R[-sy] + R[sy])) + (Rb[0] + Ra[0]);
                const T exy = (R[-sy - 1] + R[-sy + 1]) + (R[sy - 1] + R[sy + 1]);
                const T exz = (Rb[-1] + Rb[1]) + (Ra[-1] + Ra[1]);
                const T eyz = (Rb[-sy] + Rb[sy]) + (Ra[-sy] + Ra[sy]);
                const T edges = (exy + exz) + eyz;
                const T cz0 = (Rb[-sy - 1] + Rb[-sy + 1]) + (Rb[sy - 1] + Rb[sy + 1]);
                const T cz1 = (Ra[-sy - 1] + Ra[-sy + 1]) + (Ra[sy - 1] + Ra[sy + 1]);
                const T corners = cz0 + cz1;
                v = ((T(0.125) * R[0] + T(0.0625) * faces) + T(0.03125) * edges) + T(0.015625) * corners;
            }
            fc[(K * nc + J) * nc + I] = stored<ST>(v);
        }
        tail_sync<WAVE>();
    }

    // u += P u_coarse at inner nodes: a thread takes the nodes (2I..2I+1) x
    // (2J..2J+1) [x (2K..2K+1)] of one coarse cell.
    static __device__ __forceinline__ void correct(const Ctx& x) {
        constexpr int MC = M / 2, nc = MC + 1, IT = DIM == 2 ? MC * MC : MC * MC * MC;
        T* u = x.U + OFF;
        for (int q = (int)threadIdx.x; q < IT; q += NTH) {
            const int I = q & (MC - 1), J = (q >> (C - 1)) & (MC - 1);
            const int K = DIM == 3 ? q >> (2 * (C - 1)) : 0;
            const T* e = x.U + tail_off(DIM, C - 1) + (K * nc + J) * nc + I;
            T* w = u + ((2 * K) * n + 2 * J) * n + 2 * I;
            const T e00 = e[0], e10 = e[1], e01 = e[nc], e11 = e[nc + 1];
            const T ex = e00 + e10, exy = ex + (e01 + e11);
            const T w0 = w[0], w1 = w[1], w2 = w[sy], w3 = w[sy + 1];
            if constexpr (DIM == 2) {
                if (I && J) w[0] = stored<ST>(w0 + e00);
                if (J) w[1] = stored<ST>(w1 + T(0.5) * ex);
                if (I) w[sy] = stored<ST>(w2 + T(0.5) * (e00 + e01));
                w[sy + 1] = stored<ST>(w3 + T(0.25) * exy);
            } else {
                const T* g = e + nc * nc;
                T* z = w + sz;
                const T g00 = g[0], g10 = g[1], g01 = g[nc], g11 = g[nc + 1];
                const T z0 = z[0], z1 = z[1], z2 = z[sy], z3 = z[sy + 1];
                const T gx = g00 + g10;
                if (I && J && K) w[0] = stored<ST>(w0 + e00);
                if (J && K) w[1] = stored<ST>(w1 + T(0.5) * ex);
                if (I && K) w[sy] = stored<ST>(w2 + T(0.5) * (e00 + e01));
                if (K) w[sy + 1] = stored<ST>(w3 + T(0.25) * exy);
                if (I && J) z[0] = stored<ST>(z0 + T(0.5) * (e00 + g00));
                if (J) z[1] = stored<ST>(z1 + T(0.25) * (ex + gx));
                if (I) z[sy] = stored<ST>(z2 + T(0.25) * ((e00 + e01) + (g00 + g01)));
                z[sy + 1] = stored<ST>(z3 + T(0.125) * (exy + (gx + (g01 + g11))));
            }
        }
        tail_sync<WAVE>();
    }

    static __device__ __forceinline__ void clear(const Ctx& x) {
        T* u = x.U + OFF;
        for (int q = (int)threadIdx.x; q < tail_nodes(DIM, C); q += NTH) u[q] = T(0);
        tail_sync<WAVE>();
    }

    // Algorithm 1 from this level: kind 0 V (one recursive call), 1 W (two), 2
    // F (an F- then a V-cycle); zero: the iterate counts as zero.
    template <int SM>
    static __device__ __forceinline__ void cycle(const Ctx& x, int kind, bool zero) {
        if constexpr (C == 1) {
            // coarsest grid: one unknown, u = f / diag (of any iterate)
            if (threadIdx.x == 0) {
                constexpr int p = DIM == 2 ? 4 : 13;
                T diag;
                if constexpr (OP == OP_VAR) diag = x.c[C] * dsum(x, p);
                else if constexpr (OP == OP_STENCIL) diag = x.c[C] * x.s[0];
                else diag = x.c[C] * (DIM == 2 ? T(4) : T(6));
                x.U[OFF + p] = stored<ST>(x.F[OFF + p] / diag);
            }
            tail_sync<WAVE>();
        } else {
            if (zero && x.nu1 == 0) clear(x);
            for (int s = 0; s < x.nu1; ++s) sweep<SM>(x, zero && s == 0, 0);
            residual(x);
            restrict_fw(x);
            using Next = TailLevel<ST, T, DIM, OP, C - 1, CM>;
            // the coarsest solve is exact: a second call would repeat it
            const int calls = (kind == 0 || C == 2) ? 1 : 2;
            if constexpr (Next::WAVE && !WAVE) {
                if (threadIdx.x < 64)
                    for (int r = 0; r < calls; ++r) Next::template cycle<SM>(x, kind == 2 && r ? 0 : kind, r == 0);
                __syncthreads();
            } else {
                for (int r = 0; r < calls; ++r) Next::template cycle<SM>(x, kind == 2 && r ? 0 : kind, r == 0);
            }
            correct(x);
            for (int s = 0; s < x.nu2; ++s) sweep<SM>(x, false, x.post_first);
        }
    }

    // The tail of an instance whose finest tail level is C.
    template <int SM>
    static __device__ __forceinline__ void top(const Ctx& x, int kind, bool zero) {
        if constexpr (WAVE) {
            if (threadIdx.x < 64) cycle<SM>(x, kind, zero);
            __syncthreads();
        } else {
            cycle<SM>(x, kind, zero);
        }
    }
    // face coefficients from the level's nodal k: the lower and the upper node
    // of every +x, +y, +z face
    static __device__ __forceinline__ void faces(const Ctx& x, const MG_GLOBAL T* __restrict__ k) {
        for (int q = (int)threadIdx.x; q < CELLS; q += TNT) {
            const int i = q & (M - 1), j = (q >> C) & (M - 1), kk = DIM == 3 ? q >> (2 * C) : 0;
            const int p = (kk * n + j) * n + i;
            const T a = k[p];
            x.K[0][OFF + p] = kface(a, k[p + 1]);
            x.K[1][OFF + p] = kface(a, k[p + sy]);
            if constexpr (DIM == 3) x.K[2][OFF + p] = kface(a, k[p + sz]);
        }
    }
};

// Level constants (and face coefficients) of levels 1 .. nl of one instance.
template <typename ST, typename T, int DIM, int OP, int C, int CM>
__device__ __forceinline__ void tail_setup(TailCtx<T, CM>& x, const TailDesc& td, int nl) {
    if (C <= nl) {
        const GridDesc& g = td.lv[nl - C];
        x.c[C] = (T)g.c;
        x.wd[C] = (T)g.wd;
        if constexpr (OP == OP_VAR) TailLevel<ST, T, DIM, OP, C, CM>::faces(x, gp((const T*)g.k));
    } else {
        x.c[C] = x.wd[C] = T(0);
    }
    if constexpr (C > 1) tail_setup<ST, T, DIM, OP, C - 1, CM>(x, td, nl);
}
template <typename ST, typename T, int DIM, int SM, int OP, int C, int CM>
__device__ __forceinline__ void tail_run(const TailCtx<T, CM>& x, int nl, int kind, bool zero) {
    if (nl == C) TailLevel<ST, T, DIM, OP, C, CM>::template top<SM>(x, kind, zero);
    else if constexpr (C > 1) tail_run<ST, T, DIM, SM, OP, C - 1, CM>(x, nl, kind, zero);
}

// kind: 0 V, 1 W, 2 F; zero: start from a zero iterate (else from the level's u).
template <typename ST, int DIM, int SM, int OP, int CM>
__global__ __launch_bounds__(TNT) void k_tail(const TailDesc* __restrict__ descs, int nu1, int nu2, int post_first,
                                              int kind, int zero) {
    using T = arith_t<ST>;
    constexpr int TOT = tail_off(DIM, CM + 1);
    __shared__ T Us[TOT];
    __shared__ T Fs[TOT];
    __shared__ T Ws[tail_nodes(DIM, CM)];
    __shared__ T Ks[OP == OP_VAR ? DIM * TOT : 1];
    const TailDesc& td = descs[blockIdx.x];
    const int* done = td.lv[0].done;
    if (done && *gp(done)) return;
    const int nl = td.nlev;
    TailCtx<T, CM> x;
    x.U = Us;
    x.F = Fs;
    x.W = Ws;
    x.K[0] = Ks;
    x.K[1] = Ks + (OP == OP_VAR ? TOT : 0);
    x.K[2] = Ks + (OP == OP_VAR ? (DIM - 1) * TOT : 0);
    x.om = (T)td.lv[0].omega;
    if constexpr (OP == OP_STENCIL) {
#pragma unroll
        for (int q = 0; q < 7; ++q) x.s[q] = (T)td.lv[0].sc[q];
    }
    x.nu1 = nu1;
    x.nu2 = nu2;
    x.post_first = post_first;
    // every iterate starts at zero (boundaries stay there); f, and with zero ==
    // 0 the iterate, of the tail's finest level come from device memory
    const int n0 = td.lv[0].n;
    const int np0 = DIM == 2 ? n0 * n0 : n0 * n0 * n0;
    int off0 = 0;
#pragma unroll
    for (int c = 1; c < CM; ++c) off0 += c < nl ? tail_nodes(DIM, c) : 0;
    const MG_GLOBAL ST* __restrict__ f0 = gp((const ST*)td.lv[0].f);
    const MG_GLOBAL ST* u0r = gp((const ST*)td.lv[0].u);
    for (int p = threadIdx.x; p < off0; p += TNT) Us[p] = T(0);
#pragma unroll 4
    for (int p = threadIdx.x; p < np0; p += TNT) {
        Fs[off0 + p] = (T)f0[p];
        Us[off0 + p] = zero ? T(0) : (T)u0r[p];
    }
    tail_setup<ST, T, DIM, OP, CM, CM>(x, td, nl);
    __syncthreads();
    tail_run<ST, T, DIM, SM, OP, CM, CM>(x, nl, kind, zero != 0);
    // the tail's finest iterate back to device memory (inner nodes; its
    // boundary there is zero already); a row per wavefront
    MG_GLOBAL ST* __restrict__ u0 = gp((ST*)td.lv[0].u);
    const int rows = DIM == 2 ? n0 : n0 * n0;
    for (int r = threadIdx.x >> 6; r < rows; r += TNT / 64) {
        const int j = DIM == 2 ? r : r % n0, k = DIM == 2 ? 1 : r / n0;
        if (j < 1 || j > n0 - 2 || k < 1 || k > n0 - 2) continue;
        for (int i = 1 + (threadIdx.x & 63); i <= n0 - 2; i += 64) u0[r * n0 + i] = (ST)Us[off0 + r * n0 + i];
    }
}

// ---------------------------------------------------------------------------
// Conjugate gradients on a coarsest level with more than one unknown
// (Algorithm 1: the coarsest grid is solved by a direct solver or by CG), one
// workgroup per instance, every vector in LDS.  From u = 0: r = p = f on the
// inner nodes, then a fixed number of steps (fewer only if r or p^T A p
// becomes zero): q = A p, alpha = (r^T r) / (p^T q), u += alpha p,
// r -= alpha q, beta = (r_new^T r_new) / (r^T r), p = r + beta p.  Inner
// products are formed in FP64 from the vectors' values, each x-row summed
// left to right and the row sums added in row order; alpha and beta are the
// FP64 quotients rounded to the arithmetic type; the vector updates are in
// the arithmetic type and every stored vector value is rounded to the
// storage type ST.
// ---------------------------------------------------------------------------

// Inner node q (0-based over the (n-2)^dim inner nodes) -> node index.
template <int DIM>
__device__ __forceinline__ int cg_node(int q, int n) {
    const int m = n - 2;
    const int i = 1 + q % m;
    const int r = q / m;
    const int j = 1 + (DIM == 2 ? r : r % m);
    const int k = DIM == 2 ? 0 : 1 + r / m;
    return (k * n + j) * n + i;
}

template <typename T, int DIM, bool VAR>
__device__ __forceinline__ T cg_apply(const T* v, const T* k, int n, T c, int p) {
    const int sy = n, sz = n * n;
    if constexpr (VAR) {
        const T kp = k[p];
        const T kxW = kface(k[p - 1], kp), kxC = kface(kp, k[p + 1]);
        const T kyS = kface(k[p - sy], kp), kyC = kface(kp, k[p + sy]);
        if constexpr (DIM == 2) {
            const T dsum = (kxW + kxC) + (kyS + kyC);
            const T t = (kxW * v[p - 1] + kxC * v[p + 1]) + (kyS * v[p - sy] + kyC * v[p + sy]);
            return c * (dsum * v[p] - t);
        } else {
            const T kzB = kface(k[p - sz], kp), kzC = kface(kp, k[p + sz]);
            const T dsum = ((kxW + kxC) + (kyS + kyC)) + (kzB + kzC);
            const T t = ((kxW * v[p - 1] + kxC * v[p + 1]) + (kyS * v[p - sy] + kyC * v[p + sy])) +
                        (kzB * v[p - sz] + kzC * v[p + sz]);
            return c * (dsum * v[p] - t);
        }
    } else if constexpr (DIM == 2) {
        const T s = (v[p - 1] + v[p + 1]) + (v[p - sy] + v[p + sy]);
        return c * (T(4) * v[p] - s);
    } else {
        const T s = ((v[p - 1] + v[p + 1]) + (v[p - sy] + v[p + sy])) + (v[p - sz] + v[p + sz]);
        return c * (T(6) * v[p] - s);
    }
}

// FP64 inner product over the inner nodes: thread t sums inner row t (x from
// 1 to n-2), thread 0 adds the row sums in order.  Result in every thread.
template <typename T, int DIM>
__device__ __forceinline__ double cg_dot(const T* a, const T* b, int n, double* rows, double* bc) {
    const int m = n - 2;
    const int nrows = DIM == 2 ? m : m * m;
    for (int t = threadIdx.x; t < nrows; t += TNT) {
        const int j = 1 + t % m, k = DIM == 2 ? 0 : 1 + t / m;
        const int base = (k * n + j) * n;
        double s = 0.0;
        for (int i = 1; i <= m; ++i) s += (double)a[base + i] * (double)b[base + i];
        rows[t] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int t = 0; t < nrows; ++t) s += rows[t];
        *bc = s;
    }
    __syncthreads();
    const double v = *bc;
    __syncthreads();  // bc and rows are written again by the next product
    return v;
}

template <typename ST, int DIM, bool VAR, int NMAX>
__global__ __launch_bounds__(TNT) void k_cg(const GridDesc* __restrict__ descs, int iters) {
    using T = arith_t<ST>;
    constexpr int TOT = DIM == 2 ? NMAX * NMAX : NMAX * NMAX * NMAX;
    constexpr int NROWS = DIM == 2 ? NMAX : NMAX * NMAX;
    __shared__ T U[TOT], R[TOT], Pv[TOT], Q[TOT];
    __shared__ T K[VAR ? TOT : 1];
    __shared__ double rows[NROWS];
    __shared__ double bc;
    const GridDesc d = descs[blockIdx.x];
    if (d.done && *gp(d.done)) return;
    const int n = d.n;
    const int np = DIM == 2 ? n * n : n * n * n;
    const T c = (T)d.c;
    const MG_GLOBAL ST* __restrict__ f = gp((const ST*)d.f);
    const int cnt = (DIM == 2 ? (n - 2) * (n - 2) : (n - 2) * (n - 2) * (n - 2));
    for (int p = threadIdx.x; p < np; p += TNT) {
        U[p] = T(0);
        R[p] = T(0);
        Pv[p] = T(0);
        Q[p] = T(0);
        if constexpr (VAR) K[p] = gp((const T*)d.k)[p];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < cnt; q += TNT) {
        const int p = cg_node<DIM>(q, n);
        R[p] = (T)f[p];
        Pv[p] = (T)f[p];
    }
    __syncthreads();
    double rr = cg_dot<T, DIM>(R, R, n, rows, &bc);
    for (int it = 0; it < iters && rr > 0.0; ++it) {
        for (int q = threadIdx.x; q < cnt; q += TNT) {
            const int p = cg_node<DIM>(q, n);
            Q[p] = stored<ST>(cg_apply<T, DIM, VAR>(Pv, K, n, c, p));
        }
        __syncthreads();
        const double pq = cg_dot<T, DIM>(Pv, Q, n, rows, &bc);
        if (!(pq > 0.0)) break;
        const T alpha = (T)(rr / pq);
        for (int q = threadIdx.x; q < cnt; q += TNT) {
            const int p = cg_node<DIM>(q, n);
            U[p] = stored<ST>(U[p] + alpha * Pv[p]);
            R[p] = stored<ST>(R[p] - alpha * Q[p]);
        }
        __syncthreads();
        const double rr_new = cg_dot<T, DIM>(R, R, n, rows, &bc);
        const T beta = (T)(rr_new / rr);
        for (int q = threadIdx.x; q < cnt; q += TNT) {
            const int p = cg_node<DIM>(q, n);
            Pv[p] = stored<ST>(R[p] + beta * Pv[p]);
        }
        __syncthreads();
        rr = rr_new;
    }
    MG_GLOBAL ST* __restrict__ u = gp((ST*)d.u);
    for (int p = threadIdx.x; p < np; p += TNT) u[p] = (ST)U[p];
}

}  // namespace

// The tail's LDS (160 KB) holds arithmetic-type values: iterate and right-hand
// side of every level, one residual and, with a coefficient field, the face
// coefficients (a 65 x 65 FP64 tail takes 125 KB, with faces it would take
// 217).
int tail_max_edge(int dim, int elem, int op) {
    if (op == OP_CC) return cc_tail_max_edge(dim);
    const bool big = elem <= 4 || op != OP_VAR;
    return dim == 2 ? (big ? 65 : 33) : (big ? 17 : 9);
}
// Conjugate gradients keep four vectors and a coefficient in LDS.
int cg_max_edge(int dim, int elem) {
    if (dim == 2) return elem <= 4 ? 65 : 33;
    return elem <= 4 ? 17 : 9;
}

template <typename T>
hipError_t launch_tail(int dim, int sm, int op, const TailDesc* d, int ninst, int nu1, int nu2, int post_first,
                       int kind, bool zero, hipStream_t s) {
    if (ninst <= 0) return hipSuccess;
    if (op == OP_CC) return cc_launch_tail(dim, sm, d, ninst, nu1, nu2, post_first, kind, zero, s);
    constexpr bool F = sizeof(arith_t<T>) == 4;
    const int z = zero ? 1 : 0;
#define MG_TAIL(DIMV, OPV, CMV)                                                                                \
    do {                                                                                                       \
        if (sm == SM_RBGS) k_tail<T, DIMV, SM_RBGS, OPV, CMV><<<ninst, TNT, 0, s>>>(d, nu1, nu2, post_first, kind, z); \
        else k_tail<T, DIMV, SM_JACOBI, OPV, CMV><<<ninst, TNT, 0, s>>>(d, nu1, nu2, post_first, kind, z);     \
        return hipGetLastError();                                                                              \
    } while (0)
    if (op == OP_LAP) {
        if (dim == 2) MG_TAIL(2, OP_LAP, 6);
        else MG_TAIL(3, OP_LAP, 4);
    }
    if constexpr (sizeof(T) >= 4) {  // binary16 storage: Laplacian only; a constant stencil: FP64 only
        if (op == OP_VAR) {
            if (dim == 2) MG_TAIL(2, OP_VAR, (F ? 6 : 5));
            else MG_TAIL(3, OP_VAR, (F ? 4 : 3));
        }
    }
    if constexpr (sizeof(T) == 8) {
        if (op == OP_STENCIL) {
            if (dim == 2) MG_TAIL(2, OP_STENCIL, 6);
            else MG_TAIL(3, OP_STENCIL, 4);
        }
    }
#undef MG_TAIL
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_cg(int dim, bool var, const GridDesc* d, int ninst, int n, int iters, hipStream_t s) {
    const bool f = sizeof(arith_t<T>) == 4;
    if (ninst <= 0) return hipSuccess;
    if (n > cg_max_edge(dim, f ? 4 : 8) || n < 3 || iters < 0) return hipErrorInvalidValue;
    if constexpr (sizeof(T) == 2) {
        if (var) return hipErrorInvalidValue;
        if (dim == 2) k_cg<T, 2, false, 65><<<ninst, TNT, 0, s>>>(d, iters);
        else k_cg<T, 3, false, 17><<<ninst, TNT, 0, s>>>(d, iters);
    } else if constexpr (sizeof(T) == 4) {
        if (dim == 2) {
            if (var) k_cg<T, 2, true, 65><<<ninst, TNT, 0, s>>>(d, iters);
            else k_cg<T, 2, false, 65><<<ninst, TNT, 0, s>>>(d, iters);
        } else {
            if (var) k_cg<T, 3, true, 17><<<ninst, TNT, 0, s>>>(d, iters);
            else k_cg<T, 3, false, 17><<<ninst, TNT, 0, s>>>(d, iters);
        }
    } else {
        if (dim == 2) {
            if (var) k_cg<T, 2, true, 33><<<ninst, TNT, 0, s>>>(d, iters);
            else k_cg<T, 2, false, 33><<<ninst, TNT, 0, s>>>(d, iters);
        } else {
            if (var) k_cg<T, 3, true, 9><<<ninst, TNT, 0, s>>>(d, iters);
            else k_cg<T, 3, false, 9><<<ninst, TNT, 0, s>>>(d, iters);
        }
    }
    return hipGetLastError();
}

template hipError_t launch_cg<double>(int, bool, const GridDesc*, int, int, int, hipStream_t);
template hipError_t launch_cg<float>(int, bool, const GridDesc*, int, int, int, hipStream_t);
template hipError_t launch_cg<half_t>(int, bool, const GridDesc*, int, int, int, hipStream_t);
template hipError_t launch_tail<double>(int, int, int, const TailDesc*, int, int, int, int, int, bool, hipStream_t);
template hipError_t launch_tail<float>(int, int, int, const TailDesc*, int, int, int, int, int, bool, hipStream_t);
template hipError_t launch_tail<half_t>(int, int, int, const TailDesc*, int, int, int, int, int, bool, hipStream_t);

}  // namespace mg
