// 2D: one leg of a cycle on a level in one launch (red-black, two sweeps):
//   down  the two pre-smoothing sweeps, the residual and full weighting
//   up    the correction and the two post-smoothing sweeps
// A workgroup holds a 64-wide box of the level in registers; each half-sweep
// is valid on one ring less, and four half-sweeps, the residual and full
// weighting need six rings, so a down box owns 26 coarse columns (52 fine
// ones) of 64, an up box 56 columns.
//
// A leg reads the level once and writes it once.  On levels too small to fill
// the chip it takes one launch where sweeps and restriction cost 3.3 .. 6 us
// each whatever they do; what bounds it there is the chain of half-sweeps (4.7
// .. 5.2 us), on many boxes going down vector-ALU issue (0.72 of the time at
// 4097^2 FP32, where it moves no byte twice at 3.3 TB/s), going up issue and
// memory together (0.55, 4.8 TB/s).  Lane = x, and a thread holds P vertical
// pairs of nodes; colours alternate, so of each pair it holds one red and one
// black node (A, B), and a half-sweep updates one register per pair on every
// lane.  Its neighbours are the other colour's registers: the adjacent lanes'
// of the same pair along x, along y the own pair's and the pair's above or
// below by the lane's parity.  Only the rows next to another wavefront's pass
// through LDS: one word read and one written per lane and half-sweep.  (A box
// in LDS, each half-sweep reading its five nodes there: 110 and 107 us down and
// up on 22 grids of 1025 x 1025 against 94 and 75.)  Per node the expressions
// are those of the level kernels, in the same order, stored values rounded in
// between.
//
// Measured per V(2,2) cycle and solve step against sweeps (or pairs of them)
// and restriction apart, whole solves: FP64 1025^2 131 -> 85 us, 4097^2 685 ->
// 349; FP32 refinement 4097^2 398 -> 316, 8193^2 1313 -> 1003; variable
// coefficients FP32 2049^2 370 -> 195.  At 4097^2 FP32 a leg down takes 47 us
// (151 MB it cannot do without: 24 us at 6.2 TB/s), up 46 us (218 MB: 35).
#include "mg_kern.h"

namespace mg {
namespace {

constexpr int LW = 8;              // wavefronts
constexpr int LCX = 26;            // coarse columns of a down box
constexpr int LUX = 56;            // columns of an up box
constexpr int leg_rows(int P) { return 2 * P * LW; }
constexpr int leg_cy(int P) { return (leg_rows(P) - 12) / 2; }  // coarse rows of a down box
constexpr int leg_uy(int P) { return leg_rows(P) - 8; }         // rows of an up box

template <typename ST, int OP, int P>
struct LegBox {
    using T = arith_t<ST>;
    static constexpr bool VAR = OP == OP_VAR;
    static constexpr int RT = 2 * P, LB = leg_rows(P);
    int n, xs, ys, lane, w, gx, r0;  // r0: first row of the thread in the box
    bool s;                          // the red node of a pair is in its second row
    T c, wd, om;
    T sc[7];
    T A[P], B[P], fA[P], fB[P];
    bool inA[P], inB[P];
    unsigned rb[RT];                 // byte offset of each row's node (clamped)
    // VAR: faces of the red and black nodes: -x, +x, towards the own pair's other node, away from it
    T kA[VAR ? P : 1][4], kB[VAR ? P : 1][4];
    T si, so;                        // stencil: coefficient of a red node's neighbour in / outside its pair
    T *rdA, *rdB, *wrA, *wrB;        // exchange of the rows next to other wavefronts'

    __device__ __forceinline__ void init(const GridDesc& d, int xs_, int ys_, T (*E)[2][BX]) {
        n = d.n;
        xs = xs_;
        ys = ys_;
        lane = threadIdx.x & 63;
        w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        gx = xs + lane;
        r0 = RT * w;
        s = ((gx + ys) & 1) != 0;
        c = (T)d.c;
        wd = (T)d.wd;
        om = (T)d.omega;
        load_stencil<OP>(d, sc);
        if constexpr (OP == OP_STENCIL) {
            si = pick(s, sc[3], sc[4]);
            so = pick(s, sc[4], sc[3]);
        }
        const bool coli = gx >= 1 && gx <= n - 2 && lane >= 1 && lane <= BX - 2;
        const int xc = min(max(gx, 0), n - 1);
#pragma unroll
        for (int r = 0; r < RT; ++r)
            rb[r] = (unsigned)(min(max(ys + r0 + r, 0), n - 1) * n + xc) * (unsigned)sizeof(ST);
        bool in[RT];
#pragma unroll
        for (int r = 0; r < RT; ++r)
            in[r] = coli && ys + r0 + r >= 1 && ys + r0 + r <= n - 2 && r0 + r >= 1 && r0 + r <= LB - 2;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            inA[p] = (s && in[2 * p + 1]) || (!s && in[2 * p]);
            inB[p] = (s && in[2 * p]) || (!s && in[2 * p + 1]);
        }
        // E[w + 1]: first and last row of wavefront w
        wrA = &E[w + 1][s ? 1 : 0][lane];
        wrB = &E[w + 1][s ? 0 : 1][lane];
        rdA = &E[s ? w + 2 : w][s ? 0 : 1][lane];
        rdB = &E[s ? w : w + 2][s ? 1 : 0][lane];
    }
    __device__ __forceinline__ void sort(const T (&v)[RT], T (&a)[P], T (&b)[P]) const {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            a[p] = pick(s, v[2 * p + 1], v[2 * p]);
            b[p] = pick(s, v[2 * p], v[2 * p + 1]);
        }
    }
    __device__ __forceinline__ void rows(const T (&a)[P], const T (&b)[P], T (&v)[RT]) const {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            v[2 * p] = pick(s, b[p], a[p]);
            v[2 * p + 1] = pick(s, a[p], b[p]);
        }
    }
    __device__ __forceinline__ void load(const void* a, T (&v)[RT]) const {
        const PlaneBuf<ST> b(gp((const ST*)a), (size_t)n * n);
#pragma unroll
        for (int r = 0; r < RT; ++r) v[r] = (T)b.load(rb[r]);
    }
    __device__ __forceinline__ void load_f(const GridDesc& d) {
        T v[RT];
        load(d.f, v);
        sort(v, fA, fB);
        if constexpr (VAR) {
            const PlaneBuf<T> b(gp((const T*)d.k), (size_t)n * n);
            const int xc = min(max(gx, 0), n - 1);
            T k[RT + 2], kx[RT], kw[RT], ky[RT + 1];  // rows -1 .. RT
#pragma unroll
            for (int r = 0; r < RT + 2; ++r)
                k[r] = b.load((unsigned)(min(max(ys + r0 + r - 1, 0), n - 1) * n + xc) * (unsigned)sizeof(T));
#pragma unroll
            for (int r = 0; r <= RT; ++r) ky[r] = kface(k[r], k[r + 1]);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                kx[r] = kface(k[r + 1], lane_next(k[r + 1]));
                kw[r] = lane_prev(kx[r]);
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const int r = 2 * p;
                kA[p][0] = pick(s, kw[r + 1], kw[r]);
                kB[p][0] = pick(s, kw[r], kw[r + 1]);
                kA[p][1] = pick(s, kx[r + 1], kx[r]);
                kB[p][1] = pick(s, kx[r], kx[r + 1]);
                kA[p][2] = kB[p][2] = ky[r + 1];
                kA[p][3] = pick(s, ky[r + 2], ky[r]);
                kB[p][3] = pick(s, ky[r], ky[r + 2]);
            }
        }
    }
    // The rows next to other wavefronts' into LDS: red, black.
    __device__ __forceinline__ void putA() const { *wrA = pick(s, A[P - 1], A[0]); }
    __device__ __forceinline__ void putB() const { *wrB = pick(s, B[0], B[P - 1]); }
    // Residual of pair p's red (RED) or black node; e: the neighbour in LDS of
    // the pair at the thread's edge.
    template <bool RED>
    __device__ __forceinline__ T res(int p, T e, T& ds) const {
        const T u = RED ? A[p] : B[p], f = RED ? fA[p] : fB[p];
        const T in = RED ? B[p] : A[p];
        const T uW = lane_prev(in), uE = lane_next(in);
        const T lo = p > 0 ? (RED ? B[p > 0 ? p - 1 : 0] : A[p > 0 ? p - 1 : 0]) : e;
        const T hi = p < P - 1 ? (RED ? B[p < P - 1 ? p + 1 : p] : A[p < P - 1 ? p + 1 : p]) : e;
        const T out = RED ? pick(s, hi, lo) : pick(s, lo, hi);
        ds = T(0);
        if constexpr (VAR) {
            const T* k = RED ? kA[p] : kB[p];
            return res_var2f(u, uW, uE, in, out, k[0], k[1], k[2], k[3], f, c, ds);
        } else if constexpr (OP == OP_STENCIL) {
            const T ci = RED ? si : so, co = RED ? so : si;
            const T t = (sc[1] * uW + sc[2] * uE) + (ci * in + co * out);
            return f - c * (sc[0] * u + t);
        } else {
            return res_lap2(u, uW, uE, in, out, f, c);
        }
    }
    template <bool RED>
    __device__ __forceinline__ void half() {
        const T e = RED ? *rdA : *rdB;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            T& u = RED ? A[p] : B[p];
            T ds;
            const T r = res<RED>(p, e, ds);
            const T v = stored<ST>(relax<T, VAR>(u, r, ds, c, wd, om));
            u = pick(RED ? inA[p] : inB[p], v, u);
        }
        if constexpr (RED) putA();
        else putB();
        __syncthreads();
    }
    __device__ __forceinline__ void residuals(T (&a)[P], T (&b)[P]) const {
        const T ea = *rdA, eb = *rdB;
        T ds;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            a[p] = pick(inA[p], res<true>(p, ea, ds), T(0));
            b[p] = pick(inB[p], res<false>(p, eb, ds), T(0));
        }
    }
    // the iterate's nodes of lanes l0 .. l1-1 and box rows q0 .. q1-1
    __device__ __forceinline__ void store(void* dst, int l0, int l1, int q0, int q1) const {
        const PlaneBuf<ST> b(gp((const ST*)dst), (size_t)n * n);
        T v[RT];
        rows(A, B, v);
        if (lane >= l0 && lane < l1 && gx >= 1 && gx <= n - 2) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                const int q = r0 + r, gy = ys + q;
                if (q >= q0 && q < q1 && gy >= 1 && gy <= n - 2) b.store(rb[r], (ST)v[r]);
            }
        }
    }
};

// FL: 0, SWEEP_ZERO_GUESS or SWEEP_NORM (FP64: also sums r^2 of the incoming
// iterate over the owned nodes).  Reads buffer 'sel', writes its partner.
template <typename ST, int OP, int FL, int P>
__global__ __launch_bounds__(64 * LW) void k_down2d(const GridDesc* __restrict__ descs, int sel, int ns) {
    using T = arith_t<ST>;
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    constexpr int CY = leg_cy(P), RT = 2 * P;
    __shared__ T E[LW + 2][2][BX];
    __shared__ T R[LW + 1][BX];  // residual of each wavefront's last row
    const int n = d.n, nc = (n - 1) / 2 + 1;
    const int ntx = (nc - 1 + LCX - 1) / LCX;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    // coarse nodes I0 .. I0+LCX-1 own fine columns 2I-1 and 2I (likewise rows)
    const int I0 = 1 + (tile % ntx) * LCX, J0 = 1 + (tile / ntx) * CY;
    LegBox<ST, OP, P> b;
    b.init(d, 2 * I0 - 6, 2 * J0 - 6, E);
    // owned: lanes 5 .. 5+2LCX-1, box rows 5 .. 5+2CY-1
    constexpr int L0 = 5, L1 = 5 + 2 * LCX, Q1 = 5 + 2 * CY;
    {
        T v[RT];
        if constexpr ((FL & SWEEP_ZERO_GUESS) != 0) {
#pragma unroll
            for (int r = 0; r < RT; ++r) v[r] = T(0);
        } else {
            b.load((sel & 1) ? d.t : d.u, v);
        }
        b.load_f(d);
        b.sort(v, b.A, b.B);
        b.putA();
        b.putB();
        __syncthreads();
    }
    T ra[P], rv[P], R4[RT];
    if constexpr ((FL & SWEEP_NORM) != 0) {
        b.residuals(ra, rv);
        b.rows(ra, rv, R4);
        double acc = 0.0;
#pragma unroll
        for (int r = 0; r < RT; ++r)
            if (b.lane >= L0 && b.lane < L1 && b.r0 + r >= L0 && b.r0 + r < Q1) acc += R4[r] * R4[r];
        __shared__ double red[LW];
        const double tot = block_sum_w<LW>(acc, red);  // a barrier: every wavefront has read its neighbours' rows
        if (threadIdx.x == 0) gp(d.npart)[blockIdx.x] = tot;
    }
    b.template half<true>();
    b.template half<false>();
    if (ns == 2) {
        b.template half<true>();
        b.template half<false>();
    }
    b.store((sel & 1) ? d.u : d.t, L0, L1, L0, Q1);
    b.residuals(ra, rv);
    b.rows(ra, rv, R4);
    R[b.w + 1][b.lane] = R4[RT - 1];
    __syncthreads();
    // full weighting at the even lanes' even rows (box lane 2(I - I0) + 6, likewise rows)
    T prev = R[b.w][b.lane];
    T prevx = lane_prev(prev) + lane_next(prev);
    const int I = I0 + (b.lane - 6) / 2;
    const bool coli = (b.lane & 1) == 0 && b.lane >= 6 && b.lane < 6 + 2 * LCX && I <= nc - 2;
    MG_GLOBAL ST* __restrict__ fc = gp((ST*)d.fc);
#pragma unroll
    for (int r = 0; r < RT; r += 2) {
        const T x0 = lane_prev(R4[r]) + lane_next(R4[r]), x1 = lane_prev(R4[r + 1]) + lane_next(R4[r + 1]);
        const T edges = x0 + (prev + R4[r + 1]);
        const T corners = prevx + x1;
        const T v = (T(0.25) * R4[r] + T(0.125) * edges) + T(0.0625) * corners;
        const int q = b.r0 + r, J = J0 + (q - 6) / 2;
        if (coli && q >= 6 && q < 6 + 2 * CY && J <= nc - 2) fc[(size_t)J * nc + I] = (ST)v;
        prev = R4[r + 1];
        prevx = x1;
    }
}

// Reads buffer 'sel' (bit 2: black first), writes its partner.
template <typename ST, int OP, int P>
__global__ __launch_bounds__(64 * LW) void k_up2d(const GridDesc* __restrict__ descs, int sel, int ns) {
    using T = arith_t<ST>;
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    constexpr int UY = leg_uy(P), RT = 2 * P;
    __shared__ T E[LW + 2][2][BX];
    const int n = d.n, nc = (n - 1) / 2 + 1;
    const int ntx = (n - 2 + LUX - 1) / LUX;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    LegBox<ST, OP, P> b;
    b.init(d, 1 + (tile % ntx) * LUX - 4, 1 + (tile / ntx) * UY - 4, E);
    T v[RT], e[P + 1];
    b.load((sel & 1) ? d.t : d.u, v);
    // Bilinear correction.  A box starts at odd x and y: a thread's rows are
    // odd, even, .. over P + 1 coarse rows; a lane loads its coarse column x/2
    // and at odd x takes the other one from the next lane (the last lane's x
    // is even).
    const PlaneBuf<ST> ec(gp((const ST*)d.uc), (size_t)nc * nc);
    const int cx = min(max(b.gx, 0), n - 1) >> 1, j0 = (b.ys + b.r0 - 1) / 2;
#pragma unroll
    for (int q = 0; q <= P; ++q)
        e[q] = (T)ec.load((unsigned)(min(max(j0 + q, 0), nc - 1) * nc + cx) * (unsigned)sizeof(ST));
    b.load_f(d);
    const bool xo = (b.gx & 1) != 0, coln = b.gx >= 1 && b.gx <= n - 2;
    T sx[P + 1];  // the coarse column's value, or the sum of the two at odd x
#pragma unroll
    for (int q = 0; q <= P; ++q) sx[q] = pick(xo, e[q] + lane_next(e[q]), e[q]);
    const T wo = pick(xo, T(0.25), T(0.5)), we = pick(xo, T(0.5), T(1));
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        const int gy = b.ys + b.r0 + r;
        const T corr = (r & 1) ? we * sx[r / 2 + 1] : wo * (sx[r / 2] + sx[r / 2 + 1]);
        if (gy >= 1 && gy <= n - 2) v[r] = pick(coln, stored<ST>(v[r] + corr), v[r]);
    }
    b.sort(v, b.A, b.B);
    b.putA();
    b.putB();
    __syncthreads();
    if (sel & SEL_BLACK_FIRST) {
        b.template half<false>();
        b.template half<true>();
        if (ns == 2) {
            b.template half<false>();
            b.template half<true>();
        }
    } else {
        b.template half<true>();
        b.template half<false>();
        if (ns == 2) {
            b.template half<true>();
            b.template half<false>();
        }
    }
    b.store((sel & 1) ? d.u : d.t, 4, 4 + LUX, 4, 4 + UY);
}

}  // namespace

namespace {
int down_tiles(int n, int P) {
    const int m = (n - 1) / 2;
    return cdiv(m, LCX) * cdiv(m, leg_cy(P));
}
template <typename T, int OPV, int P>
hipError_t down2d_op(const GridDesc* d, int ninst, int n, int sel, int ns, int flags, hipStream_t s) {
    const dim3 grid(down_tiles(n, P), ninst);
    switch (flags) {
        case 0: k_down2d<T, OPV, 0, P><<<grid, 64 * LW, 0, s>>>(d, sel, ns); break;
        case SWEEP_ZERO_GUESS: k_down2d<T, OPV, SWEEP_ZERO_GUESS, P><<<grid, 64 * LW, 0, s>>>(d, sel, ns); break;
        case SWEEP_NORM:
            if constexpr (sizeof(T) == 8) {
                k_down2d<T, OPV, SWEEP_NORM, P><<<grid, 64 * LW, 0, s>>>(d, sel, ns);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T, int OPV, int P>
hipError_t up2d_op(const GridDesc* d, int ninst, int n, int sel, int ns, hipStream_t s) {
    const dim3 grid(cdiv(n - 2, LUX) * cdiv(n - 2, leg_uy(P)), ninst);
    k_up2d<T, OPV, P><<<grid, 64 * LW, 0, s>>>(d, sel, ns);
    return hipGetLastError();
}
}  // namespace

// Row pairs per thread.  A taller box computes fewer nodes twice (it owns 52 of
// 64 rows against 20 of 32, going up 56 of 64 against 24 of 32), but there are
// fewer of them and their steps are longer: taken where the taller boxes alone
// cover the chip.  One 1025 x 1025 grid (400 boxes), FP32: down 7.5 us against
// 8.5, up 6.6 / 6.6; 513 x 513 (100 boxes): down 6.1 against 5.2; 22 grids of
// 1025 x 1025: down 60 against 94, up 68 against 75.  Variable coefficients
// keep four faces per node in registers: no taller boxes.
int leg_p(int op, int n, int ninst) {
    if (op == OP_VAR) return 2;
    return down_tiles(n, 4) * ninst >= 256 ? 4 : 2;
}

int down2d_tiles(int op, int n) { return down_tiles(n, leg_p(op, n, 1)); }

template <typename T>
hipError_t launch_down2d(int op, const GridDesc* d, int ninst, int n, int sel, int ns, int flags, hipStream_t s) {
    if (n < 5 || n > kLegMaxN || ninst <= 0 || ns < 1 || ns > 2) return hipErrorInvalidValue;
    const bool tall = leg_p(op, n, ninst) == 4;
    if (op == OP_LAP)
        return tall ? down2d_op<T, OP_LAP, 4>(d, ninst, n, sel, ns, flags, s)
                    : down2d_op<T, OP_LAP, 2>(d, ninst, n, sel, ns, flags, s);
    if constexpr (sizeof(T) >= 4) {  // binary16 storage: Laplacian only
        if (op == OP_VAR) return down2d_op<T, OP_VAR, 2>(d, ninst, n, sel, ns, flags, s);
    }
    if constexpr (sizeof(T) == 8) {
        if (op == OP_STENCIL)
            return tall ? down2d_op<T, OP_STENCIL, 4>(d, ninst, n, sel, ns, flags, s)
                        : down2d_op<T, OP_STENCIL, 2>(d, ninst, n, sel, ns, flags, s);
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t launch_up2d(int op, const GridDesc* d, int ninst, int n, int sel, int ns, hipStream_t s) {
    if (n < 5 || n > kLegMaxN || ninst <= 0 || ns < 1 || ns > 2) return hipErrorInvalidValue;
    const bool tall = leg_p(op, n, ninst) == 4;
    if (op == OP_LAP)
        return tall ? up2d_op<T, OP_LAP, 4>(d, ninst, n, sel, ns, s) : up2d_op<T, OP_LAP, 2>(d, ninst, n, sel, ns, s);
    if constexpr (sizeof(T) >= 4) {
        if (op == OP_VAR) return up2d_op<T, OP_VAR, 2>(d, ninst, n, sel, ns, s);
    }
    if constexpr (sizeof(T) == 8) {
        if (op == OP_STENCIL)
            return tall ? up2d_op<T, OP_STENCIL, 4>(d, ninst, n, sel, ns, s)
                        : up2d_op<T, OP_STENCIL, 2>(d, ninst, n, sel, ns, s);
    }
    return hipErrorInvalidValue;
}

#define MG_LEG(T)                                                                                      \
    template hipError_t launch_down2d<T>(int, const GridDesc*, int, int, int, int, int, hipStream_t);  \
    template hipError_t launch_up2d<T>(int, const GridDesc*, int, int, int, int, hipStream_t);
MG_LEG(double)
MG_LEG(float)
MG_LEG(half_t)
#undef MG_LEG

}  // namespace mg
