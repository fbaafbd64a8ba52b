// 3D: two red-black sweeps of a constant operator in one launch (included by
// mg_smooth3d.inl).
#pragma once

namespace mg {
namespace {

// A workgroup marches a 64 x 2 P LW box along z, its LW wavefronts stacked in
// y, the nodes of a wavefront's 2 P rows in registers by colour (PairTile).
// The four half-sweeps trail each other by one plane; step kk (plane kk
// enters):
//   first sweep   A of plane kk-1, B of plane kk-2
//   second sweep  A of plane kk-3, B of plane kk-4, which is the output
// and each is valid on one ring less, so the box owns 56 x (2 P LW - 8) nodes.
// A half-sweep's neighbours along z are the thread's own registers, and what
// it needs of the rows next to its wavefront's was final one step ago: a step
// ends with four words per lane put into LDS (of each half-sweep's operand the
// row that the adjacent wavefront will ask for, by the lane's parity) and one
// barrier.
//
// Two sweeps apart read u and f and write u twice; here once.  What bounds this
// kernel on large grids is memory: at 513^3 FP32 it moves 2.96 GB (1.67 needed;
// halo rows and planes miss L2) at 5.9 TB/s, next to vector-ALU issue for half of
// the time (40 .. 50 operations per row and plane for the four half-sweeps, 1.5
// times over for the rings).  On fewer boxes it is the 2 .. 4 wavefronts per
// SIMD (the ring of planes is 100 .. 216 registers), too few to cover either:
// 257^3 FP64 4.5 TB/s, issue 0.4.  So the steps have no branches but the
// output's, and the plane's parity is known where a step is compiled.
// Measured: 513^3 FP32 correction and two sweeps 489 us against 452 + 379 apart
// (270 us at 6.2 TB/s for the bytes needed); 257^3 FP64 with the norm 110 us
// against 113 + 93, with the correction 108 against 115 + 93 (66 us).
// Boxes of 64 rows (four pairs per thread): 520 us at 513^3; loading two planes
// ahead: 511 us.
//
// FL: 0, SWEEP_ZERO_GUESS, SWEEP_PROLONG (the incoming iterate is u + P uc) or
// SWEEP_NORM (FP64; sums r^2 of the incoming iterate; cells: of u - mean).
template <typename ST, int OP, int P, int LW, int FL, bool YE>
struct Sweep2X : CorrectedTile<ST, OP, P, (FL & SWEEP_PROLONG) != 0, YE> {
    using Base = CorrectedTile<ST, OP, P, (FL & SWEEP_PROLONG) != 0, YE>;
    using T = arith_t<ST>;
    using Storage = ST;
    using Base::coli, Base::gx, Base::lane, Base::n, Base::pl, Base::rb, Base::yin, Base::y0r;
    static constexpr bool PRO = (FL & SWEEP_PROLONG) != 0, NRM = (FL & SWEEP_NORM) != 0, CC = OP == OP_CC;
    static constexpr bool ZG = (FL & SWEEP_ZERO_GUESS) != 0;
    static constexpr int H = 4, TX = BX - 2 * H, LB = 2 * P * LW, TY = LB - 2 * H;
    static constexpr int R = 6;   // ring of planes kk-5 .. kk
    static constexpr int NX = NRM ? 5 : 4;
    static constexpr bool KO = !CC;  // the march starts at an odd plane
    using Exchange = T[2][NX][LW + 2][BX];

    const MG_GLOBAL ST* __restrict__ uin;
    MG_GLOBAL ST* __restrict__ uout;
    const MG_GLOBAL ST* __restrict__ f;
    T* ex;  // this lane's word of the first exchange
    int w, z0, z1;
    bool s;                                // A of plane kk is in its pair's second row
    T raw[2 * P], rawf[2 * P];             // plane kk+1 of u, plane kk of f (in flight)
    T A[R][P], B[R][P], fA[R][P], fB[R][P];  // slot = plane mod 6 (dead slots take no registers)
    T Ao[NRM ? P : 1];                     // A of plane kk-2 before its update
    T mean;
    double acc;

    static __device__ __forceinline__ constexpr int at(int buf, int x) { return (buf * NX + x) * (LW + 2) * BX; }
    // row r of the wavefront's is one the box owns
    __device__ __forceinline__ bool own(int r) const { return 2 * P * w + r >= H && 2 * P * w + r < LB - H; }

    template <int Q>
    __device__ __forceinline__ void step(int kk) {
        constexpr int Q0 = Q, Q1 = (Q + 5) % R, Q2 = (Q + 4) % R, Q3 = (Q + 3) % R, Q4 = (Q + 2) % R, Q5 = (Q + 1) % R;
        constexpr int buf = Q & 1;
        s = !s;
        // half-sweeps of this step relax nodes in the second row where !s
        const T* rd = ex + (s ? -BX : BX);
        T e[NX];
#pragma unroll
        for (int x = 0; x < 4; ++x) e[x] = rd[at(buf ^ 1, x)];
        if constexpr (NRM) e[4] = ex[at(buf ^ 1, 4) + (s ? BX : -BX)];
        if constexpr (PRO) this->correct(kk, buf == 0 ? KO : !KO, raw);
        if constexpr (NRM && CC) {
#pragma unroll
            for (int r = 0; r < 2 * P; ++r) raw[r] = raw[r] - mean;
        }
        Base::sort(raw, s, A[Q0], B[Q0]);
        if constexpr (!ZG) this->template load<0, 2 * P>(uin, kk + 1, raw);
        // f of plane kk-1 (issued one step ago)
        Base::sort(rawf, !s, fA[Q1], fB[Q1]);
        this->template load<0, 2 * P>(f, kk, rawf);
        const int m1 = kk - 1, m2 = kk - 2, m3 = kk - 3, m4 = kk - 4;
        const bool tile = coli && lane >= H && lane <= BX - 1 - H;
        const bool z1in = this->zin(m1), z2in = this->zin(m2), z3in = this->zin(m3);
        if constexpr (NRM) {
            const bool own1 = tile && m1 >= z0 && m1 < z1;
#pragma unroll
            for (int p = 0; p < P; ++p) {  // r of B on the incoming values
                const T r = this->res(B[Q1], A[Q1], Ao, A[Q0], fB[Q1][p], s, m1, p, e[4]);
                const bool o = own1 && this->inner(s, p) && pick(s, own(2 * p + 1), own(2 * p));
                acc += pick(o, r * r, T(0));
            }
#pragma unroll
            for (int p = 0; p < P; ++p) Ao[p] = A[Q1][p];
        }
        T edge4 = T(0);
        if constexpr (NRM) edge4 = pick(s, A[Q0][P - 1], A[Q0][0]);
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T r = this->res(A[Q1], B[Q1], B[Q2], B[Q0], fA[Q1][p], !s, m1, p, e[0]);
            const bool in = z1in && this->inner(!s, p);
            if constexpr (NRM) {
                const bool o = tile && m1 >= z0 && m1 < z1 && in && pick(s, own(2 * p), own(2 * p + 1));
                acc += pick(o, r * r, T(0));
            }
            A[Q1][p] = pick(in, this->relaxed(A[Q1][p], r, !s, m1, p), A[Q1][p]);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T r = this->res(B[Q2], A[Q2], A[Q3], A[Q1], fB[Q2][p], !s, m2, p, e[1]);
            B[Q2][p] = pick(z2in && this->inner(!s, p), this->relaxed(B[Q2][p], r, !s, m2, p), B[Q2][p]);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T r = this->res(A[Q3], B[Q3], B[Q4], B[Q2], fA[Q3][p], !s, m3, p, e[2]);
            A[Q3][p] = pick(z3in && this->inner(!s, p), this->relaxed(A[Q3][p], r, !s, m3, p), A[Q3][p]);
        }
        T v[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T r = this->res(B[Q4], A[Q4], A[Q5], A[Q3], fB[Q4][p], !s, m4, p, e[3]);
            v[p] = this->relaxed(B[Q4][p], r, !s, m4, p);
        }
        if (m4 >= z0 && m4 < z1) {
            const PlaneBuf<ST> out(uout + (size_t)m4 * pl, pl);
#pragma unroll
            for (int p = 0; p < P; ++p) {
                if (tile && own(2 * p) && yin(2 * p)) out.store(rb[2 * p], (ST)pick(s, v[p], A[Q4][p]));
                if (tile && own(2 * p + 1) && yin(2 * p + 1)) out.store(rb[2 * p + 1], (ST)pick(s, A[Q4][p], v[p]));
            }
        }
        ex[at(buf, 0)] = pick(s, B[Q0][0], B[Q0][P - 1]);
        ex[at(buf, 1)] = pick(s, A[Q1][0], A[Q1][P - 1]);
        ex[at(buf, 2)] = pick(s, B[Q2][0], B[Q2][P - 1]);
        ex[at(buf, 3)] = pick(s, A[Q3][0], A[Q3][P - 1]);
        if constexpr (NRM) ex[at(buf, 4)] = edge4;
        __syncthreads();
    }

    __device__ __forceinline__ void run(int cfirst) {
        // from an odd plane (cells: an even one), so that the parity of a step's
        // plane is known where it is compiled
        int kk = z0 - H;
        if (((kk & 1) != 0) != KO) --kk;
        const int kend = z1 - 1 + H;
        s = ((gx + y0r + kk + cfirst) & 1) == 0;  // of plane kk - 1 (step flips it first)
        // Planes before the march: what is computed from them is what the
        // half-sweeps' shrinking ranges leave out.
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) raw[r] = rawf[r] = T(0);
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
            for (int p = 0; p < P; ++p) A[q][p] = B[q][p] = fA[q][p] = fB[q][p] = T(0);
        acc = 0.0;
        if constexpr (PRO) this->correct_start(kk);
        if constexpr (!ZG) this->template load<0, 2 * P>(uin, kk, raw);
        for (;;) {
            step<0>(kk);
            if (++kk > kend) break;
            step<1>(kk);
            if (++kk > kend) break;
            step<2>(kk);
            if (++kk > kend) break;
            step<3>(kk);
            if (++kk > kend) break;
            step<4>(kk);
            if (++kk > kend) break;
            step<5>(kk);
            if (++kk > kend) break;
        }
    }
};

template <typename S, int P, int LW>
__device__ __forceinline__ void sweep_x2_tile(const GridDesc& d, int sel, int zchunk, int tx, int ty, int tz,
                                              typename S::Exchange& E) {
    S t;
    using ST = typename S::Storage;
    const int n = d.n;
    t.w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    t.init(d, S::LO + tx * S::TX - S::H + (int)(threadIdx.x & 63), S::LO + ty * S::TY - S::H + 2 * P * t.w);
    t.ex = &E[0][0][t.w + 1][t.lane];
    t.z0 = S::LO + tz * zchunk;
    t.z1 = min(t.z0 + zchunk, n - S::LO);
    t.uin = gp((const ST*)((sel & 1) ? d.t : d.u));
    t.uout = gp((ST*)((sel & 1) ? d.u : d.t));
    t.f = gp((const ST*)d.f);
    t.ec = gp((const ST*)d.uc);
    t.nc = S::CC ? n / 2 : (n - 1) / 2 + 1;
    if constexpr (S::NRM && S::CC) t.mean = *gp(d.mean);
    t.run((sel & SEL_BLACK_FIRST) ? 1 : 0);
    if constexpr (S::NRM) {
        __shared__ double red[LW];
        const double tot = block_sum_w<LW>(t.acc, red);
        if (threadIdx.x == 0) gp(d.npart)[blockIdx.x] = tot;
    }
}

template <typename ST, int OP, int P, int LW, int FL>
__global__ __launch_bounds__(64 * LW) void k_smooth3d_x2(const GridDesc* __restrict__ descs, int sel, int zchunk) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    using S = Sweep2X<ST, OP, P, LW, FL, false>;
    __shared__ typename S::Exchange E;
    const int n = d.n, m = n - 2 * S::LO;
    const int ntx = (m + S::TX - 1) / S::TX, nty = (m + S::TY - 1) / S::TY;
    const int tile = sweep_tile(sel, blockIdx.x, gridDim.x);
    const int tx = tile % ntx, t2 = tile / ntx, ty = t2 % nty, tz = t2 / nty;
    const int y0r = S::LO + ty * S::TY - S::H;
    // a box without boundary rows (cells: rows whose neighbours all exist)
    if (y0r >= 1 && y0r + S::LB - 1 <= n - 2) sweep_x2_tile<S, P, LW>(d, sel, zchunk, tx, ty, tz, E);
    else sweep_x2_tile<Sweep2X<ST, OP, P, LW, FL, true>, P, LW>(d, sel, zchunk, tx, ty, tz, E);
}

}  // namespace
}  // namespace mg
