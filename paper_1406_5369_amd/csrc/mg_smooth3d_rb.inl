// 3D red-black sweeps of constant operators with one wavefront per tile, the
// tile's nodes in registers, held by colour (included by mg_smooth3d.inl).
#pragma once

namespace mg {
namespace {

// ---------------------------------------------------------------------------
// A wavefront marches a 64 x 2P box along z; lane = x position, the thread
// holds the rows of its column as P row pairs (rows 2p, 2p+1).  Colours
// alternate along x and y, so of each pair a lane holds one node of each
// colour: A the one the first half-sweep relaxes, B the other.  A half-sweep
// then updates one register per pair on every lane, and finds its neighbours
// in registers of the other colour without a choice, but for one:
//   x  the same row of the adjacent lanes holds the other colour: their B[p]
//   z  so does the same node of the adjacent planes: their B[p]
//   y  the pair's own B[p], and one node of the pair above (p+1) or below
//      (p-1), by the lane's parity
// (likewise from A for the second half-sweep).  What bounds these sweeps is
// memory, with vector-ALU issue behind it (129^3 FP64: 4.9 TB/s, issue 0.27 of
// the time; the two sweeps from zero below at 513^3 FP32: 1.62 GB at 5.6 TB/s,
// 0.52): 12 lane operations per update and 4 per node to sort rows into colours
// and back, where the form that keeps rows (both colours evaluated in every
// half-sweep, one kept) spends twice that.  No LDS, no barrier.
//
// s: the lane's A node of the plane is in the pair's second row; it flips
// from plane to plane.  YE: the box has rows that are not inner rows (its
// code alone checks them).
// ---------------------------------------------------------------------------
template <typename ST, int OP, int P, bool YE>
struct PairTile {
    using T = arith_t<ST>;
    static_assert(OP != OP_VAR, "constant operators");
    static constexpr bool CC = OP == OP_CC;
    static constexpr int LO = CC ? 0 : 1;  // first unknown of an axis (the last is n - 1 - LO)
    int n, lane, gx, y0r;  // y0r: y of row 0
    T c, wd;
    T sc[7];
    T wl[3];               // cells: the relaxation weights of the lane's cells with 0, 1, 2 boundary faces in y and z
    bool coli;
    unsigned rb[2 * P];  // byte offset of the lane's node of each row in a plane (clamped)
    size_t pl;

    __device__ __forceinline__ int gy(int r) const { return y0r + r; }  // wave-uniform
    __device__ __forceinline__ bool yin(int r) const { return !YE || (gy(r) >= LO && gy(r) <= n - 1 - LO); }
    __device__ __forceinline__ bool zin(int z) const { return z >= LO && z <= n - 1 - LO; }

    __device__ __forceinline__ void init(const GridDesc& d, int gx_, int y0r_) {
        n = d.n;
        lane = threadIdx.x & 63;
        gx = gx_;
        y0r = y0r_;
        c = (T)d.c;
        wd = (T)d.wd;
        load_stencil<OP>(d, sc);
        coli = gx >= LO && gx <= n - 1 - LO;
        if constexpr (CC) {
            const bool xb = gx == 0 || gx == n - 1;
#pragma unroll
            for (int m = 0; m < 3; ++m) wl[m] = pick(xb, (T)d.sc[m + 1], (T)d.sc[m]);
        }
        pl = (size_t)n * n;
        const int xc = min(max(gx, 0), n - 1);
#pragma unroll
        for (int r = 0; r < 2 * P; ++r)
            rb[r] = (unsigned)(min(max(gy(r), 0), n - 1) * n + xc) * (unsigned)sizeof(ST);
    }
    // Rows R0 .. R1-1 of plane z from clamped (always in-bounds) addresses;
    // values at positions outside the grid are never used.
    template <int R0, int R1>
    __device__ __forceinline__ void load(const MG_GLOBAL ST* __restrict__ a, int z, T (&dst)[2 * P]) const {
        const PlaneBuf<ST> b(a + (size_t)min(max(z, 0), n - 1) * pl, pl);
#pragma unroll
        for (int r = R0; r < R1; ++r) dst[r] = (T)b.load(rb[r]);
    }
    static __device__ __forceinline__ void sort(const T (&raw)[2 * P], bool s, T (&A)[P], T (&B)[P]) {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T r0 = raw[2 * p], r1 = raw[2 * p + 1];
            A[p] = pick(s, r1, r0);
            B[p] = pick(s, r0, r1);
        }
    }
    // Residual at the nodes X[p] of plane z: O, Ob, Oa the other colour of the
    // plane, the planes below and above; up: the lane's node is in the pair's
    // second row (its third y-neighbour is in pair p + 1).  A cell's neighbour
    // outside the domain takes the cell's own value.
    // ed: what the first and last pair take for the neighbour outside the tile.
    __device__ __forceinline__ T res(const T (&X)[P], const T (&O)[P], const T (&Ob)[P], const T (&Oa)[P], T f, bool up,
                                     int z, int p, T ed) const {
        T w = lane_prev(O[p]), e = lane_next(O[p]);
        const T hi = O[p + 1 < P ? p + 1 : p], lo = O[p > 0 ? p - 1 : p];
        T y = pick(up, p + 1 < P ? hi : ed, p > 0 ? lo : ed);
        T b = Ob[p], a = Oa[p];
        if constexpr (CC) {
            w = pick(gx == 0, X[p], w);
            e = pick(gx == n - 1, X[p], e);
            if constexpr (YE) y = pick(up ? gy(2 * p + 1) == n - 1 : gy(2 * p) == 0, X[p], y);
            b = pick(z == 0, X[p], b);
            a = pick(z == n - 1, X[p], a);
        }
        if constexpr (OP == OP_STENCIL) {
            const T so = pick(up, sc[3], sc[4]), sy = pick(up, sc[4], sc[3]);
            T t = (sc[1] * w + sc[2] * e) + (so * O[p] + sy * y);
            t = t + (sc[5] * b + sc[6] * a);
            return f - c * (sc[0] * X[p] + t);
        } else {
            return res_lap3(X[p], w, e, O[p], y, b, a, f, c);
        }
    }
    __device__ __forceinline__ T res(const T (&X)[P], const T (&O)[P], const T (&Ob)[P], const T (&Oa)[P], T f, bool up,
                                     int z, int p) const {
        return res(X, O, Ob, Oa, f, up, z, p, O[p]);
    }
    // The relaxed value of u at a node of pair p, plane z, with residual r.
    __device__ __forceinline__ T relaxed(T u, T r, bool up, int z, int p) const {
        T k = wd;
        if constexpr (CC) {
            const bool zb = z == 0 || z == n - 1;
            const T k0 = pick(zb, wl[1], wl[0]), k1 = pick(zb, wl[2], wl[1]);
            k = k0;
            if constexpr (YE) k = pick(up ? gy(2 * p + 1) == n - 1 : gy(2 * p) == 0, k1, k0);
        }
        return stored<ST>(relax<T, false>(u, r, T(0), c, k, T(0)));
    }
    // The lane's node X[p] is an inner node of an inner plane.
    __device__ __forceinline__ bool inner(bool up, int p) const { return coli && (up ? yin(2 * p + 1) : yin(2 * p)); }
};

// A tile whose incoming planes take the coarse-grid correction P uc (PRO), in
// order of z.
template <typename ST, int OP, int P, bool PRO, bool YE>
struct CorrectedTile : PairTile<ST, OP, P, YE> {
    using Base = PairTile<ST, OP, P, YE>;
    using T = arith_t<ST>;
    using Base::CC, Base::coli, Base::gx, Base::n, Base::yin, Base::y0r;

    // ---- coarse-grid correction: row 0 has odd y, lane 0 odd x, so pair p
    // needs coarse rows p (with p+1 for its first, odd row) and p+1, counted
    // from j0, and an odd-x lane its own column x/2 and the next lane's.
    const MG_GLOBAL ST* __restrict__ ec;
    int nc;
    unsigned cxb;
    T cr[PRO ? P + 1 : 1];      // the pending coarse plane's rows
    T sy[PRO ? 2 * P : 1];      // x-then-y sums of the latest completed coarse plane, per row
    T wx[3];                    // weights by the number of odd coordinates beside x

    __device__ __forceinline__ void issue_c(int K) {
        const PlaneBuf<ST> b(ec + (size_t)min(max(K, 0), nc - 1) * ((size_t)nc * nc), (size_t)nc * nc);
#pragma unroll
        for (int j = 0; j <= P; ++j)
            cr[j] = (T)b.load(cxb + (unsigned)(min(max((y0r >> 1) + j, 0), nc - 1) * nc) * (unsigned)sizeof(ST));
    }
    __device__ __forceinline__ void coarse_sums(T (&out)[2 * P]) const {
        const bool xo = (gx & 1) != 0;
        T xs[P + 1];
#pragma unroll
        for (int j = 0; j <= P; ++j) {
            const T a = cr[j], an = lane_next(a);
            xs[j] = xo ? a + an : a;
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            out[2 * p] = xs[p] + xs[p + 1];
            out[2 * p + 1] = xs[p + 1];
        }
    }
    // Cells: both rows of a pair, both lanes of an x pair and planes 2K, 2K+1 have one parent.
    __device__ __forceinline__ void correct_cells(int kk, bool zo, T (&raw)[2 * P]) {
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) raw[r] = raw[r] + cr[r / 2];
        if (zo) issue_c((kk + 1) >> 1);
    }
    __device__ __forceinline__ void correct_entering(int kk, bool zo, T (&raw)[2 * P]) {
        const bool zin = this->zin(kk);
        T sum[2 * P];
        if (zo) {
            T sn[2 * P];
            coarse_sums(sn);
#pragma unroll
            for (int r = 0; r < 2 * P; ++r) {
                sum[r] = sy[r] + sn[r];
                sy[r] = sn[r];
            }
        } else {
#pragma unroll
            for (int r = 0; r < 2 * P; ++r) sum[r] = sy[r];
            issue_c((kk + 2) >> 1);
        }
        const T w1 = zo ? wx[1] : wx[0], w2 = zo ? wx[2] : wx[1];
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) {
            const T v = stored<ST>(raw[r] + ((r & 1) ? w1 : w2) * sum[r]);
            raw[r] = pick(zin && coli && yin(r), v, raw[r]);
        }
    }

    // zo: kk is odd
    __device__ __forceinline__ void correct(int kk, bool zo, T (&raw)[2 * P]) {
        if constexpr (CC) correct_cells(kk, zo, raw);
        else correct_entering(kk, zo, raw);
    }
    // before plane kk, the march's first
    __device__ __forceinline__ void correct_start(int kk) {
        cxb = (unsigned)(min(max(gx, 0), n - 1) >> 1) * (unsigned)sizeof(ST);
        if constexpr (CC) {
            issue_c(kk >> 1);
        } else {
            T w = (gx & 1) ? T(0.5) : T(1);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                wx[q] = w;
                w = T(0.5) * w;
            }
            // plane kk needs the coarse plane kk/2 (rounded down) completed, and for odd kk the next one pending
            issue_c((kk - (kk & 1)) >> 1);
            coarse_sums(sy);
            if (kk & 1) issue_c((kk + 1) >> 1);
        }
    }
};

// One red-black sweep.  Step kk (plane kk enters): the first colour on plane
// kk-1, the second on plane kk-2, written out.  FL: 0, SWEEP_ZERO_GUESS,
// SWEEP_PROLONG (the incoming iterate is u + P uc) or, on cells, SWEEP_NORM
// (the incoming iterate is u - mean; sums its r^2 over the output cells).
template <typename ST, int OP, int P, int FL, bool YE>
struct SweepRB : CorrectedTile<ST, OP, P, (FL & SWEEP_PROLONG) != 0, YE> {
    using Base = CorrectedTile<ST, OP, P, (FL & SWEEP_PROLONG) != 0, YE>;
    using T = arith_t<ST>;
    using Base::c, Base::coli, Base::gx, Base::gy, Base::lane, Base::n, Base::pl, Base::rb, Base::yin, Base::y0r;
    static constexpr int H = 2, TX = BX - 2 * H, TY = 2 * P - 2 * H;
    static constexpr bool PRO = (FL & SWEEP_PROLONG) != 0, NRM = (FL & SWEEP_NORM) != 0, CC = OP == OP_CC;
    static constexpr bool ZG = (FL & SWEEP_ZERO_GUESS) != 0;
    using Storage = ST;

    const MG_GLOBAL ST* __restrict__ uin;
    MG_GLOBAL ST* __restrict__ uout;
    const MG_GLOBAL ST* __restrict__ f;
    int z0, z1;
    bool s;  // of plane kk
    T raw[2 * P], rawf[2 * P];             // plane kk+1 of u, plane kk of f (in flight)
    T A[4][P], B[4][P], fA[4][P], fB[4][P];  // slot = plane mod 4 (dead slots take no registers)
    T Ao[NRM ? P : 1];                     // first-colour nodes of plane kk-2 before their update
    T mean;
    double acc;

    template <int Q>
    __device__ __forceinline__ void step(int kk) {
        constexpr int Q0 = Q & 3, Q1 = (Q + 3) & 3, Q2 = (Q + 2) & 3, Q3 = (Q + 1) & 3;  // planes kk .. kk-3
        s = !s;
        if constexpr (PRO) this->correct(kk, (kk & 1) != 0, raw);
        if constexpr (NRM) {
#pragma unroll
            for (int r = 0; r < 2 * P; ++r) raw[r] = raw[r] - mean;
        }
        Base::sort(raw, s, A[Q0], B[Q0]);
        if constexpr (!ZG) this->template load<0, 2 * P>(uin, kk + 1, raw);
        // f of plane kk-1 (issued one step ago)
        Base::sort(rawf, !s, fA[Q1], fB[Q1]);
        this->template load<1, 2 * P - 1>(f, kk, rawf);
        const int m1 = kk - 1, m2 = kk - 2;
        const bool tile = coli && lane >= H && lane <= BX - 1 - H;
        if constexpr (NRM) {
            // r of the second colour on the incoming values
            if (m1 >= z0 && m1 < z1) {
#pragma unroll
                for (int p = 1; p < P - 1; ++p) {
                    const T r = this->res(B[Q1], A[Q1], Ao, A[Q0], fB[Q1][p], s, m1, p);
                    if (tile && this->inner(s, p)) acc += r * r;
                }
            }
#pragma unroll
            for (int p = 0; p < P; ++p) Ao[p] = A[Q1][p];
        }
        if (m1 >= z0 - 1 && this->zin(m1)) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const T r = this->res(A[Q1], B[Q1], B[Q2], B[Q0], fA[Q1][p], !s, m1, p);
                const bool in = this->inner(!s, p);
                if constexpr (NRM) {
                    if (p >= 1 && p < P - 1 && m1 >= z0 && m1 < z1 && tile && in) acc += r * r;
                }
                A[Q1][p] = pick(in, this->relaxed(A[Q1][p], r, !s, m1, p), A[Q1][p]);
            }
        }
        if (m2 >= z0 && m2 < z1) {
            const PlaneBuf<ST> out(uout + (size_t)m2 * pl, pl);
#pragma unroll
            for (int p = 1; p < P - 1; ++p) {
                const T r = this->res(B[Q2], A[Q2], A[Q3], A[Q1], fB[Q2][p], !s, m2, p);
                const T v = this->relaxed(B[Q2][p], r, !s, m2, p);
                if (tile && yin(2 * p)) out.store(rb[2 * p], (ST)pick(s, v, A[Q2][p]));
                if (tile && yin(2 * p + 1)) out.store(rb[2 * p + 1], (ST)pick(s, A[Q2][p], v));
            }
        }
    }

    __device__ __forceinline__ void run(int cfirst) {
        int kk = z0 - H;
        const int kend = z1 - 1 + H;
        // of plane kk - 1 (step flips it first): row 0's node has the first colour when its coordinates say so
        s = ((gx + y0r + kk + cfirst) & 1) == 0;
        // values of planes before the march are never used (the conditions of the half-sweeps)
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) raw[r] = rawf[r] = T(0);
        acc = 0.0;
        if constexpr (NRM) {
#pragma unroll
            for (int p = 0; p < P; ++p) A[3][p] = T(0);
        }
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
        }
    }
};

template <typename S>
__device__ __forceinline__ void sweep_rb_tile(const GridDesc& d, int sel, int zchunk, int tx, int ty, int tz) {
    S t;
    const int n = d.n;
    using ST = typename S::Storage;
    t.init(d, S::LO + tx * S::TX - S::H + (int)threadIdx.x, S::LO + ty * S::TY - S::H);
    t.z0 = S::LO + tz * zchunk;
    t.z1 = min(t.z0 + zchunk, n - S::LO);
    t.uin = gp((const ST*)((sel & 1) ? d.t : d.u));
    t.uout = gp((ST*)((sel & 1) ? d.u : d.t));
    t.f = gp((const ST*)d.f);
    t.ec = gp((const ST*)d.uc);
    t.nc = S::CC ? n / 2 : (n - 1) / 2 + 1;
    if constexpr (S::NRM) t.mean = *gp(d.mean);
    t.run((sel & SEL_BLACK_FIRST) ? 1 : 0);
    if constexpr (S::NRM) {
        // per-workgroup partial in a fixed order (finalised in block order)
        double v = t.acc;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
        if (threadIdx.x == 0) gp(d.npart)[blockIdx.x] = v;
    }
}

template <typename ST, int OP, int BY, int FL>
__global__ __launch_bounds__(64) void k_smooth3d_rb(const GridDesc* __restrict__ descs, int sel, int zchunk) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    using S = SweepRB<ST, OP, BY / 2, FL, false>;
    const int n = d.n, m = n - 2 * S::LO;
    const int ntx = (m + S::TX - 1) / S::TX, nty = (m + S::TY - 1) / S::TY;
    const int tile = sweep_tile(sel, blockIdx.x, gridDim.x);
    const int tx = tile % ntx, t2 = tile / ntx, ty = t2 % nty, tz = t2 / nty;
    const int y0r = S::LO + ty * S::TY - S::H;
    // a box without boundary rows (cells: rows whose neighbours all exist)
    if (y0r >= 1 && y0r + BY - 1 <= n - 2) sweep_rb_tile<S>(d, sel, zchunk, tx, ty, tz);
    else sweep_rb_tile<SweepRB<ST, OP, BY / 2, FL, true>>(d, sel, zchunk, tx, ty, tz);
}

// ---------------------------------------------------------------------------
// The first two red-black pre-smoothing sweeps of a level whose iterate starts
// at zero, in one launch.  The four half-sweeps trail each other by one plane:
// step kk (f of plane kk enters)
//   R1  red of plane kk:     wd f (the relaxation of a zero iterate)
//   B1  black of plane kk-1  from the red values R1 left
//   R2  red of plane kk-2    from the black values B1 left
//   B2  black of plane kk-3  from the red values R2 left; plane kk-3 is the output
// Half-sweep q (B1 = 1) is valid on the box minus q rings, so the output tile
// is the box minus three rings: 58 x (2P - 6) nodes.  The per-node expressions
// are those of two separate sweeps, stored values rounded in between.
// ---------------------------------------------------------------------------
template <typename ST, int P, bool YE>
struct Sweep2RB : PairTile<ST, OP_LAP, P, YE> {
    using Base = PairTile<ST, OP_LAP, P, YE>;
    using T = arith_t<ST>;
    using Base::c, Base::coli, Base::gx, Base::lane, Base::n, Base::pl, Base::rb, Base::yin, Base::y0r;
    using Storage = ST;
    static constexpr int H = 3, TX = BX - 2 * H, TY = 2 * P - 2 * H;
    static constexpr int R = 5;  // ring of planes kk-4 .. kk

    const MG_GLOBAL ST* __restrict__ f;
    MG_GLOBAL ST* __restrict__ uout;
    int z0, z1;
    bool s;  // of plane kk
    T rawf[2 * P];  // f of plane kk+1 (in flight)
    T A[R][P], B[R][P], fA[R][P], fB[R][P];

    template <int Q>
    __device__ __forceinline__ void step(int kk) {
        constexpr int Q0 = Q, Q1 = (Q + 4) % R, Q2 = (Q + 3) % R, Q3 = (Q + 2) % R, Q4 = (Q + 1) % R;
        s = !s;
        Base::sort(rawf, s, fA[Q0], fB[Q0]);
        this->template load<0, 2 * P>(f, kk + 1, rawf);
        const bool zin = kk >= 1 && kk <= n - 2;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const T zero = T(0);
            const T r = res_lap3(zero, zero, zero, zero, zero, zero, zero, fA[Q0][p], c);
            const T v = this->relaxed(zero, r, s, kk, p);
            A[Q0][p] = (zin && this->inner(s, p)) ? v : zero;
            B[Q0][p] = zero;
        }
        const int p1 = kk - 1, p2 = kk - 2, p3 = kk - 3;
        if (p1 >= z0 - 2 && p1 >= 1 && p1 <= n - 2) {
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const T v = this->relaxed(T(0), this->res(B[Q1], A[Q1], A[Q2], A[Q0], fB[Q1][p], s, p1, p), s, p1, p);
                B[Q1][p] = this->inner(s, p) ? v : T(0);
            }
        }
        if (p2 >= z0 - 1 && p2 >= 1 && p2 <= n - 2) {
#pragma unroll
            for (int p = 1; p < P - 1; ++p) {
                const T v = this->relaxed(A[Q2][p], this->res(A[Q2], B[Q2], B[Q3], B[Q1], fA[Q2][p], s, p2, p), s, p2, p);
                A[Q2][p] = pick(this->inner(s, p), v, A[Q2][p]);
            }
        }
        if (p3 >= z0 && p3 < z1) {
            const bool ok = coli && lane >= H && lane <= BX - 1 - H;
            const PlaneBuf<ST> out(uout + (size_t)p3 * pl, pl);
#pragma unroll
            for (int p = 1; p < P - 1; ++p) {
                // plane kk-3 has the other parity: its second colour is in the pair's second row where s holds
                const T v = this->relaxed(B[Q3][p], this->res(B[Q3], A[Q3], A[Q4], A[Q2], fB[Q3][p], s, p3, p), s, p3, p);
                if (p > 1 && ok && yin(2 * p)) out.store(rb[2 * p], (ST)pick(s, A[Q3][p], v));
                if (p == 1 && ok && yin(2 * p + 1)) out.store(rb[2 * p + 1], (ST)pick(s, v, A[Q3][p]));
                if (p > 1 && p < P - 2 && ok && yin(2 * p + 1))
                    out.store(rb[2 * p + 1], (ST)pick(s, v, A[Q3][p]));
            }
        }
    }

    __device__ __forceinline__ void run() {
        int kk = z0 - H;
        const int kend = z1 - 1 + H;
        s = ((gx + y0r + kk) & 1) == 0;  // of plane kk - 1
        this->template load<0, 2 * P>(f, kk, rawf);
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
        }
    }
};

template <typename S>
__device__ __forceinline__ void sweep2_rb_tile(const GridDesc& d, int sel, int zchunk, int tx, int ty, int tz) {
    S t;
    using ST = typename S::Storage;
    t.init(d, 1 + tx * S::TX - S::H + (int)threadIdx.x, 1 + ty * S::TY - S::H);
    t.z0 = 1 + tz * zchunk;
    t.z1 = min(t.z0 + zchunk, d.n - 1);
    // the second sweep's output buffer (its input is the first sweep's, which
    // never leaves the registers)
    t.uout = gp((ST*)((sel & 1) ? d.u : d.t));
    t.f = gp((const ST*)d.f);
    t.run();
}

template <typename ST, int BY>
__global__ __launch_bounds__(64) void k_smooth3d_zg2(const GridDesc* __restrict__ descs, int sel, int zchunk) {
    const GridDesc& d = descs[blockIdx.y];
    if (d.done && *gp(d.done)) return;
    using S = Sweep2RB<ST, BY / 2, false>;
    const int n = d.n;
    const int ntx = (n - 2 + S::TX - 1) / S::TX, nty = (n - 2 + S::TY - 1) / S::TY;
    const int tile = sweep_tile(sel, blockIdx.x, gridDim.x);
    const int tx = tile % ntx, t2 = tile / ntx, ty = t2 % nty, tz = t2 / nty;
    const int y0r = 1 + ty * S::TY - S::H;
    if (y0r >= 1 && y0r + BY - 1 <= n - 2) sweep2_rb_tile<S>(d, sel, zchunk, tx, ty, tz);
    else sweep2_rb_tile<Sweep2RB<ST, BY / 2, true>>(d, sel, zchunk, tx, ty, tz);
}

}  // namespace
}  // namespace mg
