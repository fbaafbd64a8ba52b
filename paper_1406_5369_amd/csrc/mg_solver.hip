// Solver core: the V-cycle driver of Algorithm 1 over groups of equal-size
// grids, default launch geometry, and helper kernels for hierarchy setup.
#include <algorithm>
#include <cstdlib>
#include <cstring>

#include "mg_cc.h"
#include "mg_solver.h"

namespace mg {

size_t npts(int dim, int n) { return dim == 2 ? (size_t)n * n : (size_t)n * n * n; }

int count_levels(int n) {
    int L = 1;
    while (n > 3) {
        n = (n - 1) / 2 + 1;
        ++L;
    }
    return L;
}

int heuristic_zchunk(int dim, int n, int by, int halo, int target_blocks) {
    if (dim == 2) return 1;
    const int m = n - 2;
    const int TX = 64 - 2 * halo, TY = by - 2 * halo;
    const int cols = ((m + TX - 1) / TX) * ((m + TY - 1) / TY);
    const int chunks = std::max(1, (target_blocks + cols - 1) / cols);
    return std::max(2, (m + chunks - 1) / chunks);
}

Tiles lds_tiles(int dim, int n, int smoother) {
    Tiles t;
    const int H = smoother == SM_RBGS ? 2 : 1;
    const int target = 2048;
    if (dim == 2) {
        const int by = n >= 257 ? 32 : (n >= 65 ? 16 : 8);
        t.smooth = t.smooth_zg = t.smooth_pro = t.smooth_nrm = {by, 1};
        t.restr = {by < 16 ? 16 : by, 1};
        t.norm = {by, 1};
        return t;
    }
    // two rows per thread: within the register limit of every precision
    const int by = n >= 129 ? 16 : 8;
    t.smooth = t.smooth_zg = t.smooth_pro = t.smooth_nrm = {by, heuristic_zchunk(3, n, by, H, target), 1,
                                                           by >= 16 ? 8 : 4};
    const int nc = (n - 1) / 2 + 1;
    // restriction columns: 30 x 4 coarse nodes per chunk of coarse planes
    {
        const int mc = nc - 2, cols = ((mc + 29) / 30) * ((mc + 3) / 4);
        t.restr = {16, std::max(2, mc * cols / 2048)};
    }
    t.norm = {by, heuristic_zchunk(3, n, by, 1, target)};
    return t;
}

// Two sweeps in one launch: long chunks, since a chunk costs eight planes more
// than it owns (257^3 FP64, with the norm: 165 / 140 / 123 / 110 us with 8 / 16 / 32
// / 64 planes), but enough of them where grids of a batch make up the chip's load.
static void default_pairs(Tiles& t, int n, bool zg) {
    t.pair = t.pair_pro = t.pair_nrm = {32, n <= 129 ? 32 : 64, 1, 8};
    if (zg) t.pair_zg = t.pair;
}

Tiles default_tiles(int dim, int elem_bytes, int n, int smoother, int op) {
    if (op == OP_CC) {  // edges down to one cell
        Tiles t;
        if (dim == 2) t.smooth = {n <= 512 ? 8 : 16, 1};
        else t.smooth = {8, std::min(32, std::max(2, n / 16)), 1, 1};
        t.smooth_zg = t.smooth_pro = t.smooth_nrm = t.smooth;
        if (dim == 3 && smoother == SM_RBGS) default_pairs(t, n, true);
        return t;
    }
    Tiles t = lds_tiles(dim, n, smoother);
    t.restr.by = restrict_rows(dim, elem_bytes, op == OP_VAR, t.restr.by);
    if (dim == 3 && smoother == SM_RBGS && op != OP_VAR) {
        // One wavefront per 64 x 8 tile, nodes held by colour: measured against
        // the LDS tiles above, 33^3 4.5 / 6.5 us, 65^3 4.9 / 6.5 us, 129^3 9.0 /
        // 17.2 us, 257^3 36.5 / 52.2 us (FP32 plain sweep; with the correction
        // 11.5 / 25.6 us at 129^3; FP64 14.3 / 20.5 and 18.4 / 35.2 us there).
        // Chunks: enough wavefronts on small grids, then few re-read planes
        // (129^3 FP32: 10.7 / 9.0 / 9.3 / 11.5 us with 2 / 4 / 8 / 16 planes).
        const int zc = std::min(32, std::max(2, n / (elem_bytes == 8 ? 16 : 32)));
        t.smooth = t.smooth_zg = t.smooth_pro = {8, zc, 1, 1};
        // The two sweeps from zero in one launch: 33^3 5.5 us against 3.9 + 4.5,
        // 65^3 7.2 / 8.7, 129^3 13.4 / 15.9 us.
        if (elem_bytes <= 4 && op == OP_LAP) t.smooth_zg2 = {12, zc};
        default_pairs(t, n, t.smooth_zg2.zchunk == 0);
    }
    return t;
}

// One wavefront per column, six owned rows (four with coefficients); chunks as
// short as leave enough wavefronts.  Seven grids of 129^3: 100 us (105 with 32
// planes a chunk, LDS tiles 127); six of 65^3: 20 us (25); seven of 33^3: 7.7 us
// (8.1); 257^3 with coefficients 163 us (181).
TileCfg ir3d_tiles(int n, bool var) {
    return {var ? 6 : 8, std::max(2, std::min(32, n / 16)), 1, 1};
}

template <typename T>
hipError_t launch_smooth(int dim, int sm, int op, const GridDesc* d, int ninst, int n, int sel, int flags,
                         TileCfg cfg, hipStream_t s) {
    if (op == OP_CC) {
        if constexpr (sizeof(T) == 8) return cc_launch_smooth(dim, sm, d, ninst, n, sel, flags, cfg, s);
        return hipErrorInvalidValue;
    }
    if (n < 5 || ninst <= 0) return hipErrorInvalidValue;
    if ((flags & SWEEP_NORM) && ninst != 1) return hipErrorInvalidValue;  // one partial row
    const dim3 grid(smooth_tiles(dim, sm, n, cfg), ninst);
    const hipError_t e = dim == 2 ? launch_smooth2d<T>(sm, op, d, sel, flags, cfg, grid, s)
                                  : launch_smooth3d<T>(sm, op, d, sel, flags, cfg, grid, s);
    if (e != hipSuccess) return e;
    return hipGetLastError();
}
template hipError_t launch_smooth<double>(int, int, int, const GridDesc*, int, int, int, int, TileCfg, hipStream_t);
template hipError_t launch_smooth<float>(int, int, int, const GridDesc*, int, int, int, int, TileCfg, hipStream_t);
template hipError_t launch_smooth<half_t>(int, int, int, const GridDesc*, int, int, int, int, TileCfg, hipStream_t);

namespace {

// Launch + optional event bracket (finest-level smoothing measurement).
struct Prof {
    hipEvent_t* ev;
    int* n;
    int cap;
    hipStream_t s;
    bool on() const { return ev && n && *n + 2 <= cap; }
    void begin() {
        if (on()) (void)hipEventRecord(ev[*n], s);
    }
    void end() {
        if (on()) {
            (void)hipEventRecord(ev[*n + 1], s);
            *n += 2;
        }
    }
};

}  // namespace

#define MG_TRY(x)                          \
    do {                                   \
        hipError_t e_ = (x);               \
        if (e_ != hipSuccess) return e_;   \
    } while (0)

int tail_first_level(int dim, int elem, int op, const std::vector<int>& n, bool zero_top) {
    if (std::getenv("MG_NO_TAIL")) return -1;
    if (n.empty() || n.back() != (op == OP_CC ? 1 : 3)) return -1;  // the tail ends in the exact coarsest solve
    const int tmax = tail_max_edge(dim, elem, op);
    // (not for the coarsest level alone, whose own launch is shorter: stencil V-cycle
    // at 5^3 28.7 us a call, with a tail for the 3-node grid 31.3)
    for (int l = zero_top ? 0 : 1; l + 1 < (int)n.size(); ++l)
        if (n[(size_t)l] <= tmax && (int)n.size() - l <= kMaxTailLevels) return l;
    return -1;
}

// Coarsest level: exact solve of the single unknown (n = 3) or conjugate
// gradients (n > 3), from a zero iterate.
template <typename T>
hipError_t coarse_solve(const Problem& P, const Group& g, hipStream_t s) {
    if (P.cc) return launch_zero_u<T>(P.dim, g.d, g.ninst, g.n, s);  // one cell: zero correction
    if (g.n == 3) return launch_coarsest<T>(P.dim, P.op(), g.d, g.ninst, s);
    return launch_cg<T>(P.dim, P.var, g.d, g.ninst, g.n, P.cg_iters > 0 ? P.cg_iters : 4 * (g.n - 1), s);
}

// The fused last pre-smoothing sweep + restriction applies to 3D Laplacian
// red-black levels in FP32 or binary16 storage whose tiles chose it.
template <typename T>
bool fused_restrict_ok(const Problem& P, int dim, const Tiles& t) {
    return sizeof(T) <= 4 && dim == 3 && P.op() == OP_LAP && P.smoother == SM_RBGS && t.fused.zchunk > 0 &&
           std::getenv("MG_NO_FUSED_RESTRICT") == nullptr;
}

// The first two pre-smoothing sweeps from a zero iterate in one launch:
// Laplacian red-black levels in FP32 or binary16 storage whose tiles chose it.
template <typename T>
bool smooth2_ok(const Problem& P, int dim, const Tiles& t, bool zero) {
    return zero && sizeof(T) <= 4 && (dim == 2 || dim == 3) && P.op() == OP_LAP && P.smoother == SM_RBGS && P.nu1 >= 2 &&
           t.smooth_zg2.zchunk > 0 && std::getenv("MG_NO_FUSED_SMOOTH2") == nullptr;
}
// 'sel' names the output buffer (1: u, 0: t; the input is the zero iterate).
template <typename T>
hipError_t launch_smooth2(int dim, const Group& g, const Tiles& t, int sel, hipStream_t s) {
    return dim == 2 ? launch_smooth2d_zg2<T>(g.d, g.ninst, g.n, sel, t.smooth_zg2, s)
                    : launch_smooth3d_zg2<T>(g.d, g.ninst, g.n, sel, t.smooth_zg2, s);
}
// The first two post-smoothing sweeps (correction fused into the first) in one
// launch: 2D Laplacian red-black levels in FP32 or binary16 storage whose
// tiles chose it.
template <typename T>
bool post2_ok(const Problem& P, int dim, const Tiles& t) {
    return sizeof(T) <= 4 && dim == 2 && P.op() == OP_LAP && P.smoother == SM_RBGS && P.nu2 >= 2 &&
           t.smooth_pro2.zchunk > 0 && std::getenv("MG_NO_FUSED_POST2") == nullptr;
}

int leg_max_edge() {
    const char* e = std::getenv("MG_LEG_MAX_EDGE");
    return e ? std::min(std::atoi(e), kLegMaxN) : kLegMaxN;
}

// Legs are taken wherever they run: per V(2,2) cycle and solve step they were
// faster than sweeps (or pairs of them) and restriction apart on every size, type
// and sweep count timed (us, apart -> legs).  FP64: 257^2 90 -> 50, 1025^2 161 ->
// 88, 4097^2 694 -> 370, 8193^2 2297 -> 1191, V(1,1) 4097^2 447 -> 357; FP32: 257^2
// 86 -> 46, 4097^2 457 -> 313, 8193^2 1385 -> 1028, V(3,3) 4097^2 656 -> 470;
// binary16: 4097^2 478 -> 290; coefficients FP64: 257^2 143 -> 60, 1025^2 265 ->
// 116, 2049^2 480 -> 211, 4097^2 1382 -> 621, V(1,1) 841 -> 576, V(3,3) 1916 ->
// 1135; coefficients FP32: 2049^2 406 -> 201, 4097^2 1063 -> 545.
bool leg_ok(const Problem& P, int n) {
    return P.dim == 2 && P.smoother == SM_RBGS && P.op() != OP_CC && P.nu1 >= 1 && P.nu2 >= 1 && n >= 5 &&
           n <= P.leg_max;
}

bool leg_leaves(const Problem& P, int flags) {
    if (flags & SWEEP_PROLONG) return false;
    return P.nu1 > 2 || (flags == 0 && P.nu2 > 2);
}

// Two sweeps in one launch where its boxes cover most of the chip: a box's march
// is long (about 1 us a plane when it has the compute unit to itself), and on
// fewer boxes one-wavefront tiles finish sooner.  129^3 FP32, one grid (72
// boxes): 38 us against 11.5 + 9; seven grids (504): 49 us against 52 + 48.
bool pair_ok(const Problem& P, const Tiles& t, int flags, int n, int ninst) {
    const TileCfg& c = t.pair_of(flags);
    return P.dim == 3 && P.smoother == SM_RBGS && P.op() != OP_VAR && c.zchunk > 0 &&
           (size_t)smooth3d_x2_tiles(P.op(), n, c) * (size_t)ninst >= kPairBoxes;
}

int first_sweeps(const Problem& P, const Tiles& t, int n) {
    if (P.nu1 < 2) return 1;
    if (leg_ok(P, n)) return P.nu1 == 2 ? 2 : 1;
    return pair_ok(P, t, SWEEP_NORM, n, 1) ? 2 : 1;
}

// Post-smoothing select bits: the symmetric red-black smoother relaxes black first.
inline int post_sel(const Problem& P, int cur) { return cur | (P.sym ? SEL_BLACK_FIRST : 0); }

// Launches of a level's ascending leg that change the iterate's buffer.
template <typename T>
int up_launches(const Problem& P, const Tiles& t, int n, int ninst) {
    if (P.nu2 == 0) return 0;
    int i = 0, k = 0;
    if (leg_ok(P, n) || post2_ok<T>(P, P.dim, t)) {
        i = P.nu2 >= 2 ? 2 : 1;
        k = 1;
    }
    for (; i < P.nu2; ++k) i += i + 1 < P.nu2 && pair_ok(P, t, i == 0 ? SWEEP_PROLONG : 0, n, ninst) ? 2 : 1;
    return k;
}

// The descending leg of a level: nu1 sweeps, the residual and its restriction,
// as few launches as the level's rules give.  top: level 0, whose plain sweeps
// are measured; first_done as in vcycle.  'cur' is the buffer of the iterate (0
// u, 1 t).
template <typename T>
hipError_t descend(const Problem& P, const Group& g, const Tiles& t, bool top, bool zero, bool first_done, int& cur,
                   hipStream_t s, Prof& prof) {
    cur = first_done ? 1 : 0;
    int i = first_done ? first_sweeps(P, t, g.n) : 0;
    const bool leg = leg_ok(P, g.n);
    const int ns = P.nu1 >= 2 ? 2 : 1;
    if (leg && first_done && i == P.nu1) return hipSuccess;
    const int last = leg ? P.nu1 - ns : P.nu1;  // the leg's launch takes the others
    if (!leg && i == 0 && smooth2_ok<T>(P, P.dim, t, zero)) {
        // sweeps 1 and 2 from the zero iterate, into the buffer that an even
        // number of launches brings to u
        int k = up_launches<T>(P, t, g.n, g.ninst);
        for (int j = 2; j < P.nu1; j += pair_ok(P, t, 0, g.n, g.ninst) && j + 1 < P.nu1 ? 2 : 1) ++k;
        cur = k & 1;
        MG_TRY(launch_smooth2<T>(P.dim, g, t, cur ^ 1, s));
        i = 2;
    }
    bool fused = false;
    while (i < last) {
        const int flags = (i == 0 && zero) ? SWEEP_ZERO_GUESS : 0;
        if (i + 1 < last && pair_ok(P, t, flags, g.n, g.ninst)) {
            MG_TRY(launch_smooth3d_x2<T>(P.op(), g.d, g.ninst, g.n, cur, flags, t.pair_of(flags), s));
            i += 2;
        } else if (!leg && i == P.nu1 - 1 && flags == 0 && fused_restrict_ok<T>(P, P.dim, t)) {
            // the last sweep carries the residual and restriction
            MG_TRY(launch_smooth_restrict3d<T>(g.d, g.ninst, g.n, cur, t.fused, s));
            fused = true;
            ++i;
        } else {
            const bool timed = top && flags == 0;  // plain finest-level sweeps only
            if (timed) prof.begin();
            MG_TRY(launch_smooth<T>(P.dim, P.smoother, P.op(), g.d, g.ninst, g.n, cur, flags, t.sweep(flags), s));
            if (timed) prof.end();
            ++i;
        }
        cur ^= 1;
    }
    if (leg) {
        MG_TRY(launch_down2d<T>(P.op(), g.d, g.ninst, g.n, cur, ns, (i == 0 && zero) ? SWEEP_ZERO_GUESS : 0, s));
        cur ^= 1;
        return hipSuccess;
    }
    if (P.nu1 == 0 && zero) MG_TRY(launch_zero_u<T>(P.dim, g.d, g.ninst, g.n, s));
    if (!fused) MG_TRY(launch_restrict<T>(P.dim, P.op(), g.d, g.ninst, g.n, cur, t.restr, s));
    return hipSuccess;
}

// The ascending leg of a level: the correction and nu2 sweeps; the iterate
// ends in u.
template <typename T>
hipError_t ascend(const Problem& P, const Group& g, const Tiles& t, bool top, int cur, hipStream_t s, Prof& prof) {
    int i = 0;
    if (P.nu2 == 0) {
        MG_TRY(launch_prolong<T>(P.dim, P.op(), g.d, g.ninst, g.n, cur, s));
    } else if (leg_ok(P, g.n)) {
        i = P.nu2 >= 2 ? 2 : 1;
        MG_TRY(launch_up2d<T>(P.op(), g.d, g.ninst, g.n, post_sel(P, cur), i, s));
        cur ^= 1;
    } else if (post2_ok<T>(P, P.dim, t) && (cur == 1 || (up_launches<T>(P, t, g.n, g.ninst) & 1) == cur)) {
        // (from u only where the sweeps after it bring the iterate back there)
        MG_TRY(launch_smooth2d_pro2<T>(g.d, g.ninst, g.n, post_sel(P, cur), t.smooth_pro2, s));
        cur ^= 1;
        i = 2;
    }
    while (i < P.nu2) {
        const int flags = i == 0 ? SWEEP_PROLONG : 0;  // the first sweep adds P uc while loading
        if (i + 1 < P.nu2 && pair_ok(P, t, flags, g.n, g.ninst)) {
            MG_TRY(launch_smooth3d_x2<T>(P.op(), g.d, g.ninst, g.n, post_sel(P, cur), flags, t.pair_of(flags), s));
            i += 2;
        } else {
            const bool timed = top && flags == 0;
            if (timed) prof.begin();
            MG_TRY(launch_smooth<T>(P.dim, P.smoother, P.op(), g.d, g.ninst, g.n, post_sel(P, cur), flags,
                                    t.sweep(flags), s));
            if (timed) prof.end();
            ++i;
        }
        cur ^= 1;
    }
    if (cur == 1) MG_TRY(launch_copy_t_to_u<T>(P.dim, g.d, g.ninst, g.n, s));
    return hipSuccess;
}

// Algorithm 1 on level l with gamma recursive calls: kind 0 V (one call), 1 W
// (two), 2 F (an F-cycle then a V-cycle).  The zero guess precedes the first
// call only; later calls continue from the coarse iterate the previous call
// left.  Level by level down to the tail's finest level, whose whole recursion
// is one launch.
template <typename T>
hipError_t cycle_rec(const Problem& P, const std::vector<Group>& G, int l, int kind, bool zero,
                     const std::vector<Tiles>& tiles, hipStream_t s, Prof& prof, const TailPlan* tail,
                     bool first_done = false) {
    const int L = (int)G.size();
    const int dim = P.dim;
    const Group& g = G[(size_t)l];
    if (tail && l == tail->first && !first_done)
        return launch_tail<T>(dim, P.smoother, P.op(), tail->d, tail->ninst, P.nu1, P.nu2, P.sym ? 1 : 0, kind, zero,
                              s);
    if (l == L - 1) return coarse_solve<T>(P, g, s);
    int cur;
    MG_TRY(descend<T>(P, g, tiles[(size_t)l], l == 0, zero, first_done, cur, s, prof));
    if (kind == 0) {
        MG_TRY(cycle_rec<T>(P, G, l + 1, 0, true, tiles, s, prof, tail));
    } else if (kind == 1) {
        MG_TRY(cycle_rec<T>(P, G, l + 1, 1, true, tiles, s, prof, tail));
        MG_TRY(cycle_rec<T>(P, G, l + 1, 1, false, tiles, s, prof, tail));
    } else {
        MG_TRY(cycle_rec<T>(P, G, l + 1, 2, true, tiles, s, prof, tail));
        MG_TRY(cycle_rec<T>(P, G, l + 1, 0, false, tiles, s, prof, tail));
    }
    return ascend<T>(P, g, tiles[(size_t)l], l == 0, cur, s, prof);
}

template <typename T>
hipError_t vcycle(const Problem& P, const std::vector<Group>& G, bool zero_top, const std::vector<Tiles>& tiles,
                  hipStream_t s, hipEvent_t* prof_ev, int* prof_n, int prof_cap, const TailPlan* tail,
                  bool first_done) {
    const int L = (int)G.size();
    const int dim = P.dim;
    Prof prof{prof_ev, prof_n, prof_cap, s};
    // a first sweep that already ran needs a level-0 pre-smoothing sweep to have been
    if (first_done && (L < 2 || P.nu1 < 1 || zero_top)) return hipErrorInvalidValue;
    const bool use_tail = tail && tail->first >= 0 && tail->first < L && tail->d;
    if (P.cycle != 0)
        return cycle_rec<T>(P, G, 0, P.cycle, zero_top, tiles, s, prof, use_tail ? tail : nullptr, first_done);
    // levels [0, stop) run level by level; the rest is the tail (or the coarsest solve)
    const int stop = use_tail ? tail->first : L - 1;
    if (first_done && stop == 0) return hipErrorInvalidValue;
    if (stop == 0 && !use_tail) return coarse_solve<T>(P, G[0], s);
    std::vector<int> sel((size_t)L, 0);
    // descending leg: presmoothing, residual, restriction (Algorithm 1)
    for (int l = 0; l < stop; ++l)
        MG_TRY(descend<T>(P, G[(size_t)l], tiles[(size_t)l], l == 0, l == 0 ? zero_top : true, l == 0 && first_done,
                          sel[(size_t)l], s, prof));
    if (use_tail) {
        // every level from 'stop' to the coarsest in one launch, from a zero guess
        MG_TRY(launch_tail<T>(dim, P.smoother, P.op(), tail->d, tail->ninst, P.nu1, P.nu2, P.sym ? 1 : 0, 0, true,
                              s));
    } else {
        // coarsest grid from the zero guess
        MG_TRY(coarse_solve<T>(P, G[(size_t)L - 1], s));
    }
    // ascending leg: interpolation + correction, postsmoothing
    for (int l = stop - 1; l >= 0; --l)
        MG_TRY(ascend<T>(P, G[(size_t)l], tiles[(size_t)l], l == 0, sel[(size_t)l], s, prof));
    return hipSuccess;
}

template hipError_t vcycle<double>(const Problem&, const std::vector<Group>&, bool, const std::vector<Tiles>&,
                                   hipStream_t, hipEvent_t*, int*, int, const TailPlan*, bool);
template hipError_t vcycle<float>(const Problem&, const std::vector<Group>&, bool, const std::vector<Tiles>&,
                                  hipStream_t, hipEvent_t*, int*, int, const TailPlan*, bool);
template hipError_t vcycle<half_t>(const Problem&, const std::vector<Group>&, bool, const std::vector<Tiles>&,
                                   hipStream_t, hipEvent_t*, int*, int, const TailPlan*, bool);

}  // namespace mg
