// Pair loops: density + Newton-Raphson h solve, hydro forces, neighbour
// export, MFV geometry.
//
// Work decomposition (the GPU analogue of the paper's per-leaf-cell neighbour
// gathering, section 4.2, with a leaf as the unit of work as in its OpenMP
// loop, section 5.2.1): one wavefront per home leaf of at most G sorted
// particles, 64/G lanes per particle.  The wave walks the box tree to collect
// the leaves that can hold neighbours of its particles into an LDS list.
// Candidate leaves are then handled 128/G at a time (128 candidate slots):
//   stage  -- one coalesced load per field brings their positions into LDS;
//   test   -- each (home particle, staged leaf) combination is first judged
//             by the distance from the particle to the leaf's box; the
//             passing ones are dealt out over the 64 lanes, which test their
//             candidates and set hit bits in a per-particle 128-bit mask
//             (no pair arithmetic yet);
//   flush  -- each particle's lanes evaluate the pair terms of its hits.
// The test is cheap and runs for every candidate of a passing combination;
// the expensive pair terms run only for hits, with the lanes compacted (a
// wave-wide branch on "any lane hit" would otherwise execute them for almost
// every candidate).  Each output is accumulated by its own lanes in a fixed
// order, so results are deterministic and need no atomics.
//
// This header holds the kernels, templated on the smoothing kernel; it is
// compiled by pairs_m4.hip and pairs_quintic.hip only.
#pragma once

#include "pairs_args.hpp"

#include <algorithm>
#include <type_traits>

namespace sph {
namespace {

// Views of pointers the pair kernels only read.  Through the constant address
// space a load with a wave-uniform address becomes a scalar load into SGPRs
// (the argument blocks, the home leaf's node); through the global address
// space a per-lane load is a plain vector load instead of a flat access, whose
// completion LDS waits would otherwise also have to cover.
template <class T>
__device__ inline const __attribute__((address_space(4))) T *as_const(const T *p)
{
    return (const __attribute__((address_space(4))) T *)p;
}
template <class T>
__device__ inline const __attribute__((address_space(1))) T *as_global(const T *p)
{
    return (const __attribute__((address_space(1))) T *)p;
}
// A whole read-only record, word by word through one of those views.
template <class T>
__device__ inline T load_const(const T *p)
{
    static_assert(sizeof(T) % 4 == 0 && alignof(T) >= 4, "word-sized record");
    T v;
    const auto *src = as_const((const uint32_t *)p);
    uint32_t *dst = (uint32_t *)&v;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); k++) dst[k] = src[k];
    return v;
}
template <class T>
__device__ inline T load_global(const T *p)
{
    static_assert(sizeof(T) % 4 == 0 && alignof(T) >= 4, "word-sized record");
    T v;
    const auto *src = as_global((const uint32_t *)p);
    uint32_t *dst = (uint32_t *)&v;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); k++) dst[k] = src[k];
    return v;
}

// The same pointer, but the compiler cannot tell: what is loaded through it
// again is loaded again (a scalar load) instead of staying in scalar registers
// from the first load on, which spilled them by the hundred.
template <class T>
__device__ inline T *reload(T *p)
{
    asm volatile("" : "+s"(p));
    return p;
}

__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Cross-lane moves inside a 16-lane DPP row, for butterfly reductions: the
// value of lane l ^ O for O = 1, 2 (quad permutes); for O = 4 and 8 the value
// of the mirrored lane of l's 8- or 16-lane group, which is lane l ^ O's value
// wherever the value is already uniform over groups of O lanes -- as it is at
// that step of a butterfly.  No LDS and no lane-address registers.
template <int O>
__device__ inline int xlane(int v)
{
    static_assert(O == 1 || O == 2 || O == 4 || O == 8, "within one DPP row");
    constexpr int ctrl = O == 1 ? 0xB1 : O == 2 ? 0x4E : O == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(v, v, ctrl, 0xF, 0xF, false);
}
template <int O>
__device__ inline double xlane(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)xlane<O>((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)xlane<O>((int)(uint32_t)(b >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over each group of K consecutive lanes (K = 1, 2, 4, 8, 16), the same
// bits on every lane of the group (IEEE addition is commutative).
template <int K, class T>
__device__ inline T group_sum(T v)
{
    if constexpr (K >= 2) v += xlane<1>(v);
    if constexpr (K >= 4) v += xlane<2>(v);
    if constexpr (K >= 8) v += xlane<4>(v);
    if constexpr (K >= 16) v += xlane<8>(v);
    return v;
}
template <int K>
__device__ inline double group_max(double v)
{
    if constexpr (K >= 2) v = fmax(v, xlane<1>(v));
    if constexpr (K >= 4) v = fmax(v, xlane<2>(v));
    if constexpr (K >= 8) v = fmax(v, xlane<4>(v));
    if constexpr (K >= 16) v = fmax(v, xlane<8>(v));
    return v;
}

// Wave-wide maxima: each 16-lane row by DPP, then the four rows' values read
// into scalar registers (wave-uniform result).
__device__ inline double wave_max(double v)
{
    v = group_max<16>(v);
    auto row = [&](int l) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
        const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    };
    return fmax(fmax(row(0), row(16)), fmax(row(32), row(48)));
}

template <int K>
__device__ inline int group_max_int(int v)
{
    if constexpr (K >= 2) { const int w = xlane<1>(v); v = w > v ? w : v; }
    if constexpr (K >= 4) { const int w = xlane<2>(v); v = w > v ? w : v; }
    if constexpr (K >= 8) { const int w = xlane<4>(v); v = w > v ? w : v; }
    if constexpr (K >= 16) { const int w = xlane<8>(v); v = w > v ? w : v; }
    return v;
}

// Wave-wide sum of small non-negative per-lane counts, wave-uniform.
__device__ inline int64_t wave_sum_int(int v)
{
    v = group_sum<16>(v);
    return (int64_t)__builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
           (int64_t)__builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}

// Wave-wide sum in a fixed order, wave-uniform.
__device__ inline double wave_sum(double v)
{
    v = group_sum<16>(v);
    auto row = [&](int l) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
        const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
        return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
    };
    return (row(0) + row(16)) + (row(32) + row(48));
}

__device__ inline int wave_max_int(int v)
{
    int w = xlane<1>(v);
    v = w > v ? w : v;
    w = xlane<2>(v);
    v = w > v ? w : v;
    w = xlane<4>(v);
    v = w > v ? w : v;
    w = xlane<8>(v);
    v = w > v ? w : v;
    const int a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const int c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    const int ab = a > b ? a : b, cd = c > d ? c : d;
    return ab > cd ? ab : cd;
}

// Persistent work loop over the leaves.  Blocks are dispatched round-robin
// over the 8 XCDs, so block b runs on XCD b % 8; each XCD first claims leaves
// from its own contiguous eighth of the leaf range (neighbouring leaves then
// share that XCD's L2), then helps the others.  Claims go through one atomic
// counter per eighth, `claim` consecutive leaves at a time; every leaf is
// processed by exactly one wave, so results do not depend on which wave took
// it.  Atomics on one address serialise (~0.1 us each), so claims are kept
// few: a block's first claim in its own eighth is static (its rank among the
// eighth's blocks; the counter hands out the claims after those), and after
// draining its own eighth a block helps the following eighths in turn and
// stops at the first one it finds exhausted.  Every eighth is still drained
// by its own blocks; a block makes no atomic at start and one failing claim
// on another counter at the end, instead of one on each of them (for a small
// set that finishes early, those tail claims were a large part of the
// launch).
template <class Fn>
__device__ inline void for_each_home_leaf(int64_t L, uint32_t *__restrict__ work, int claim,
                                          Fn fn)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t per = (L + kXcds - 1) / kXcds;
    const int x0 = (int)(blockIdx.x % kXcds);
    const uint32_t rank = blockIdx.x / kXcds;          // among the blocks of eighth x0
    const uint32_t nstatic = gridDim.x / kXcds;        // static first claims per eighth
    for (int r = 0; r < kXcds; r++) {
        const int x = (x0 + r) % kXcds;
        const int64_t beg = x * per;
        const int64_t end = beg + per < L ? beg + per : L;
        if (beg >= end) continue;
        bool got = false;
        for (int k = 0;; k++) {
            uint32_t c = rank;
            if (r > 0 || k > 0 || rank >= nstatic) {   // (a grid not a multiple of 8)
                if (lane == 0) c = nstatic + atomicAdd(&work[x], 1u);
                // wave-uniform from here on (scalar registers): the leaf's
                // argument block, node and particle range are then loaded once
                // per wave
                c = (uint32_t)__builtin_amdgcn_readlane((int)c, 0);
            }
            const int64_t leaf0 = beg + (int64_t)c * claim;
            if (leaf0 >= end) break;
            got = true;
            const int64_t leaf1 = leaf0 + claim < end ? leaf0 + claim : end;
            for (int64_t leaf = leaf0; leaf < leaf1; leaf++) fn(leaf);
        }
        if (r > 0 && !got) break;   // a helped eighth was already exhausted
    }
}

// Status of a wave's particles: when any lane raises `cond`, set `flag` in
// status[0] and add the number of such lanes to status[word], one atomic
// each per wave (a set whose particles all fail then costs one atomic per
// leaf, not one per particle).  Called by every lane of the wave.
__device__ inline void report(int32_t *status, bool cond, int32_t flag, int word)
{
    const int cnt = (int)__popcll(__ballot(cond));
    if (cnt && (threadIdx.x & (kWave - 1)) == 0) {
        atomicOr(&status[0], flag);
        atomicAdd(&status[word], cnt);
    }
}

// Copy the device tree description into LDS once per block.
__device__ inline void load_tree(const TreeInfo *__restrict__ src, TreeInfo &dst)
{
    const auto *s = as_global((const int64_t *)src);
    int64_t *d = (int64_t *)&dst;
    for (int k = threadIdx.x; k < kTreeWords; k += blockDim.x) d[k] = s[k];
    __syncthreads();
}

// Squared gap between two nodes' boxes (0 if they overlap), with the periodic
// images when the box is periodic: along an axis the nearest image of two
// intervals is that of their centres.
__device__ inline double box_gap2(const Node &a, const Node &b, const Box &bx)
{
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        double d = fabs(a.c[k] - b.c[k]);
        if (bx.periodic) d = fmin(d, fabs(bx.len[k] - d));
        const double g = fmax(d - (a.e[k] + b.e[k]), 0.0);
        s += g * g;
    }
    return s;
}

// r_ij^2 exactly as (dx*dx + dy*dy) + dz*dz, each operation rounded on its
// own, so neighbour predicates agree bit for bit with any other evaluation
// written the same way.
__device__ inline double exact_r2(double dx, double dy, double dz)
{
#pragma clang fp contract(off)
    double a = dx * dx;
    double b = dy * dy;
    double c = dz * dz;
    return (a + b) + c;
}

// a*b + c*d with both products rounded before the sum and no fused
// multiply-add, so swapping (a, b) with (c, d) gives the same bits: keeps the
// pair force of (i, j) the exact negative of that of (j, i).
template <class T>
__device__ inline T sym_dot2(T a, T b, T c, T d)
{
#pragma clang fp contract(off)
    T p = a * b;
    T q = c * d;
    return p + q;
}

// Kernel gradients of a pair and their sum, each product rounded before the
// sum: keeps 0.5 (G_i + G_j) identical for (i, j) and (j, i).
template <class T>
__device__ inline void sym_grads(T gfi, T dfi, T gfj, T dfj, T &gi, T &gj, T &gsum)
{
#pragma clang fp contract(off)
    gi = gfi * dfi;
    gj = gfj * dfj;
    gsum = gi + gj;
}

__device__ inline double min_image(double d, double L, double half)
{
    if (d > half) d -= L;
    else if (d < -half) d += L;
    return d;
}

__device__ inline float min_image_f(float d, float L, float half)
{
    if (d > half) d -= L;
    else if (d < -half) d += L;
    return d;
}

// 1/sqrt(x) for x > 0: the hardware estimate refined by two Newton-Raphson
// steps on 1/y^2 - x (each squares the relative error), to about 1 ulp in
// eight operations instead of a correctly rounded square root and division.
__device__ inline double rsqrt_nr(double x)
{
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const double r = fma(-x * y, y, 1.0);
        y = fma(0.5 * y, r, y);
    }
    return y;
}

// 1/sqrt(x) for x > 0 with one Newton-Raphson step on the hardware estimate:
// the estimate's relative error is squared once, to well below 1e-13 -- the
// density sums need q = r/h to far better than their 1e-10 parity bound, not
// to the last bit.
__device__ inline double rsqrt_nr1(double x)
{
    double y = __builtin_amdgcn_rsq(x);
    const double r = fma(-x * y, y, 1.0);
    return fma(0.5 * y, r, y);
}

// 1/x for x > 0: the hardware estimate refined by two Newton-Raphson steps
// on 1/y - x, to about 1 ulp.
__device__ inline double rcp_nr(double x)
{
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int k = 0; k < 2; k++) {
        const double e = fma(-x, y, 1.0);
        y = fma(y, e, y);
    }
    return y;
}

// Kernel shapes f(q) and f'(q), branch-free in B-spline form:
// M4: f = a^3/4 - b^3, f' = 3 b^2 - 3/4 a^2 with a = (2-q)_+, b = (1-q)_+;
// quintic: f = a^5 - 6 b^5 + 15 c^5, f' = -5 a^4 + 30 b^4 - 75 c^4 with
// a = (3-q)_+, b = (2-q)_+, c = (1-q)_+.
template <int K, class T>
__device__ inline void kern(T qq, T &f, T &df)
{
    if constexpr (K == SPH_KERNEL_QUINTIC) {
        const T a = fmax(T(3) - qq, T(0));
        const T b = fmax(T(2) - qq, T(0));
        const T c = fmax(T(1) - qq, T(0));
        const T a2 = a * a, b2 = b * b, c2 = c * c;
        const T a4 = a2 * a2, b4 = b2 * b2, c4 = c2 * c2;
        f = a4 * a - T(6) * (b4 * b) + T(15) * (c4 * c);
        df = T(30) * b4 - T(5) * a4 - T(75) * c4;
    } else {
        const T a = fmax(T(2) - qq, T(0));
        const T b = fmax(T(1) - qq, T(0));
        const T a2 = a * a, b2 = b * b;
        f = T(0.25) * a2 * a - b2 * b;
        df = T(3) * b2 - T(0.75) * a2;
    }
}

// ---------------------------------------------------------------------------
// Tree walk
// ---------------------------------------------------------------------------
// The walk's result stays in `list`; the second frontier buffer a walk needs
// is lent by the caller (the pair loops lend their staging slots, which hold
// nothing while a walk runs).
struct WalkBuf {
    uint32_t list[kFront];
    uint32_t tmp[kWave];
};

// Breadth-first walk of the 8-ary tree, 64 child tests per step.  Result: n
// nodes of level `lev` in `list` that pass the test.  Normally lev = 0 (the
// candidate leaves).  If expanding a level would overflow the LDS frontier,
// the walk stops there and returns that level's nodes; the caller then tests
// the leaves under each of them directly (bounded extra work instead of a
// scan of every leaf).
struct WalkResult {
    int n;
    int lev;
    const uint32_t *list;
};

// Leaves the walk's result in wb.list, copying it there from the spare
// buffer when the last expansion wrote it there.
__device__ inline WalkResult walk_result(WalkBuf &wb, const uint32_t *cur, int n, int lev)
{
    if (cur != wb.list) {
        const int lane = threadIdx.x & (kWave - 1);
        for (int t = lane; t < n; t += kWave) wb.list[t] = cur[t];
        wave_lds_sync();
    }
    return WalkResult{n, lev, wb.list};
}

// spare: kFront entries of LDS the walk may overwrite
template <class Test>
__device__ WalkResult walk(const TreeInfo &T, const Node *nodes, Test test, WalkBuf &wb,
                           uint32_t *spare)
{
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lt = __lanemask_lt();
    uint32_t *cur = wb.list, *nxt = spare;
    const int top = T.nlev - 1;
    if (lane == 0) cur[0] = 0;
    wave_lds_sync();
    if (top == 0) {
        bool pass = lane == 0 && test(nodes[0]);
        return WalkResult{__ballot(pass) ? 1 : 0, 0, cur};
    }
    int ncur = 1;
    for (int lev = top; lev > 0; lev--) {
        const Node *cl = nodes + T.off[lev - 1];
        const int64_t nchild = T.cnt[lev - 1];
        const int total = ncur * 8;
        int nout = 0;
        for (int b = 0; b < total; b += kWave) {
            int t = b + lane;
            bool valid = t < total;
            int64_t node = valid ? (int64_t)cur[t >> 3] * 8 + (t & 7) : 0;
            valid = valid && node < nchild;
            bool pass = valid && test(load_global(cl + node));
            uint64_t mask = __ballot(pass);
            int pos = nout + (int)__popcll(mask & lt);
            if (pass && pos < kFront) nxt[pos] = (uint32_t)node;
            nout += (int)__popcll(mask);
        }
        wave_lds_sync();
        if (nout > kFront) return walk_result(wb, cur, ncur, lev);
        uint32_t *tmp = cur;
        cur = nxt;
        nxt = tmp;
        ncur = nout;
        if (ncur == 0) break;
    }
    return walk_result(wb, cur, ncur, 0);
}

// Visit the candidate leaves in groups of at most `depth` (<= NL, the LDS
// tile): fn(leaves, count) with a wave-uniform count.  After a truncated walk
// the leaves under each returned node are tested 64 at a time and the
// passing ones grouped.
template <int NL, class Test, class Fn>
__device__ int64_t for_each_leaf_group(const TreeInfo &T, const Node *nodes, const WalkResult &wr,
                                       Test test, WalkBuf &wb, Fn fn, int depth = NL)
{
    const int D = depth >= 1 && depth <= NL ? depth : NL;
    if (wr.lev == 0) {
        for (int t0 = 0; t0 < wr.n; t0 += D) fn(wr.list + t0, wr.n - t0 < D ? wr.n - t0 : D);
        return wr.n;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const uint64_t lt = __lanemask_lt();
    const int64_t L = T.cnt[0];
    int64_t span = 1;
    for (int l = 0; l < wr.lev; l++) span *= 8;
    int64_t tested = 0;
    for (int k = 0; k < wr.n; k++) {
        const int64_t b0 = (int64_t)wr.list[k] * span;
        const int64_t b1 = b0 + span < L ? b0 + span : L;
        for (int64_t b = b0; b < b1; b += kWave) {
            const int64_t c = b + lane;
            const bool pass = c < b1 && test(load_global(nodes + c));
            const uint64_t mask = __ballot(pass);
            if (pass) wb.tmp[__popcll(mask & lt)] = (uint32_t)c;
            wave_lds_sync();
            const int cnt = (int)__popcll(mask);
            for (int t0 = 0; t0 < cnt; t0 += D) fn(wb.tmp + t0, cnt - t0 < D ? cnt - t0 : D);
            wave_lds_sync();
            tested += b1 - b < kWave ? b1 - b : kWave;
        }
    }
    return tested;
}

// Per candidate leaf: the periodic shift that the minimum image gives every
// pair (i in home, j in the leaf) closer than `reach`, when that shift is
// unique (both boxes small against the period); otherwise the pair loop
// applies the minimum image pair by pair.
struct Shift {
    double s[3];
    bool per_pair;
};

__device__ inline Shift leaf_shift(const Node &home, const Node &cand, const Box &bx, double reach)
{
    Shift sh{{0.0, 0.0, 0.0}, false};
    if (!bx.periodic) return sh;
    for (int a = 0; a < 3; a++) {
        const double dc = home.c[a] - cand.c[a];
        sh.s[a] = dc > bx.half[a] ? -bx.len[a] : (dc < -bx.half[a] ? bx.len[a] : 0.0);
        const double span = reach + (home.e[a] + cand.e[a]);
        if (!(span < 0.49 * bx.len[a])) sh.per_pair = true;
    }
    return sh;
}

// ---------------------------------------------------------------------------
// Candidate groups and the tests shared by the pair loops
// ---------------------------------------------------------------------------
// A wave holds the G home particles of one leaf, LPP = 64 / G lanes each when
// it evaluates pair terms.  To find the pairs it turns round: a lane holds a
// candidate, the home particle is the same for all lanes.
//
// Candidate leaves come in groups of at most 64, one per lane, which set up a
// table in LDS (first particle, particle count, periodic shift) and measure,
// for every home particle, the distance to the leaf's box: a 64-bit ballot
// per home particle says which leaves of the group can hold neighbours of it.
// The candidates are then loaded into registers, kRows rows of 64 slots at a
// time (slot s = particle s % G of leaf s / G), and tested against each home
// particle in turn, skipping rows none of whose leaves passed.  A test is a
// handful of instructions for 64 candidates, its result a ballot in scalar
// registers, and the hits' ranks are bit counts of that ballot: no hit masks
// in LDS, no bit-by-bit walk over them, every lane at work.
//
// What bounds it: instruction issue.  Testing (particle, leaf) combinations
// dealt out over the lanes from LDS, with hit masks by LDS atomics and a flush
// that popped mask bits, spent about 16,600 vector instructions per home leaf
// on C1-like sets (2.1M particles, G = 16, 92 candidate leaves per home leaf).
constexpr int kGroup = kWave;       // candidate leaves per group
constexpr int kRows = 4;            // rows of 64 candidates held in registers

// How the separations of a group see the periodic box: no shift at all, one
// shift per leaf, or the minimum image pair by pair (boxes so small that a
// leaf's shift is ambiguous).  A pair closer than the reach has the same
// image under the last two.
enum : int { kImgNone = 0, kImgShift = 1, kImgPair = 2 };

// Home particles as the tests read them (one broadcast read each): position
// and the threshold on r^2 (< 0: takes no part); FP32-pair tests read the
// offsets from the leaf centre instead.
struct alignas(32) HomeRow { double x, y, z, thr; };
struct alignas(16) HomeRowF { float x, y, z, thr; };

template <int G, int PREC>
struct HomeTab {
    HomeRow d[G];
    HomeRowF f[PREC == SPH_FP32_PAIR ? G : 1];
};

// Per leaf of the group: first particle and particle count (jm), the shift
// added to x_i - x_j (FP64), or the distance of the leaf centres with the
// shift (FP32-pair).  lm: per home particle, the leaves near enough to hold a
// pair.
template <int G, int PREC>
struct LeafTab {
    using T = std::conditional_t<PREC == SPH_FP64, double, float>;
    uint2 jm[kGroup];
    T ox[kGroup], oy[kGroup], oz[kGroup];
    uint64_t lm[G];
};

// The relative slack of the box test: it must accept every combination whose
// candidates the record test can accept (rounding of the two differently
// formed distances; FP32-pair separations carry single-precision error).  The
// leaf's half extents grow by this part of the reach.
template <int PREC>
__device__ constexpr double box_slack() { return PREC == SPH_FP64 ? 1e-6 : 1e-4; }

// The next group of at most `depth` candidate leaves of a walk's result
// (0: none left): a slice of the list, or after a truncated walk the passing
// ones of the next 64 leaves under the listed nodes (written to wb.tmp).
template <class Test>
__device__ inline int next_group(const TreeInfo &T, const Node *nodes, const WalkResult &wr,
                                 Test test, WalkBuf &wb, int depth, int64_t &pos,
                                 const uint32_t *&leaves)
{
    if (wr.lev == 0) {
        const int left = wr.n - (int)pos;
        if (left <= 0) return 0;
        leaves = wr.list + pos;
        const int n = left < depth ? left : depth;
        pos += n;
        return n;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int sh = 3 * wr.lev;
    const int64_t L = T.cnt[0], total = (int64_t)wr.n << sh;
    while (pos < total) {
        const int64_t t = pos + lane;
        const int64_t c = t < total ? ((int64_t)wr.list[t >> sh] << sh) + (t & ((1ll << sh) - 1)) : L;
        const bool pass = c < L && test(load_global(nodes + c));
        const uint64_t mask = __ballot(pass);
        pos += kWave;
        if (mask) {
            wave_lds_sync();   // the last group's readers of wb.tmp
            if (pass) wb.tmp[__popcll(mask & __lanemask_lt())] = (uint32_t)c;
            wave_lds_sync();
            leaves = wb.tmp;
            return (int)__popcll(mask);
        }
    }
    return 0;
}

// Leaves per group of a list of n: groups of equal size (whole rows), at most
// `most`.
template <int G>
__device__ inline int group_depth(int n, int most)
{
    constexpr int LPR = kWave / G;
    const int groups = (n + most - 1) / most;
    const int d = groups > 0 ? (n + groups - 1) / groups : most;
    const int r = (d + LPR - 1) / LPR * LPR;
    return r < most ? r : most;
}

// Set up a group (lane l: leaf leaves[l]): the table, and in `lmask` (lane p
// for home particle p) the leaves whose box is near enough to home particle p
// to hold a pair.  hcov < 0: symmetric force criterion (reach R max(h) over
// both leaves).  Returns how separations see the box.
template <int G, int PREC, int K>
__device__ inline int open_group(const uint32_t *leaves, int count, const uint32_t *__restrict__ lstart,
                                 const Node *__restrict__ nodes, const Node &home, const Box &bx,
                                 double hcov, const HomeTab<G, PREC> &H, uint64_t takes_part,
                                 LeafTab<G, PREC> &tab, uint64_t &lmask)
{
    constexpr double RK = Kern<K>::R;
    const int lane = threadIdx.x & (kWave - 1);
    // (a missing leaf is far away)
    double cx = 1e150, cy = 0.0, cz = 0.0, ex = 0.0, ey = 0.0, ez = 0.0, reach2 = -1.0;
    bool per_pair = false, shifted = false;
    uint2 jm{0u, 0u};
    if (lane < G) tab.lm[lane] = 0;
    if (lane < count) {
        const uint32_t c = leaves[lane];
        const uint32_t j0 = as_global(lstart)[c];
        jm.x = j0;
        jm.y = as_global(lstart)[c + 1] - j0;
        const Node cand = load_global(nodes + c);
        const double reach = RK * (hcov < 0.0 ? fmax(home.hmax, cand.hmax) : hcov);
        const Shift sh = leaf_shift(home, cand, bx, reach);
        per_pair = sh.per_pair;
        shifted = sh.s[0] != 0.0 || sh.s[1] != 0.0 || sh.s[2] != 0.0;
        // the box as the home particles see it; a leaf with pair-by-pair
        // images is near to all of them
        cx = cand.c[0] - sh.s[0];
        cy = cand.c[1] - sh.s[1];
        cz = cand.c[2] - sh.s[2];
        const double slack = per_pair ? INFINITY : box_slack<PREC>() * reach;
        ex = cand.e[0] + slack;
        ey = cand.e[1] + slack;
        ez = cand.e[2] + slack;
        if (hcov < 0.0) {
            const double hk = RK * cand.hmax;
            reach2 = hk * hk;
        }
        if constexpr (PREC == SPH_FP64) {
            tab.ox[lane] = sh.s[0];
            tab.oy[lane] = sh.s[1];
            tab.oz[lane] = sh.s[2];
        } else {
            tab.ox[lane] = (float)((home.c[0] - cand.c[0]) + (per_pair ? 0.0 : sh.s[0]));
            tab.oy[lane] = (float)((home.c[1] - cand.c[1]) + (per_pair ? 0.0 : sh.s[1]));
            tab.oz[lane] = (float)((home.c[2] - cand.c[2]) + (per_pair ? 0.0 : sh.s[2]));
        }
    }
    tab.jm[lane] = jm;
    const int img = __ballot(per_pair) ? kImgPair : (__ballot(shifted) ? kImgShift : kImgNone);
#pragma unroll
    for (int p = 0; p < G; p++) {
        if (!((takes_part >> p) & 1)) continue;
        const HomeRow h = H.d[p];
        const double dx = fmax(fabs(h.x - cx) - ex, 0.0);
        const double dy = fmax(fabs(h.y - cy) - ey, 0.0);
        const double dz = fmax(fabs(h.z - cz) - ez, 0.0);
        const double d2 = (dx * dx + dy * dy) + dz * dz;
        // (every lane stores the same value)
        tab.lm[p] = __ballot(d2 <= fmax(h.thr, reach2));
    }
    wave_lds_sync();
    lmask = tab.lm[lane < G ? lane : 0];
    if (lane >= G) lmask = 0;
    return img;
}

// One row of candidates in this lane's registers.
template <int PREC>
struct Cand {
    using T = std::conditional_t<PREC == SPH_FP64, double, float>;
    T x, y, z;      // position, or the offset from its leaf's centre
    T ox, oy, oz;   // shift (FP64, kImgShift) or leaf-centre distance (FP32-pair)
};

// x_i - x_j and r^2 of one home particle and one candidate: the expression
// every test and evaluation uses, so all see the same bits (r^2 in FP64 as
// exact_r2 forms it).
template <int PREC, int IMG, class T>
__device__ inline T separation(const Box &bx, T hx, T hy, T hz, T x, T y, T z, T ox, T oy, T oz,
                               T &dx, T &dy, T &dz)
{
    if constexpr (PREC == SPH_FP64) {
        dx = hx - x;
        dy = hy - y;
        dz = hz - z;
        if constexpr (IMG == kImgPair) {
            dx = min_image(dx, bx.len[0], bx.half[0]);
            dy = min_image(dy, bx.len[1], bx.half[1]);
            dz = min_image(dz, bx.len[2], bx.half[2]);
        } else if constexpr (IMG == kImgShift) {
            dx += ox;
            dy += oy;
            dz += oz;
        }
        return exact_r2(dx, dy, dz);
    } else {
        dx = (hx - x) + ox;
        dy = (hy - y) + oy;
        dz = (hz - z) + oz;
        if constexpr (IMG == kImgPair) {
            dx = min_image_f(dx, (float)bx.len[0], (float)bx.half[0]);
            dy = min_image_f(dy, (float)bx.len[1], (float)bx.half[1]);
            dz = min_image_f(dz, (float)bx.len[2], (float)bx.half[2]);
        }
        return dx * dx + dy * dy + dz * dz;
    }
}

// Candidate of this lane in row `row` of the open group; an empty slot's is far
// away (its tests fail).  Returns its index (a valid one in any case).
template <int G, int PREC, int IMG>
__device__ inline uint32_t load_cand(const LeafTab<G, PREC> &tab, int row, const Pos4 *__restrict__ pos,
                                     const Off4 *__restrict__ off, Cand<PREC> &c)
{
    using T = typename Cand<PREC>::T;
    const int s = row * kWave + (int)(threadIdx.x & (kWave - 1));
    const int k = s / G, slot = s % G;
    const uint2 jm = tab.jm[k];
    const bool ok = slot < (int)jm.y;
    const uint32_t j = jm.x + (ok ? slot : 0);   // (a missing leaf's entry is particle 0)
    if constexpr (PREC == SPH_FP64) {
        const auto *q = as_global((const double *)(pos + j));
        c.x = q[0];
        c.y = q[1];
        c.z = q[2];
    } else {
        const auto *q = as_global((const float *)(off + j));
        c.x = q[0];
        c.y = q[1];
        c.z = q[2];
    }
    if constexpr (PREC != SPH_FP64 || IMG == kImgShift) {
        c.ox = tab.ox[k];
        c.oy = tab.oy[k];
        c.oz = tab.oz[k];
    }
    c.x = ok ? c.x : (PREC == SPH_FP64 ? (T)1e150 : (T)1e18f);
    return j;
}

__device__ inline uint64_t readlane64(uint64_t v, int l)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}
__device__ inline double readlane_d(double v, int l)
{
    return __builtin_bit_cast(double, readlane64(__builtin_bit_cast(uint64_t, v), l));
}

// Number of set bits of a ballot below this lane.
__device__ inline uint32_t rank_of(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// The open group's candidates against the home particles.  hit(r2, thr, w) is
// the ballot of a row's test (w: the value load(j) gave for the candidate), and
// put(at, rank, slot, r2, w) takes a hit at place at + rank of the lists (`cap`
// >= 64 places for each home particle, one after the other).  cnt (lane p)
// counts the hits held.  Returns the home
// particle whose hit list is full: the caller empties that list (or all of
// them), sets cnt to match and calls again to go on (lmask then holds what is
// left of the group); -1 when the group is done.  Which hits a list holds when
// it is full depends on the particle and the rows alone.
template <int G, int PREC, int IMG, int NR, class Load, class Hit, class Put>
__device__ inline int test_rows(const LeafTab<G, PREC> &tab, const HomeTab<G, PREC> &H, int count,
                                const Box &bx, const Pos4 *__restrict__ pos,
                                const Off4 *__restrict__ off, uint64_t &lmask, int &cnt, int cap,
                                bool diag, int &tested, Load load, Hit hit, Put put)
{
    constexpr int LPR = kWave / G;                      // leaves per row
    constexpr uint32_t RM = (1u << LPR) - 1;            // one row's leaves
    constexpr uint32_t BM = NR * LPR >= 32 ? ~0u : (1u << (NR * LPR)) - 1;
    static_assert(NR * LPR <= 32, "a block's leaves fit 32 bits");
    using T = typename Cand<PREC>::T;
    const int lane = threadIdx.x & (kWave - 1);
    const int nrows = (count + LPR - 1) / LPR;
    for (int r0 = 0; r0 < nrows; r0 += NR) {
        // home particles with a near leaf among these rows
        const uint32_t near = (uint32_t)(lmask >> (r0 * LPR)) & BM;
        uint64_t todo = __ballot(near != 0);
        if (todo == 0) continue;
        if (diag)
            for (int r = 0; r < NR; r++)
                tested += (int)__popcll(__ballot(((near >> (r * LPR)) & RM) != 0));
        Cand<PREC> c[NR];
        decltype(load(0u)) w[NR];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int r = 0; r < NR; r++) w[r] = load(load_cand<G, PREC, IMG>(tab, r0 + r, pos, off, c[r]));
        __builtin_amdgcn_s_setprio(0);
        do {
            const int p = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            T hx, hy, hz, thr;
            if constexpr (PREC == SPH_FP64) {
                const HomeRow h = H.d[p];
                hx = h.x; hy = h.y; hz = h.z; thr = h.thr;
            } else {
                const HomeRowF h = H.f[p];
                hx = h.x; hy = h.y; hz = h.z; thr = h.thr;
            }
            const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)near, p);
            int have = __builtin_amdgcn_readlane(cnt, p);
            int full = -1;
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (!((bits >> (r * LPR)) & RM)) continue;
                T dx, dy, dz;
                const T r2 = separation<PREC, IMG>(bx, hx, hy, hz, c[r].x, c[r].y, c[r].z, c[r].ox,
                                                   c[r].oy, c[r].oz, dx, dy, dz);
                const uint64_t m = hit(r2, thr, w[r]);
                const int to = have + (int)__popcll(m);
                if (to > cap) {
                    full = r;
                    goto filled;
                }
                if (__builtin_amdgcn_inverse_ballot_w64(m))
                    put((uint32_t)(p * cap + have), rank_of(m), (r0 + r) * kWave + lane, r2, w[r]);
                have = to;
            }
        filled:
            cnt = lane == p ? have : cnt;
            if (full >= 0) {
                // what is done leaves the masks: these rows of the particles
                // before p, and of p the rows before the full one
                const uint32_t mine = lane < p ? BM : (lane == p ? (1u << (full * LPR)) - 1u : 0u);
                lmask &= ~((uint64_t)mine << (r0 * LPR));
                return p;
            }
        } while (todo);
        // these rows are done for every home particle
        lmask &= ~((uint64_t)BM << (r0 * LPR));
    }
    return -1;
}

// ---------------------------------------------------------------------------
// Batches: one launch evaluates many independent particle sets.  Every
// request has its own argument block in device memory; a wave claims a
// global leaf index over the concatenation of the requests' leaves and maps
// it back to (request, leaf) through an LDS prefix of the leaf counts.  The
// work done for a leaf depends on its own request only, so a set gives the
// same bits alone and inside any mix.
// ---------------------------------------------------------------------------
// Waves per SIMD the pair kernels are built for (<= 128 VGPRs, <= 10 KB of
// LDS per wave).  Measured on MI355X: occupancy decides these latency-bound
// loops; each step from 2 to 4 waves per SIMD pays for the register spills it
// costs.
template <int PREC>
constexpr int pair_waves_per_simd() { return 4; }


template <class Args>
__device__ inline void batch_prefix(const Batch<Args> &B, uint32_t *pre)
{
    // the host keeps the total leaf count (<= total particles) below 2^32
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        pre[0] = 0;
        for (int r = 0; r < B.nreq; r++) {
            const uint32_t *lc = B.req[r]->leaf_count;
            acc += lc ? *lc : (uint32_t)B.req[r]->tree->cnt[0];
            pre[r + 1] = acc;
        }
    }
    __syncthreads();
}

// request holding global leaf g: largest r with pre[r] <= g
__device__ inline int find_req(const uint32_t *pre, int nreq, int64_t g)
{
    int lo = 0, hi = nreq - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int64_t)pre[mid] <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// ---------------------------------------------------------------------------
// Density loop + h solve
// ---------------------------------------------------------------------------

// FP64 evaluations keep, instead of the sums of m f and m q f' alone, what
// gives the kernel sum at any nearby h without another pass over the
// neighbours.  With q' = q / (1 + x) for h' = h (1 + x), a' = (R - q')_+ is
// (a + R x) / (1 + x) while no neighbour enters or leaves the support of one
// of the kernel's pieces, so
//   sum m f(q') = (1 + x)^-N (D0 + x D1 + x^2 D2 + x^3 D3 ...),
// N = 3 (M4: exact with D0..D3) or 5 (quintic: D4 and D5 left out, an error of
// order x^4), and the h-rho relation sum m f = eta^3 m_i / sigma is a
// polynomial in x.
template <int K>
struct Sums {
    double d0 = 0.0, d1 = 0.0, d2 = 0.0;
    double wn = 0.0;                       // D3 of unequal masses, quintic's D3
    double edge = 1e300;                   // smallest |q - knot| met
    int n = 0, n1 = 0;                     // entries inside R h, inside h
    static constexpr int N = K == SPH_KERNEL_QUINTIC ? 5 : 3;
};

template <int K, bool EQ>
__device__ inline void add_entry(Sums<K> &s, double r2, double m, double hinv, double h2)
{
    // r = r^2 / sqrt(r^2) without a branch (r^2 = 0 gives 0 * finite = 0; the
    // 1e-300 leaves any r^2 above 1e-284 unchanged); one refinement of the
    // hardware estimate
    const double q = (r2 * rsqrt_nr1(r2 + 1e-300)) * hinv;
    const bool in = r2 < h2;
    s.n += in ? 1 : 0;
    if constexpr (K == SPH_KERNEL_QUINTIC) {
        const double t3 = 3.0 - q;
        const double a = fmax(t3, 0.0), b = fmax(2.0 - q, 0.0), c = fmax(1.0 - q, 0.0);
        s.edge = fmin(s.edge, fabs(t3));
        const double a2 = a * a, b2 = b * b, c2 = c * c;
        const double a3 = a2 * a, b3 = b2 * b, c3 = c2 * c;
        const double a4 = a2 * a2, b4 = b2 * b2, c4 = c2 * c2;
        const double e0 = a4 * a - 6.0 * (b4 * b) + 15.0 * (c4 * c);
        const double e1 = 15.0 * a4 - 60.0 * b4 + 75.0 * c4;
        const double e2 = 90.0 * a3 - 240.0 * b3 + 150.0 * c3;
        const double e3 = 270.0 * a2 - 480.0 * b2 + 150.0 * c2;
        if constexpr (EQ) {
            s.d0 += e0;
            s.d1 += e1;
            s.d2 += e2;
            s.wn += e3;
        } else {
            s.d0 += m * e0;
            s.d1 += m * e1;
            s.d2 += m * e2;
            s.wn += m * e3;
        }
    } else {
        const double t2 = 2.0 - q, t1 = 1.0 - q;
        const double a = fmax(t2, 0.0), b = fmax(t1, 0.0);
        s.edge = fmin(fmin(s.edge, fabs(t2)), fabs(t1));
        const double a2 = a * a, b2 = b * b;
        const double e0 = (0.25 * a2) * a - b2 * b;
        const double e1 = 0.5 * a2 - b2;     // x 3
        const double e2 = a - b;             // x 3
        const bool in1 = t1 > 0.0;
        if constexpr (EQ) {
            s.d0 += e0;
            s.d1 += e1;
            s.d2 += e2;
            s.n1 += in1 ? 1 : 0;
        } else {
            s.d0 += m * e0;
            s.d1 += m * e1;
            s.d2 += m * e2;
            s.wn += m * ((in ? 2.0 : 0.0) - (in1 ? 1.0 : 0.0));
        }
    }
}

template <int KK>
__device__ inline double group_min(double v)
{
    if constexpr (KK >= 2) v = fmin(v, xlane<1>(v));
    if constexpr (KK >= 4) v = fmin(v, xlane<2>(v));
    if constexpr (KK >= 8) v = fmin(v, xlane<4>(v));
    if constexpr (KK >= 16) v = fmin(v, xlane<8>(v));
    return v;
}

// A tight tolerance: the result then does not depend on how the root was
// approached, and the polynomial above may stand in for a pass.  With a loose
// one (the paper's 1 %) the solve stops at whatever h meets it, so it keeps to
// the plain Newton path.
constexpr double kTightTol = 1e-9;

template <int G, int PREC, int K>
__global__ __launch_bounds__(kWave, pair_waves_per_simd<PREC>()) void k_density(Batch<DensArgs> B)
{
    constexpr int LPP = kWave / G;   // lanes per home particle
    constexpr int KP = Kern<K>::list;
    constexpr double RK = Kern<K>::R, SIG = Kern<K>::sigma;
    constexpr bool F64 = PREC == SPH_FP64;
    // list entries that the lanes of a particle read per step: 4 each
    constexpr int CHUNK = 4 * LPP;
    static_assert(KP % CHUNK == 0, "lists hold whole steps");
    __shared__ WalkBuf wb;
    __shared__ TreeInfo T;
    __shared__ union {
        LeafTab<G, PREC> tab;
        uint32_t walk_spare[kFront];   // lent to walks, which run between sweeps
    } S;
    __shared__ HomeTab<G, PREC> H;
    __shared__ uint32_t pre[kMaxBatch + 1];
    batch_prefix(B, pre);
    const int lane = threadIdx.x;
    const int p = lane / LPP, q = lane % LPP;
    // Candidate lists of this block: for every home particle up to KP entries
    // (r^2, and m unless all masses are equal) of the candidates within R Rc
    // of it, in the order a sweep meets them, one particle after the other.
    // FP32-pair forms every r^2 in single precision, so its list holds them
    // as floats (half the bytes, the same values); FP64 lists hold doubles.
    // A particle's lanes read 64 consecutive bytes of its list per load.
    using ListR2 = std::conditional_t<F64, double, float>;
    double *const cslice = B.cache + (size_t)blockIdx.x * (2 * KP * G);
    ListR2 *const cr2 = reinterpret_cast<ListR2 *>(cslice);
    double *const cm = cslice + KP * G;
    // the request's counters, lane k for counts[k] (no scalar registers)
    int64_t tally = 0;
    auto count_up = [&](int k, int v) { tally += lane == k ? v : 0; };
    int cur = -1;
    const __attribute__((address_space(4))) DensArgs *Ap = nullptr;
    // flushed when the wave moves to another request
    auto flush_counts = [&]() {
        if (cur >= 0 && tally != 0) {
            unsigned long long *to = (unsigned long long *)&Ap->counts[lane];
            if (lane == kCntNrMax) atomicMax(to, (unsigned long long)tally);
            else atomicAdd(to, (unsigned long long)tally);
        }
        tally = 0;
    };
    for_each_home_leaf(pre[B.nreq], B.work, B.claim, [&](int64_t gleaf) {
        // the request and its argument block are wave-uniform (scalar registers)
        const int r = __builtin_amdgcn_readfirstlane(find_req(pre, B.nreq, gleaf));
        if (r != cur) {
            flush_counts();
            cur = r;
            Ap = as_const(B.req[r]);
            load_tree(Ap->tree, T);
        }
        const auto &A = *Ap;
        const int64_t li = gleaf - (int64_t)__builtin_amdgcn_readfirstlane(pre[r]);
        const int64_t leaf = A.leaf_list ? (int64_t)as_const(A.leaf_list)[li] : li;
        if (A.leaf_act && as_const(A.leaf_act)[leaf] == 0) return;   // no active particle
        const int64_t first = as_const(A.lstart)[leaf];
        const int nhome = (int)(as_const(A.lstart)[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome && (!A.active || as_global(A.active)[i] != 0);
        const int64_t ii = active ? i : first;
        const double mi = as_global(A.m)[ii];
        const double mu = as_const(A.mrange)[0];
        const bool equal_m = mu == as_const(A.mrange)[1];
        const bool tight = F64 && A.h_rtol <= kTightTol;
        double h = as_global((const double *)A.h)[ii];
        double lo_b = 0.0, hi_b = INFINITY;
        bool conv = !active;
        double h_out = h, rho_out = 0.0, om_out = 1.0;
        int n_out = 0;
        if (q == 0) {
            H.d[p].x = as_global(A.x)[ii];
            H.d[p].y = as_global(A.y)[ii];
            H.d[p].z = as_global(A.z)[ii];
            if constexpr (!F64) {
                const auto *o = as_global((const float *)(A.off + ii));
                H.f[p].x = o[0];
                H.f[p].y = o[1];
                H.f[p].z = o[2];
            }
        }

        double hcov = A.walk_margin * wave_max(active ? h : 0.0);
        auto near_home = [&](const Node &home, const Box &bx) {
            const double R = RK * hcov * (1.0 + 1e-10);
            const double R2 = R * R;
            return [&bx, &home, R2](const Node &nd) { return box_gap2(home, nd, bx) < R2; };
        };
        auto walk_home = [&]() {
            const Node home = load_const(reload(A.nodes) + leaf);
            const Box bx = load_const(&reload(B.req[r])->box);
            const WalkResult w = walk(T, A.nodes, near_home(home, bx), wb, S.walk_spare);
            count_up(kCntDensWalks, 1);
            if (w.lev) count_up(kCntDensOverflows, 1);
            return w;
        };
        // the walk and the candidate loads are chains of dependent loads: the
        // wave issues them at raised priority, ahead of waves in their
        // arithmetic (measured: the force loop 1 % faster, the density loop
        // unchanged)
        __builtin_amdgcn_s_setprio(2);
        WalkResult wr = walk_home();
        __builtin_amdgcn_s_setprio(0);
        int iter = 0;
        int evals_leaf = 0;   // this lane's density pairs evaluated for this leaf
        // list state of this particle: `cached` = the list holds every
        // candidate within R Rc; valid while h <= Rc.  count: its entries.
        bool cached = false;
        double Rc = 0.0;
        int count = 0;
        for (;;) {
            const double hinv = 1.0 / h;
            const double h2x4 = (RK * h) * (RK * h);
            Sums<K> sm;
            double s0 = 0.0, s2 = 0.0;   // FP32-pair sums
            const float h2x4f = (float)h2x4, hinvf = (float)hinv;
            // the pair terms of this particle's list entries [0, n), its lanes
            // sharing them four at a time; entries past n up to a whole step
            // are far away and add nothing
            auto eval_list = [&](int n) {
                const ListR2 *l = cr2 + p * KP;
                const double *lm = cm + p * KP;
                if constexpr (F64) {
                    using D2 = double __attribute__((ext_vector_type(2)));
                    auto sums = [&](auto eq) {
                        constexpr bool EQ = decltype(eq)::value;
                        for (int e = 2 * q; e < n; e += CHUNK) {
                            const D2 u = *(const __attribute__((address_space(1))) D2 *)(l + e);
                            const D2 v = *(const __attribute__((address_space(1))) D2 *)(l + e + 2 * LPP);
                            D2 mu2{}, mv2{};
                            if constexpr (!EQ) {
                                mu2 = *(const __attribute__((address_space(1))) D2 *)(lm + e);
                                mv2 = *(const __attribute__((address_space(1))) D2 *)(lm + e + 2 * LPP);
                            }
                            add_entry<K, EQ>(sm, u.x, mu2.x, hinv, h2x4);
                            add_entry<K, EQ>(sm, u.y, mu2.y, hinv, h2x4);
                            add_entry<K, EQ>(sm, v.x, mv2.x, hinv, h2x4);
                            add_entry<K, EQ>(sm, v.y, mv2.y, hinv, h2x4);
                        }
                    };
                    if (equal_m) sums(std::true_type{});
                    else sums(std::false_type{});
                } else {
                    using F4 = float __attribute__((ext_vector_type(4)));
                    using D4 = double __attribute__((ext_vector_type(4)));
                    for (int e = 4 * q; e < n; e += CHUNK) {
                        const F4 u = *(const __attribute__((address_space(1))) F4 *)(l + e);
                        D4 mw{mu, mu, mu, mu};
                        if (!equal_m) mw = *(const __attribute__((address_space(1))) D4 *)(lm + e);
#pragma unroll
                        for (int k = 0; k < 4; k++) {
                            // branch-free: an entry outside R h adds 0 * f
                            const bool in = u[k] < h2x4f;
                            const double mj = in ? mw[k] : 0.0;
                            float f, df;
                            const float qq = sqrtf(u[k]) * hinvf;
                            kern<K>(qq, f, df);
                            s0 += mj * (double)f;
                            s2 += mj * (double)(qq * df);
                            sm.n += in ? 1 : 0;
                        }
                    }
                }
            };
            // the n entries of home particle pp's list, which is full, added to
            // its sums (on its first lane) by the whole wave; the list starts
            // afresh.  n and the order depend on the particle and the rows
            // alone
            auto empty_list = [&](int pp, int n) {
                Sums<K> t;
                double t0 = 0.0, t2 = 0.0;
                const double hv = readlane_d(hinv, pp * LPP), hh = readlane_d(h2x4, pp * LPP);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                for (int e = lane; e < n; e += kWave) {
                    const ListR2 r2 = as_global(cr2)[pp * KP + e];
                    const double mw = equal_m ? mu : as_global(cm)[pp * KP + e];
                    if constexpr (F64) {
                        if (equal_m) add_entry<K, true>(t, r2, mw, hv, hh);
                        else add_entry<K, false>(t, r2, mw, hv, hh);
                    } else {
                        const bool in = r2 < (float)hh;
                        const double mj = in ? mw : 0.0;
                        float f, df;
                        const float qq = sqrtf(r2) * (float)hv;
                        kern<K>(qq, f, df);
                        t0 += mj * (double)f;
                        t2 += mj * (double)(qq * df);
                        t.n += in ? 1 : 0;
                    }
                }
                const int n0 = (int)wave_sum_int(t.n), n1 = (int)wave_sum_int(t.n1);
                const bool own = lane == pp * LPP;
                sm.n += own ? n0 : 0;
                if constexpr (F64) {
                    sm.n1 += own ? n1 : 0;
                    const double d0 = wave_sum(t.d0), d1 = wave_sum(t.d1), d2 = wave_sum(t.d2);
                    const double wn = wave_sum(t.wn);
                    sm.d0 += own ? d0 : 0.0;
                    sm.d1 += own ? d1 : 0.0;
                    sm.d2 += own ? d2 : 0.0;
                    sm.wn += own ? wn : 0.0;
                } else {
                    t0 = wave_sum(t0);
                    t2 = wave_sum(t2);
                    s0 += own ? t0 : 0.0;
                    s2 += own ? t2 : 0.0;
                }
            };
            // entries [n, whole step) of this particle's list: far away
            auto pad_list = [&](int n) {
                const int end = (n + CHUNK - 1) / CHUNK * CHUNK;
                for (int e = n + q; e < end; e += LPP) {
                    cr2[p * KP + e] = F64 ? (ListR2)1e300 : (ListR2)1e30f;
                    if (!equal_m) cm[p * KP + e] = 0.0;
                }
                // the lanes read what other lanes of the wave stored
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            };
            if (__ballot(!conv && !cached) != 0ull) {
                // sweep: every particle still iterating rebuilds its list
                // around its current h.  A list that fills up is added to the
                // sums and started afresh; it cannot serve later steps then
                double rc2 = -1.0;
                if (!conv) {
                    Rc = fmin(kCacheGrow * h, hcov);
                    rc2 = (RK * Rc) * (RK * Rc) * (1.0 + 1e-6);   // far above rounding
                }
                wave_lds_sync();
                if (q == 0) {
                    H.d[p].thr = rc2;
                    if constexpr (!F64) H.f[p].thr = (float)rc2;
                }
                wave_lds_sync();
                const uint64_t lanes_in = __ballot(!conv);
                uint64_t takes_part = 0;   // bit p: home particle p
#pragma unroll
                for (int k = 0; k < G; k++)
                    takes_part |= ((lanes_in >> (k * LPP)) & 1ull) << k;
                const int depth = group_depth<G>(wr.n, B.stage > 0 ? B.stage * G / 2 : kGroup);
                uint64_t emptied = 0;      // bit p: the list of home particle p is not complete
                int held = 0;              // lane p: entries in the list of home particle p
                int64_t at = 0;
                const uint32_t *leaves = nullptr;
                const auto &Q = *reload(Ap);
                const Node home = load_const(reload(A.nodes) + leaf);
                const Box bx = load_const(&reload(B.req[r])->box);
                auto test = near_home(home, bx);
                for (;;) {
                    const int ng = next_group(T, Q.nodes, wr, test, wb, depth, at, leaves);
                    if (ng == 0) break;
                    uint64_t lmask;
                    const int img = open_group<G, PREC, K>(leaves, ng, Q.lstart, Q.nodes, home, bx, hcov,
                                                           H, takes_part, S.tab, lmask);
                    count_up(kCntDensVisits, ng);
                    int tested = 0;
                    const bool diag = Q.count_tests != 0;
                    auto load = [&](uint32_t j) { return equal_m ? mu : as_global(Q.m)[j]; };
                    auto hit = [&](auto r2, auto thr, double) { return __ballot(r2 < thr); };
                    auto put = [&](uint32_t at, uint32_t rank, int, auto r2, double mw) {
                        // (fixed uniform base, 32-bit lane offset)
                        auto *to = (__attribute__((address_space(1))) char *)cr2;
                        *(__attribute__((address_space(1))) ListR2 *)(to + (at + rank) * (uint32_t)sizeof(ListR2)) = r2;
                        if (!equal_m) {
                            auto *tm = (__attribute__((address_space(1))) char *)cm;
                            *(__attribute__((address_space(1))) double *)(tm + (at + rank) * 8u) = mw;
                        }
                    };
                    for (;;) {
                        int full;
                        if (img == kImgNone || (img == kImgShift && !F64))
                            full = test_rows<G, PREC, kImgNone, kRows>(S.tab, H, ng, bx, Q.pos, Q.off, lmask,
                                                                       held, KP, diag, tested, load, hit, put);
                        else if (img == kImgShift)
                            full = test_rows<G, PREC, F64 ? kImgShift : kImgNone, kRows / 2>(
                                S.tab, H, ng, bx, Q.pos, Q.off, lmask, held, KP, diag, tested, load, hit, put);
                        else
                            full = test_rows<G, PREC, kImgPair, kRows / 2>(
                                S.tab, H, ng, bx, Q.pos, Q.off, lmask, held, KP, diag, tested, load, hit, put);
                        if (full < 0) break;
                        empty_list(full, __builtin_amdgcn_readlane(held, full));
                        held = lane == full ? 0 : held;
                        count_up(kCntDensListOverflows, (emptied >> full) & 1 ? 0 : 1);
                        emptied |= 1ull << full;
                    }
                    if (diag) {
                        count_up(kCntDensBoxes, ng * (int)__popcll(takes_part));
                        count_up(kCntDensTests, tested * kWave);
                    }
                    wave_lds_sync();   // the next group rewrites the table
                }
                const int mine = __shfl(held, p);   // every lane takes part
                count = conv ? 0 : mine;
                cached = !conv && !((emptied >> p) & 1);
                pad_list(count);
            }
            eval_list(conv ? 0 : count);
            // one evaluation for every particle still iterating (uniform)
            count_up(kCntNrTotal, (int)__popcll(__ballot(!conv && q == 0)));
            const int cnt = group_sum<LPP>(sm.n) - 1;   // without the particle itself
            // x: relative change of h to the root (the polynomial's, where it
            // could be solved), b1: the polynomial's derivative there
            double x = 0.0, b1 = 0.0, edge = 0.0;
            bool poly = false;
            if constexpr (F64) {
                const double sc = equal_m ? mu : 1.0;
                const double f3 = K == SPH_KERNEL_QUINTIC ? 1.0 : 3.0;
                const double D0 = sc * group_sum<LPP>(sm.d0);
                const double D1 = sc * (f3 * group_sum<LPP>(sm.d1));
                const double D2 = sc * (f3 * group_sum<LPP>(sm.d2));
                double D3 = group_sum<LPP>(sm.wn);
                if constexpr (K != SPH_KERNEL_QUINTIC) {
                    const int n1 = group_sum<LPP>(sm.n1);
                    if (equal_m) D3 = (double)(2 * (cnt + 1) - n1);
                }
                D3 *= sc;
                edge = group_min<LPP>(sm.edge);
                constexpr double N = Sums<K>::N;
                s0 = D0;
                s2 = N * D0 - D1;
                if (tight) {
                    // (1 + x)^N eta^3 m / sigma against D0 + x D1 + ..., through x^3
                    const double kt = A.eta3 * mi / SIG;
                    const double e0 = D0 - kt, e1 = D1 - N * kt;
                    const double e2 = D2 - (N * (N - 1.0) / 2.0) * kt;
                    const double e3 = D3 - (N * (N - 1.0) * (N - 2.0) / 6.0) * kt;
                    double st = 0.0;
                    for (int k = 0; k < 8; k++) {
                        const double f = ((e3 * x + e2) * x + e1) * x + e0;
                        const double g1 = (3.0 * e3 * x + 2.0 * e2) * x + e1;
                        st = f / g1;
                        x -= st;
                        // (a lane whose solve runs away ends as not solved)
                        if (__ballot(!conv && fabs(st) > 1e-16 + 1e-15 * fabs(x) && fabs(x) < 1.0) == 0ull)
                            break;
                    }
                    poly = fabs(x) < 0.5 && fabs(st) <= 1e-15 + 1e-12 * fabs(x);
                    b1 = (3.0 * D3 * x + 2.0 * D2) * x + D1;
                }
            } else {
                s0 = group_sum<LPP>(s0);
                s2 = group_sum<LPP>(s2);
            }
            if (!conv && q == 0) evals_leaf += cnt;
            if (!conv) {
                // the root of g(h) = h^3 rho(h) - eta^3 m = sigma sum m f - eta^3 m
                // (non-decreasing in h) is the h of the h-rho relation
                const double g = SIG * s0 - A.eta3 * mi;
                const double om = -s2 / (3.0 * s0);
                double step, fp = 1.0;
                if (poly) {
                    step = -h * x;
                } else {
                    // Newton on the equivalent F(h) = h - eta (m / rho(h))^(1/3),
                    // which is exactly linear where rho does not vary over the
                    // kernel and so converges in fewer steps than Newton on the
                    // cubic g; F has the sign of g, and F'(h) = 1 - (h*/h)(1 -
                    // Omega) with h* = h - F
                    const double hs = h * cbrt(A.eta3 * mi / (SIG * s0));
                    fp = 1.0 - (hs * hinv) * (1.0 - om);
                    step = fp > 0.0 ? (h - hs) / fp : INFINITY;
                }
                h_out = h;
                rho_out = SIG * s0 * hinv * hinv * hinv;
                om_out = om;
                n_out = cnt;
                // the step decides convergence before any safeguard: h and rho
                // are final once the step would change h by at most h_rtol h and rho
                // (d ln rho / d ln h = 3 (Omega - 1)) by at most h_rtol rho, down to
                // a zero step at the root
                const double sens = fmax(1.0, 3.0 * fabs(om - 1.0));
                if (g == 0.0 || fabs(step) * sens <= A.h_rtol * h) {
                    conv = true;
                } else {
                    if (g < 0.0) lo_b = fmax(lo_b, h); else hi_b = fmin(hi_b, h);
                    double hn = fp > 0.0 ? h - step : (g < 0.0 ? 2.0 * h : 0.5 * h);
                    hn = fmin(fmax(hn, 0.5 * h), 2.0 * h);
                    // outside the bracket of known signs: bisect it
                    const bool inside = hn > lo_b && hn < hi_b;
                    if (!inside) hn = hi_b < INFINITY ? 0.5 * (lo_b + hi_b) : 2.0 * h;
                    // the polynomial is the kernel sum at hn itself if no
                    // neighbour crosses a knot on the way (the 1e-13 covers the
                    // rounding of q) and the list holds every neighbour there:
                    // the solve is done without another pass
                    const bool exact = poly && inside && cached && hn <= Rc &&
                                       edge > RK * fabs(x) * (1.0 + 1e-9) + 1e-13 &&
                                       (K != SPH_KERNEL_QUINTIC || fabs(x) <= 1e-5);
                    if (!(hn == hn)) {
                        conv = true;
                    } else if (exact) {
                        conv = true;
                        constexpr double N = Sums<K>::N;
                        const double kt = A.eta3 * mi / SIG, y = 1.0 + x;
                        const double yn = K == SPH_KERNEL_QUINTIC ? (y * y) * (y * y) : y * y;
                        h_out = hn;
                        rho_out = A.eta3 * mi / (hn * hn * hn);
                        om_out = -(N * kt - b1 / yn) / (3.0 * kt);
                    } else {
                        h = hn;
                    }
                }
            }
            if (cached && !(h <= Rc)) cached = false;
            iter++;
            if (__ballot(!conv) == 0ull || iter >= A.max_iter) break;
            const double hmx = wave_max(conv ? 0.0 : h);
            if (hmx > hcov) {
                hcov = A.walk_margin * hmx;
                __builtin_amdgcn_s_setprio(2);
                wr = walk_home();
                __builtin_amdgcn_s_setprio(0);
            }
        }
        bool bad = false, slow = false, wide = false;
        if (active && q == 0) {
            A.h[i] = h_out;
            A.rho[i] = rho_out;
            A.omega[i] = om_out;
            A.nngb[i] = n_out;
            bad = !isfinite(h_out) || !isfinite(rho_out) || !isfinite(om_out) || !(rho_out > 0.0);
            slow = !bad && !conv;
            const auto &bx = reload(Ap)->box;
            if (bx.periodic) {
                const double Lmin = fmin(fmin(bx.len[0], bx.len[1]), bx.len[2]);
                wide = !(2.0 * RK * h_out < Lmin);
            }
        }
        report(A.status, bad, kFlagNonFinite, 2);
        report(A.status, slow, kFlagNotConverged, 1);
        report(A.status, wide, kFlagStencil, 3);
        tally = lane == kCntNrMax && iter > tally ? iter : tally;
        count_up(kCntDensEvals, (int)wave_sum_int(evals_leaf));
        wave_lds_sync();   // the home table is rewritten for the next leaf
    });
    flush_counts();
}

// ---------------------------------------------------------------------------
// Force loop
// ---------------------------------------------------------------------------

// Hits held per home particle between two flushes (16-bit ids, 4 KB of LDS:
// with the walk buffer and the tables a wave stays within 10 KB up to G = 16).
// At least the 64 hits that one row can give.
template <int G>
constexpr int force_list() { return 2048 / G; }

// AC: the launch carries artificial conductivity (some set of the batch has
// alpha_AC > 0; a set with alpha_AC = 0 then adds exact zeros).
// SW: the launch carries per-particle alpha or the velocity divergence and
// curl (the artificial-viscosity switches); a set without them uses alpha_AV
// for every pair as the plain variant does.
template <int G, int PREC, bool AC, bool SW, int K>
__global__ __launch_bounds__(kWave, pair_waves_per_simd<PREC>()) void k_forces(Batch<ForceArgs> B)
{
    constexpr int LPP = kWave / G;
    constexpr int CAP = force_list<G>();
    constexpr bool F64 = PREC == SPH_FP64;
    __shared__ WalkBuf wb;
    __shared__ TreeInfo T;
    __shared__ LeafTab<G, PREC> tab;
    __shared__ union {
        uint16_t id[G * CAP];          // hits of each home particle: slots of the open group
        uint32_t walk_spare[kFront];   // lent to walks, which run between groups
    } S;
    __shared__ HomeTab<G, PREC> H;
    __shared__ uint32_t pre[kMaxBatch + 1];
    batch_prefix(B, pre);
    const int lane = threadIdx.x;
    const int p = lane / LPP, q = lane % LPP;
    // the request's counters, lane k for counts[k] (no scalar registers)
    int64_t tally = 0;
    auto count_up = [&](int k, int v) { tally += lane == k ? v : 0; };
    int cur = -1;
    const __attribute__((address_space(4))) ForceArgs *Fp = nullptr;
    auto flush_counts = [&]() {
        if (cur >= 0 && tally != 0)
            atomicAdd((unsigned long long *)&Fp->counts[lane], (unsigned long long)tally);
        tally = 0;
    };
    for_each_home_leaf(pre[B.nreq], B.work, B.claim, [&](int64_t gleaf) {
        const int r = __builtin_amdgcn_readfirstlane(find_req(pre, B.nreq, gleaf));
        if (r != cur) {
            flush_counts();
            cur = r;
            Fp = as_const(B.req[r]);
            load_tree(Fp->tree, T);
        }
        const auto &F = *Fp;
        const int64_t li = gleaf - (int64_t)__builtin_amdgcn_readfirstlane(pre[r]);
        const int64_t leaf = F.leaf_list ? (int64_t)as_const(F.leaf_list)[li] : li;
        if (F.leaf_act && as_const(F.leaf_act)[leaf] == 0) return;   // no active particle
        const Box bx = load_const(&B.req[r]->box);
        const double alpha = F.alpha, beta = F.beta;
        const double *const alpha_p = SW ? F.alpha_p : nullptr;
        const double alpha_ac = AC ? F.alpha_ac : 0.0, u_per_c2 = AC ? F.u_per_c2 : 0.0;
        const double inv_gamma = AC ? F.inv_gamma : 0.0;
        const bool ac_price = AC && F.ac_price != 0;
        const int64_t first = as_const(F.lstart)[leaf];
        const int nhome = (int)(as_const(F.lstart)[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome && (!F.active || as_global(F.active)[i] != 0);
        const int64_t ii = p < nhome ? i : first;
        const double hx = as_global(F.x)[ii], hy = as_global(F.y)[ii], hz = as_global(F.z)[ii];
        float hfx = 0.f, hfy = 0.f, hfz = 0.f;
        if constexpr (!F64) {
            const auto *o = as_global((const float *)(F.off + ii));
            hfx = o[0];
            hfy = o[1];
            hfz = o[2];
        }
        const ForceRec ri = load_global(F.rec + ii);
        const double vxi = ri.vx, vyi = ri.vy, vzi = ri.vz;
        const double hi = as_global(F.h)[ii], hinvi = ri.hinv;
        const double rhoi = ri.rho, Ai = ri.A, ci = ri.c;
        const double alpha_i = (SW && alpha_p) ? as_global(alpha_p)[ii] : alpha;
        constexpr double RK = Kern<K>::R, SIG = Kern<K>::sigma;
        const double hi2x4 = (RK * hi) * (RK * hi);
        const double gfi = SIG * (hinvi * hinvi) * (hinvi * hinvi);
        const float hinvif = (float)hinvi;
        const float gfif = (float)SIG * (hinvif * hinvif) * (hinvif * hinvif);
        // FP32-pair: the home particle's values as its single-precision record holds them
        const float vxif = (float)vxi, vyif = (float)vyi, vzif = (float)vzi;
        const float Aif = (float)Ai, cif = (float)ci, rhoif = (float)rhoi;
        const Node home = load_const(F.nodes + leaf);
        if (q == 0) {
            H.d[p] = HomeRow{hx, hy, hz, active ? hi2x4 : -1.0};
            if constexpr (!F64) H.f[p] = HomeRowF{hfx, hfy, hfz, active ? (float)hi2x4 : -1.f};
        }
        const uint64_t lanes_in = __ballot(active);
        uint64_t takes_part = 0;   // bit p: home particle p
#pragma unroll
        for (int k = 0; k < G; k++) takes_part |= ((lanes_in >> (k * LPP)) & 1ull) << k;
        // symmetric criterion: a node can hold force neighbours of the home leaf
        // if its box is closer than 2 max(h over home, h over node)
        auto test = [&bx, &home](const Node &nd) {
            const double R = RK * fmax(home.hmax, nd.hmax) * (1.0 + 1e-10);
            return box_gap2(home, nd, bx) < R * R;
        };
        // walk and candidate loads at raised priority, as in the density loop
        __builtin_amdgcn_s_setprio(2);
        const WalkResult wr = walk(T, F.nodes, test, wb, S.walk_spare);
        __builtin_amdgcn_s_setprio(0);
        if (wr.lev) count_up(kCntForceOverflows, 1);

        double axi = 0.0, ayi = 0.0, azi = 0.0, dui = 0.0, vs_max = -INFINITY;
        double dvs = 0.0, cxs = 0.0, cys = 0.0, czs = 0.0;   // div v, curl v sums (SW)
        int cnt = 0, selfs = 0;
        int lmx_l = 0;                                       // block time-steps
        const int lev_i = F.lev ? as_global(F.lev)[ii] : 0;
        // FP32-pair: the neighbours' single-precision records (32 bytes)
        using JData = std::conditional_t<F64, ForceRec, ForceRec32>;
        using Real = std::conditional_t<F64, double, float>;
        auto pair_terms = [&](uint32_t j, const JData &d, Real sdx, Real sdy, Real sdz, Real sr2) {
            const double dx = sdx, dy = sdy, dz = sdz, r2 = sr2;
            const double cj = d.c;
            if (r2 == 0.0) {
                vs_max = fmax(vs_max, PREC == SPH_FP64 ? ci + cj : (double)(cif + (float)cj));
                return;
            }
            // the pair's viscosity strength: (alpha_i + alpha_j)/2 with
            // per-particle values, alpha_AV otherwise
            const double aij = (SW && alpha_p) ? 0.5 * (alpha_i + as_global(alpha_p)[j])
                                               : alpha;
            if constexpr (PREC == SPH_FP64) {
                const double rinv = rsqrt_nr(r2);
                const double rr = r2 * rinv;
                const double ex = dx * rinv, ey = dy * rinv, ez = dz * rinv;
                const double hinvj = d.hinv;
                const double gfj = SIG * (hinvj * hinvj) * (hinvj * hinvj);
                double fi, dfi, fj, dfj;
                kern<K>(rr * hinvi, fi, dfi);
                kern<K>(rr * hinvj, fj, dfj);
                double gi, gj, gsum;
                sym_grads(gfi, dfi, gfj, dfj, gi, gj, gsum);
                const double w = ((vxi - d.vx) * ex + (vyi - d.vy) * ey) + (vzi - d.vz) * ez;
                const double mj = d.m;
                double cvec = -mj * sym_dot2(Ai, gi, d.A, gj);
                double cdu = Ai * mj * gi * w;
                const double wneg = fmin(w, 0.0);
                const double vs = (ci + cj) - beta * wneg;
                vs_max = fmax(vs_max, vs);
                const double rbinv = rcp_nr(0.5 * (rhoi + d.rho));
                const double visc = (mj * rbinv) * aij * vs * wneg;
                const double gbar = 0.5 * gsum;
                cvec += visc * gbar;
                cdu -= visc * 0.5 * wneg * gbar;
                if constexpr (AC) {
                    // u and P of both particles from their sound speeds
                    const double c2i = ci * ci, c2j = cj * cj;
                    const double vc = ac_price
                        ? sqrt(fabs(rhoi * c2i - d.rho * c2j) * inv_gamma * rbinv)
                        : fabs(w);
                    cdu += (mj * rbinv) * alpha_ac * vc * ((c2i - c2j) * u_per_c2) * gbar;
                }
                axi += cvec * ex;
                ayi += cvec * ey;
                azi += cvec * ez;
                dui += cdu;
                if constexpr (SW) {
                    // v_ij . G_i = w gi and v_ij x G_i = gi (v_ij x rhat)
                    const double vxij = vxi - d.vx, vyij = vyi - d.vy, vzij = vzi - d.vz;
                    dvs += mj * w * gi;
                    cxs += mj * gi * (vyij * ez - vzij * ey);
                    cys += mj * gi * (vzij * ex - vxij * ez);
                    czs += mj * gi * (vxij * ey - vyij * ex);
                }
            } else {
                const float fdx = (float)dx, fdy = (float)dy, fdz = (float)dz;
                // hardware reciprocal square root and reciprocal (1 ulp each),
                // functions of symmetric operands, so (j, i) sees the same values
                const float rinv = __builtin_amdgcn_rsqf((float)r2);
                const float rr = (float)r2 * rinv;
                const float ex = fdx * rinv, ey = fdy * rinv, ez = fdz * rinv;
                const float hinvj = d.hinv;
                // own and other kernel factors formed by the same float
                // expression, so the (j, i) pair sees exactly the values of
                // the (i, j) pair
                const float gfjf = (float)SIG * (hinvj * hinvj) * (hinvj * hinvj);
                float fi, dfi, fj, dfj;
                kern<K>(rr * hinvif, fi, dfi);
                kern<K>(rr * hinvj, fj, dfj);
                float gi, gj, gsum;
                sym_grads(gfif, dfi, gfjf, dfj, gi, gj, gsum);
                const float w = ((vxif - d.vx) * ex + (vyif - d.vy) * ey) + (vzif - d.vz) * ez;
                const float mj = d.m;
                const float cjf = d.c;
                float cvec = -mj * sym_dot2(Aif, gi, d.A, gj);
                float cdu = Aif * mj * gi * w;
                const float wneg = fminf(w, 0.0f);
                const float vs = (cif + cjf) - (float)beta * wneg;
                vs_max = fmax(vs_max, (double)vs);
                const float rbinv = __builtin_amdgcn_rcpf(0.5f * (rhoif + d.rho));
                const float visc = (mj * rbinv) * (float)aij * vs * wneg;
                const float gbar = 0.5f * gsum;
                cvec += visc * gbar;
                cdu -= visc * 0.5f * wneg * gbar;
                if constexpr (AC) {
                    // differences of u and P formed in double precision from
                    // the single-precision values both sides of the pair see
                    const double c2i = (double)cif * cif, c2j = (double)cjf * cjf;
                    const float du_ij = (float)((c2i - c2j) * u_per_c2);
                    const float vc =
                        ac_price
                            ? sqrtf((float)(fabs((double)rhoif * c2i - (double)d.rho * c2j) *
                                            inv_gamma) * rbinv)
                            : fabsf(w);
                    cdu += (mj * rbinv) * (float)alpha_ac * vc * du_ij * gbar;
                }
                axi += (double)(cvec * ex);
                ayi += (double)(cvec * ey);
                azi += (double)(cvec * ez);
                dui += (double)cdu;
                if constexpr (SW) {
                    const float vxij = vxif - d.vx, vyij = vyif - d.vy, vzij = vzif - d.vz;
                    dvs += (double)(mj * w * gi);
                    cxs += (double)(mj * gi * (vyij * ez - vzij * ey));
                    cys += (double)(mj * gi * (vzij * ex - vxij * ez));
                    czs += (double)(mj * gi * (vxij * ey - vyij * ex));
                }
            }
        };
        // block time-steps: the deepest neighbour level, and inactive
        // neighbours more than lim levels shallower marked to wake up
        auto limiter = [&](uint32_t j) {
            if (!F.lev) return;
            const int lj = as_global(F.lev)[j];
            lmx_l = lj > lmx_l ? lj : lmx_l;
            if (lj < lev_i - F.lim && as_global(F.active)[j] == 0) atomicMax(&F.mark[j], lev_i);
        };
        // the hits this particle holds, its lanes sharing them round-robin.
        // The particle itself is among the hits of its own leaf: it takes no
        // pair terms and is not counted
        auto flush = [&](int n, int img) {
            const uint32_t self = (uint32_t)i;
            for (int e = q; e < n; e += LPP) {
                const int s = S.id[p * CAP + e];
                const int k = s / G;
                const uint32_t j = tab.jm[k].x + (uint32_t)(s % G);
                Real dx, dy, dz, r2;
                JData d;
                if constexpr (F64) {
                    d = load_global(F.rec + j);
                    const auto *o = as_global((const double *)(F.pos + j));
                    const double x = o[0], y = o[1], z = o[2];
                    if (img == kImgNone)
                        r2 = separation<PREC, kImgNone, double>(bx, hx, hy, hz, x, y, z, 0.0, 0.0, 0.0,
                                                                dx, dy, dz);
                    else if (img == kImgShift)
                        r2 = separation<PREC, kImgShift, double>(bx, hx, hy, hz, x, y, z, tab.ox[k],
                                                                 tab.oy[k], tab.oz[k], dx, dy, dz);
                    else
                        r2 = separation<PREC, kImgPair, double>(bx, hx, hy, hz, x, y, z, 0.0, 0.0, 0.0,
                                                                dx, dy, dz);
                } else {
                    d = load_global(F.rec32 + j);
                    const auto *o = as_global((const float *)(F.off + j));
                    const float x = o[0], y = o[1], z = o[2];
                    if (img != kImgPair)
                        r2 = separation<PREC, kImgNone, float>(bx, hfx, hfy, hfz, x, y, z, tab.ox[k],
                                                               tab.oy[k], tab.oz[k], dx, dy, dz);
                    else
                        r2 = separation<PREC, kImgPair, float>(bx, hfx, hfy, hfz, x, y, z, tab.ox[k],
                                                               tab.oy[k], tab.oz[k], dx, dy, dz);
                }
                if (j != self) {
                    limiter(j);
                    pair_terms(j, d, dx, dy, dz, r2);
                } else {
                    selfs++;
                }
            }
        };
        const int depth = group_depth<G>(wr.n, B.stage > 0 ? B.stage * G / 2 : kGroup);
        int64_t at = 0;
        const uint32_t *leaves = nullptr;
        for (;;) {
            const int ng = next_group(T, F.nodes, wr, test, wb, depth, at, leaves);
            if (ng == 0) break;
            uint64_t lmask;
            const int img = open_group<G, PREC, K>(leaves, ng, F.lstart, F.nodes, home, bx, -1.0, H,
                                                   takes_part, tab, lmask);
            int tested = 0;
            const bool diag = F.count_tests != 0;
            // a candidate's own squared gather reach (R h)^2
            auto load = [&](uint32_t j) {
                const double hj = as_global(F.h)[j];
                return (Real)((RK * hj) * (RK * hj));
            };
            // the particle itself passes too; the flush drops it
            auto hit = [&](Real r2, Real thr, Real w) { return __ballot(r2 < thr) | __ballot(r2 < w); };
            auto put = [&](uint32_t at, uint32_t rank, int s, Real, Real) { S.id[at + rank] = (uint16_t)s; };
            int held = 0;              // lane p: hits held of home particle p
            for (;;) {
                int full;
                if (img == kImgNone || (img == kImgShift && !F64))
                    full = test_rows<G, PREC, kImgNone, kRows>(tab, H, ng, bx, F.pos, F.off, lmask, held, CAP,
                                                               diag, tested, load, hit, put);
                else if (img == kImgShift)
                    full = test_rows<G, PREC, F64 ? kImgShift : kImgNone, kRows / 2>(
                        tab, H, ng, bx, F.pos, F.off, lmask, held, CAP, diag, tested, load, hit, put);
                else
                    full = test_rows<G, PREC, kImgPair, kRows / 2>(tab, H, ng, bx, F.pos, F.off, lmask, held,
                                                                   CAP, diag, tested, load, hit, put);
                wave_lds_sync();
                const int n = __shfl(held, p);
                cnt += n;
                flush(n, img);
                held = 0;
                wave_lds_sync();
                if (full < 0) break;
            }
            if (diag) {
                count_up(kCntForceBoxes, ng * (int)__popcll(takes_part));
                count_up(kCntForceTests, tested * kWave);
            }
        }
        axi = group_sum<LPP>(axi);
        ayi = group_sum<LPP>(ayi);
        azi = group_sum<LPP>(azi);
        dui = group_sum<LPP>(dui);
        vs_max = group_max<LPP>(vs_max);
        selfs = group_sum<LPP>(selfs);
        cnt -= selfs;
        if (F.lev) lmx_l = group_max_int<LPP>(lmx_l);
        if constexpr (SW) {
            dvs = group_sum<LPP>(dvs);
            cxs = group_sum<LPP>(cxs);
            cys = group_sum<LPP>(cys);
            czs = group_sum<LPP>(czs);
        }
        bool bad = false;
        if (active && q == 0) {
            const double vsig = cnt > 0 ? vs_max : 2.0 * ci;
            F.ax[i] = axi;
            F.ay[i] = ayi;
            F.az[i] = azi;
            F.du[i] = dui;
            F.vsig[i] = vsig;
            F.dt[i] = F.ccfl * hi / vsig;
            F.nforce[i] = cnt;
            if (F.lmx) F.lmx[i] = lmx_l;
            if (SW && F.divv) {
                const double orho = as_global(F.omega)[i] * rhoi;
                F.divv[i] = -dvs / orho;
                F.curlv[i] = sqrt((cxs * cxs + cys * cys) + czs * czs) / orho;
            }
            bad = !isfinite(axi) || !isfinite(ayi) || !isfinite(azi) || !isfinite(dui) ||
                  !isfinite(vsig);
        }
        report(F.status, bad, kFlagNonFinite, 2);
        count_up(kCntForceEvals, (int)wave_sum_int((q == 0 && active) ? cnt : 0));
        wave_lds_sync();   // the home table is rewritten for the next leaf
    });
    flush_counts();
}

// ---------------------------------------------------------------------------
// Neighbour export (tests): counts, then lists in original indices
// ---------------------------------------------------------------------------

template <int G, int K>
__global__ __launch_bounds__(kWave) void k_neighbours(NgbArgs N, int pass)
{
    constexpr double RK = Kern<K>::R;
    constexpr int LPP = kWave / G;
    constexpr int PER = G / LPP;
    __shared__ WalkBuf wb;
    __shared__ uint32_t spare[kFront];
    __shared__ TreeInfo T;
    load_tree(N.tree, T);
    const int lane = threadIdx.x;
    const int p = lane / LPP, q = lane % LPP;
    const Box &bx = N.box;
    const int32_t mode = N.mode;
    int64_t overflows = 0;
    for_each_home_leaf(T.cnt[0], N.work, 1, [&](int64_t leaf) {
        const int64_t first = N.lstart[leaf];
        const int nhome = (int)(N.lstart[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome;
        const int64_t ii = active ? i : first;
        const double xi = N.x[ii], yi = N.y[ii], zi = N.z[ii], hi = N.h[ii];
        const double hi2x4 = (RK * hi) * (RK * hi);
        const Node home = N.nodes[leaf];
        auto test = [&bx, &home, mode](const Node &nd) {
            const double hh = mode == 0 ? home.hmax : fmax(home.hmax, nd.hmax);
            const double R = RK * hh * (1.0 + 1e-10);
            return box_gap2(home, nd, bx) < R * R;
        };
        const WalkResult wr = walk(T, N.nodes, test, wb, spare);
        if (wr.lev) overflows++;
        // two sweeps in pass 2: count this lane's hits, then write them
        int64_t mine = 0, base = 0;
        for (int sweep = 0; sweep < (pass == 1 ? 1 : 2); sweep++) {
            int64_t k = 0;
            auto group = [&](const uint32_t *leaves, int count) {
                for (int g = 0; g < count; g++) {
                    const int64_t c = leaves[g];
                    const Node cand = N.nodes[c];
                    const Shift sh = leaf_shift(
                        home, cand, bx, RK * (mode == 0 ? home.hmax : fmax(home.hmax, cand.hmax)));
                    const int64_t j0 = N.lstart[c];
                    const int jn = (int)(N.lstart[c + 1] - j0);
#pragma unroll
                    for (int t = 0; t < PER; t++) {
                        const int jj = q + LPP * t;
                        if (jj >= jn) continue;
                        const int64_t j = j0 + jj;
                        double dx = xi - N.x[j], dy = yi - N.y[j], dz = zi - N.z[j];
                        if (sh.per_pair) {
                            dx = min_image(dx, bx.len[0], bx.half[0]);
                            dy = min_image(dy, bx.len[1], bx.half[1]);
                            dz = min_image(dz, bx.len[2], bx.half[2]);
                        } else {
                            dx += sh.s[0];
                            dy += sh.s[1];
                            dz += sh.s[2];
                        }
                        const double r2 = exact_r2(dx, dy, dz);
                        bool in = r2 < hi2x4;
                        if (mode == 1) {
                            const double hj = N.h[j];
                            in = in || r2 < (RK * hj) * (RK * hj);
                        }
                        if (in && j != i && active) {
                            if (sweep == 1) {
                                const int64_t pos = base + k;
                                if (pos < N.cap) N.idx[pos] = (int32_t)N.id[j];
                            }
                            k++;
                        }
                    }
                }
            };
            for_each_leaf_group<kWave>(T, N.nodes, wr, test, wb, group);
            if (sweep == 0) {
                mine = k;
                // exclusive prefix over the LPP lanes of this particle
                int64_t incl = mine;
#pragma unroll
                for (int o = 1; o < LPP; o <<= 1) {
                    int64_t v = (int64_t)__shfl_up((long long)incl, o, LPP);
                    if (q >= o) incl += v;
                }
                const int64_t total = (int64_t)__shfl((long long)incl, (p * LPP) + LPP - 1);
                if (pass == 1) {
                    if (active && q == 0) N.counts[i] = total;
                } else {
                    base = active ? N.offsets[N.id[i]] + (incl - mine) : 0;
                }
            }
        }
    });
    if (lane == 0 && overflows) atomicAdd(&N.status[4], (int)overflows);
}

// ---------------------------------------------------------------------------
// Meshless finite-volume geometry (section 2.2): for each particle, over its
// neighbours j with r_ij < R h_i (h solved on the number density), with
// d = r_j - r_i and psi_j = W(r_ij, h_i) / n_i:
//   E  = sum_j d d^T psi_j                    (EQN:MFVEMATRIX), B = E^-1
//   g  = sum_j (f_j - f_i) d psi_j,  grad f = B g   (EQN:MFVGRADIENT with
//        EQN:MFVPSI: B is constant over the sum and comes out of it)
//   gs = sum_j (f_j - f_i) grad_i W(r_ij, h_i), the SPH gradient n_i^-1 gs
//        used when cond(E) = |E|_F |B|_F / 3 exceeds 100.
// One wave per home leaf, LPP lanes per particle taking every LPP-th slot
// of each candidate leaf, sums reduced over the particle's lanes.  The
// candidate leaves are staged in LDS 64 slots at a time (positions, fields,
// per-leaf shift), so each candidate is loaded once per wave rather than by
// every home particle.  The sums of the SPH fallback are taken in a second
// pass over the same pairs, only in waves where some particle's E is
// ill-conditioned (rare), so the first pass holds fewer live sums.  Measured
// on the C1 geometry call: 15.0 ms for one pass from global memory
// (unbounded, 2 waves per SIMD), 13.1 ms with the two passes at 4 waves,
// 10.6 ms staged (11.5 ms staged at 3 waves).
// ---------------------------------------------------------------------------

template <int G, int K>
__global__ __launch_bounds__(kWave, 4) void k_mfv(MfvArgs M)
{
    constexpr double RK = Kern<K>::R;
    constexpr int LPP = kWave / G;
    // candidates staged in LDS one slot per lane (MNL leaves at a time): each
    // is loaded once per wave instead of once per home particle
    constexpr int MS = kWave, MNL = MS / G;
    __shared__ WalkBuf wb;
    __shared__ uint32_t spare[kFront];
    __shared__ TreeInfo T;
    __shared__ double st_x[MS], st_y[MS], st_z[MS], st_f[kMfvFields][MS];
    __shared__ double st_s[MNL][3];
    __shared__ int32_t st_pp[MNL], st_jn[MNL];
    load_tree(M.tree, T);
    const int lane = threadIdx.x;
    const int p = lane / LPP, q = lane % LPP;
    const Box &bx = M.box;
    const int nf = M.nf;
    int64_t overflows = 0;
    for_each_home_leaf(T.cnt[0], M.work, 1, [&](int64_t leaf) {
        const int64_t first = M.lstart[leaf];
        const int nhome = (int)(M.lstart[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome;
        const int64_t ii = active ? i : first;
        const double xi = M.x[ii], yi = M.y[ii], zi = M.z[ii], hi = M.h[ii];
        const double hinv = 1.0 / hi, ninv = 1.0 / M.ndens[ii];
        const double hi2x4 = (RK * hi) * (RK * hi);
        const double wf = Kern<K>::sigma * hinv * hinv * hinv;
        double fi[kMfvFields];
#pragma unroll
        for (int k = 0; k < kMfvFields; k++) fi[k] = k < nf ? M.f[k][ii] : 0.0;
        const Node home = M.nodes[leaf];
        auto test = [&bx, &home](const Node &nd) {
            const double R = RK * home.hmax * (1.0 + 1e-10);
            return box_gap2(home, nd, bx) < R * R;
        };
        const WalkResult wr = walk(T, M.nodes, test, wb, spare);
        if (wr.lev) overflows++;
        // The pairs (i, j) with 0 < r_ij < R h_i, candidate leaf by candidate
        // leaf, each leaf's slots q, q + LPP, ... on lane q of the particle:
        // fn(d, psi, gw, s) with d = r_j - r_i, psi = psi_j(r_i),
        // gw = -(dW/dr) / r (grad_i W = gw d) and s the staged slot of j.
        // Every use visits them in the same order.
        auto for_pairs = [&](auto fn) {
            auto group = [&](const uint32_t *leaves, int count) {
                {
                    const int k = lane / G, slot = lane % G;
                    if (k < count) {
                        const uint32_t c = leaves[k];
                        const int64_t j0 = M.lstart[c];
                        const int jn = (int)(M.lstart[c + 1] - j0);
                        if (slot < jn) {
                            const int64_t j = j0 + slot;
                            st_x[lane] = M.x[j];
                            st_y[lane] = M.y[j];
                            st_z[lane] = M.z[j];
#pragma unroll
                            for (int f = 0; f < kMfvFields; f++)
                                if (f < nf) st_f[f][lane] = M.f[f][j];
                        }
                        if (slot == 0) {
                            const Shift sh = leaf_shift(home, M.nodes[c], bx, RK * home.hmax);
                            for (int a = 0; a < 3; a++) st_s[k][a] = sh.s[a];
                            st_pp[k] = sh.per_pair ? 1 : 0;
                            st_jn[k] = jn;
                        }
                    }
                }
                wave_lds_sync();
#pragma unroll 1
                for (int t = 0; t < MS / LPP; t++) {
                    const int s = q + LPP * t;
                    const int k = s / G;
                    if (k >= count || s % G >= st_jn[k]) continue;
                    double dx = xi - st_x[s], dy = yi - st_y[s], dz = zi - st_z[s];
                    if (st_pp[k]) {
                        dx = min_image(dx, bx.len[0], bx.half[0]);
                        dy = min_image(dy, bx.len[1], bx.half[1]);
                        dz = min_image(dz, bx.len[2], bx.half[2]);
                    } else {
                        dx += st_s[k][0];
                        dy += st_s[k][1];
                        dz += st_s[k][2];
                    }
                    const double r2 = exact_r2(dx, dy, dz);
                    if (!(active && r2 < hi2x4 && r2 > 0.0)) continue;
                    const double d[3] = {-dx, -dy, -dz};   // r_j - r_i
                    const double r = sqrt(r2);
                    double fk, dfk;
                    kern<K>(r * hinv, fk, dfk);
                    const double psi = wf * fk * ninv;
                    // grad_i W = dW/dr (r_i - r_j) / r = -(dW/dr / r) d
                    const double gw = -(wf * hinv * dfk) / r;
                    fn(d, psi, gw, s);
                }
                wave_lds_sync();   // the slots are restaged for the next group
            };
            for_each_leaf_group<MNL>(T, M.nodes, wr, test, wb, group);
        };
        // first pass: E and the least-squares sums
        double E[6] = {0, 0, 0, 0, 0, 0};
        double g[3 * kMfvFields];
#pragma unroll
        for (int k = 0; k < 3 * kMfvFields; k++) g[k] = 0.0;
        for_pairs([&](const double *d, double psi, double gw, int sl) {
            E[0] += d[0] * d[0] * psi;
            E[1] += d[0] * d[1] * psi;
            E[2] += d[0] * d[2] * psi;
            E[3] += d[1] * d[1] * psi;
            E[4] += d[1] * d[2] * psi;
            E[5] += d[2] * d[2] * psi;
#pragma unroll
            for (int k = 0; k < kMfvFields; k++) {
                if (k >= nf) break;
                const double df = st_f[k][sl] - fi[k];
#pragma unroll
                for (int a = 0; a < 3; a++) g[3 * k + a] += df * d[a] * psi;
            }
        });
#pragma unroll
        for (int k = 0; k < 6; k++) E[k] = group_sum<LPP>(E[k]);
#pragma unroll
        for (int k = 0; k < 3 * kMfvFields; k++) g[k] = group_sum<LPP>(g[k]);
        // B = E^-1 of the symmetric E by cofactors, and the condition number
        const double c00 = E[3] * E[5] - E[4] * E[4];
        const double c01 = E[2] * E[4] - E[1] * E[5];
        const double c02 = E[1] * E[4] - E[2] * E[3];
        const double c11 = E[0] * E[5] - E[2] * E[2];
        const double c12 = E[1] * E[2] - E[0] * E[4];
        const double c22 = E[0] * E[3] - E[1] * E[1];
        const double det = E[0] * c00 + E[1] * c01 + E[2] * c02;
        const double id = 1.0 / det;
        const double B[6] = {c00 * id, c01 * id, c02 * id, c11 * id, c12 * id, c22 * id};
        auto frob2 = [](const double *s) {
            return (s[0] * s[0] + s[3] * s[3] + s[5] * s[5]) +
                   2.0 * (s[1] * s[1] + s[2] * s[2] + s[4] * s[4]);
        };
        const bool inv_ok = det != 0.0 && isfinite(det);
        const double cn = inv_ok ? sqrt(frob2(E)) * sqrt(frob2(B)) / 3.0 : INFINITY;
        const bool sph = !(cn <= 100.0);
        // second pass, only in a wave where some particle's E is ill-conditioned
        // (rare): the sums of the SPH estimate, in the order of the first pass
        double gs[3 * kMfvFields];
#pragma unroll
        for (int k = 0; k < 3 * kMfvFields; k++) gs[k] = 0.0;
        if (__ballot(active && sph) != 0ull) {
            for_pairs([&](const double *d, double psi, double gw, int sl) {
#pragma unroll
                for (int k = 0; k < kMfvFields; k++) {
                    if (k >= nf) break;
                    const double df = st_f[k][sl] - fi[k];
#pragma unroll
                    for (int a = 0; a < 3; a++) gs[3 * k + a] += df * gw * d[a];
                }
            });
#pragma unroll
            for (int k = 0; k < 3 * kMfvFields; k++) gs[k] = group_sum<LPP>(gs[k]);
        }
        if (active && q == 0) {
#pragma unroll
            for (int k = 0; k < 6; k++)
                if (M.B[k]) M.B[k][i] = inv_ok ? B[k] : NAN;
            if (M.cond) M.cond[i] = cn;
            for (int k = 0; k < nf; k++) {
                const double *gk = g + 3 * k;
                double out[3];
                if (!sph) {
                    out[0] = B[0] * gk[0] + B[1] * gk[1] + B[2] * gk[2];
                    out[1] = B[1] * gk[0] + B[3] * gk[1] + B[4] * gk[2];
                    out[2] = B[2] * gk[0] + B[4] * gk[1] + B[5] * gk[2];
                } else {
                    for (int a = 0; a < 3; a++) out[a] = gs[3 * k + a] * ninv;
                }
                for (int a = 0; a < 3; a++)
                    if (M.grad[3 * k + a]) M.grad[3 * k + a][i] = out[a];
            }
        }
    });
    if (lane == 0 && overflows) atomicAdd(&M.status[4], (int)overflows);
}

} // namespace

// ---------------------------------------------------------------------------
// Launches (instantiated per smoothing kernel by pairs_m4.hip and
// pairs_quintic.hip)
// ---------------------------------------------------------------------------
template <int K>
void launch_density(hipStream_t st, int G, int prec, unsigned grid, const Batch<DensArgs> &B)
{
    auto go = [&](auto g) {
        constexpr int GG = decltype(g)::value;
        if (prec == SPH_FP32_PAIR)
            hipLaunchKernelGGL((k_density<GG, SPH_FP32_PAIR, K>), dim3(grid), dim3(kWave), 0, st, B);
        else
            hipLaunchKernelGGL((k_density<GG, SPH_FP64, K>), dim3(grid), dim3(kWave), 0, st, B);
    };
    switch (G) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 32: go(std::integral_constant<int, 32>{}); break;
    default: go(std::integral_constant<int, 16>{}); break;
    }
}

template <int K>
void launch_forces(hipStream_t st, int G, int prec, bool ac, bool sw, unsigned grid,
                   const Batch<ForceArgs> &B)
{
    auto go = [&](auto g) {
        constexpr int GG = decltype(g)::value;
        auto variant = [&](auto pr, auto with_ac, auto with_sw) {
            hipLaunchKernelGGL((k_forces<GG, decltype(pr)::value, decltype(with_ac)::value,
                                         decltype(with_sw)::value, K>),
                               dim3(grid), dim3(kWave), 0, st, B);
        };
        using F32 = std::integral_constant<int, SPH_FP32_PAIR>;
        using F64 = std::integral_constant<int, SPH_FP64>;
        using T = std::true_type;
        using N = std::false_type;
        if (prec == SPH_FP32_PAIR) {
            if (sw) { if (ac) variant(F32{}, T{}, T{}); else variant(F32{}, N{}, T{}); }
            else if (ac) variant(F32{}, T{}, N{});
            else variant(F32{}, N{}, N{});
        } else {
            if (sw) { if (ac) variant(F64{}, T{}, T{}); else variant(F64{}, N{}, T{}); }
            else if (ac) variant(F64{}, T{}, N{});
            else variant(F64{}, N{}, N{});
        }
    };
    switch (G) {
    case 8: go(std::integral_constant<int, 8>{}); break;
    case 32: go(std::integral_constant<int, 32>{}); break;
    default: go(std::integral_constant<int, 16>{}); break;
    }
}

template <int K>
void launch_neighbours(hipStream_t st, int G, unsigned grid, const NgbArgs &a, int pass)
{
    switch (G) {
    case 8: hipLaunchKernelGGL((k_neighbours<8, K>), dim3(grid), dim3(kWave), 0, st, a, pass); break;
    case 32: hipLaunchKernelGGL((k_neighbours<32, K>), dim3(grid), dim3(kWave), 0, st, a, pass); break;
    default: hipLaunchKernelGGL((k_neighbours<16, K>), dim3(grid), dim3(kWave), 0, st, a, pass); break;
    }
}

template <int K>
void launch_mfv(hipStream_t st, int G, unsigned grid, const MfvArgs &a)
{
    switch (G) {
    case 8: hipLaunchKernelGGL((k_mfv<8, K>), dim3(grid), dim3(kWave), 0, st, a); break;
    case 32: hipLaunchKernelGGL((k_mfv<32, K>), dim3(grid), dim3(kWave), 0, st, a); break;
    default: hipLaunchKernelGGL((k_mfv<16, K>), dim3(grid), dim3(kWave), 0, st, a); break;
    }
}

} // namespace sph
