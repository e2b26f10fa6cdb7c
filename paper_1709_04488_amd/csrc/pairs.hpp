// Pair loops: density + Newton-Raphson h solve, hydro forces, neighbour
// export, MFV geometry.
//
// Work decomposition (the GPU analogue of the paper's per-leaf-cell neighbour
// gathering, section 4.2, with a leaf as the unit of work as in its OpenMP
// loop, section 5.2.1): one wavefront per home leaf of at most G sorted
// particles, or per share of one in small sets, its lanes divided among the home
// particles.  The wave walks the box tree to collect the leaves that can hold
// neighbours of its particles into an LDS list.  Candidate leaves are then handled
// in groups of up to 64, one per lane:
//   open  -- each lane's leaf, its particle count and its periodic shift go to a
//            table in LDS;
//   find  -- FP64 density (and small FP32-pair boxes, where images are ambiguous):
//            each home particle in turn against a candidate per lane, ballots rank
//            the hits and their r^2 goes to the particle's list in global scratch;
//            forces and FP32-pair density: matrix products
//            of candidates and home particles, whose signs are the hits, as a list
//            of candidate slots per home particle in LDS;
//   use   -- each particle's lanes share its list: pair terms, or r^2 to the
//            density loop's scratch lists, which every Newton step then reads.
// The expensive pair terms run only for hits, with the lanes compacted.  Each
// output is accumulated by its own lanes in a fixed order, so results are
// deterministic and need no atomics.  The neighbour export and the MFV geometry
// still stage candidates in LDS and test them lane by lane (for_each_leaf_group).
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
template <class T>
__device__ inline __attribute__((address_space(1))) T *as_global_out(T *p)
{
    return (__attribute__((address_space(1))) T *)p;
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

// Lanes may then read what other lanes of the wave stored to global memory.
__device__ inline void wave_mem_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
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

// Reductions over groups of `lanes` lanes (a power of two of at least K,
// wave-uniform).
template <int K, class T>
__device__ inline T lanes_sum(T v, int lanes)
{
    v = group_sum<K>(v);
    for (int o = K; o < lanes; o <<= 1) v += __shfl_xor(v, o);
    return v;
}
template <int K>
__device__ inline double lanes_max(double v, int lanes)
{
    v = group_max<K>(v);
    for (int o = K; o < lanes; o <<= 1) v = fmax(v, __shfl_xor(v, o));
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

template <int K>
__device__ inline int lanes_max_int(int v, int lanes)
{
    v = group_max_int<K>(v);
    for (int o = K; o < lanes; o <<= 1) {
        const int w = __shfl_xor(v, o);
        v = w > v ? w : v;
    }
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
    // small sets: the first claims take everything, and no block asks the
    // counters (1,000 particles as 1,008 waves: 54 -> 36 us of the force loop)
    const bool all_static = (int64_t)nstatic * claim >= per;
    for (int r = 0; r < kXcds; r++) {
        const int x = (x0 + r) % kXcds;
        const int64_t beg = x * per;
        const int64_t end = beg + per < L ? beg + per : L;
        if (beg >= end) continue;
        bool got = false;
        for (int k = 0;; k++) {
            uint32_t c = rank;
            if (r > 0 || k > 0 || rank >= nstatic) {   // (a grid not a multiple of 8)
                if (all_static) return;
                if (lane == 0) c = nstatic + atomicAdd(&work[x * kWorkStride], 1u);
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

// Visit the candidate leaves in groups of at most NL: fn(leaves, count) with a
// wave-uniform count.  After a truncated walk the leaves under each returned node
// are tested 64 at a time and the passing ones grouped.
template <int NL, class Test, class Fn>
__device__ int64_t for_each_leaf_group(const TreeInfo &T, const Node *nodes, const WalkResult &wr,
                                       Test test, WalkBuf &wb, Fn fn)
{
    if (wr.lev == 0) {
        for (int t0 = 0; t0 < wr.n; t0 += NL) fn(wr.list + t0, wr.n - t0 < NL ? wr.n - t0 : NL);
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
            for (int t0 = 0; t0 < cnt; t0 += NL) fn(wb.tmp + t0, cnt - t0 < NL ? cnt - t0 : NL);
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
// it evaluates pair terms.  Candidate leaves come in groups of at most 64, one
// per lane, which set up a table in LDS (first particle, particle count,
// periodic shift).
//
// The pairs are found by the matrix cores.  In coordinates from the home
// leaf's centre, in units of the reach,
//   r_ij^2 - T_i^2 = (x_j, y_j, z_j, |x_j|^2) . (-2x_i, -2y_i, -2z_i, 1) + |x_i|^2 - T_i^2,
// a product of inner length 4: with one candidate per lane as four halves, a
// 16x16x16 product takes 16 candidates against 16 home particles (its other
// three groups of four inner indices hold the candidates of the other lanes,
// which zeros in the second operand leave out, so a row of 64 candidates needs
// no data movement at all), and the sign bit of each result is a hit.  A lane's
// bits are those of one home particle; they go to LDS as that particle's list
// of candidate slots.  The thresholds are widened by the rounding of the
// halves, so the lists hold every pair within reach and about 1 % more; the
// lists' readers form r^2 exactly and decide.
//
// Measured on 2.1M particles (C1, FP64, G = 16: 92 candidate leaves and 1,370
// listed pairs per home leaf): testing each candidate against each home
// particle near its leaf with vector instructions took about 60 % of both
// loops' time, 4,000 vector and 4,500 scalar instructions per home leaf; this
// takes about 1,700 vector instructions and 92 matrix instructions.
constexpr int kGroup = kWave;       // candidate leaves per group

// How the separations of a group see the periodic box: no shift at all, one
// shift per leaf, or the minimum image pair by pair (boxes so small that a
// leaf's shift is ambiguous).  A pair closer than the reach has the same
// image under the last two, and the one nearest to the home leaf's centre,
// unless the reach and the home leaf span half the box (kImgWide).
enum : int { kImgNone = 0, kImgShift = 1, kImgPair = 2, kImgWide = 3 };

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

// Per leaf of the group: first particle (j0), particle count (low 8 bits of
// meta) and, in FP64, the shift added to x_i - x_j (two bits per axis from bit 8
// on: 1 a box length, 2 minus that); FP32-pair: the distance of the leaf centres
// with the shift.
template <int PREC>
struct LeafTab {
    uint2 jm[kGroup];
    float o[3][PREC == SPH_FP32_PAIR ? kGroup : 1];
};
__device__ inline double shift_of(uint32_t meta, int axis, const Box &bx)
{
    const uint32_t code = (meta >> (8 + 2 * axis)) & 3u;
    return code == 0 ? 0.0 : (code == 1 ? bx.len[axis] : -bx.len[axis]);
}

__device__ inline double readlane_d(double v, int l)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Number of set bits of a ballot below this lane.
__device__ inline uint32_t rank_of(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Above this many candidate leaves (an ordinary home leaf has 50-110) the home
// leaf's box is wide against its particles' reaches -- the outermost leaves of a
// condensed set see every leaf of it -- and the walk is repeated with a test of
// each node against every home particle.  Plummer sphere of 100,003 particles:
// 1 % of the home leaves had 2,000 to 6,400 candidate leaves, and the launch
// lasted as long as they did.
constexpr int kManyLeaves = 160;

// A home leaf with more candidate leaves than this after the second walk is left to
// the launch after this one, where a wave has one of its particles: each of them has
// thousands of neighbours, and one wave with all 16 lasted as long as everything
// else.  Plummer spheres: 78,446 particles FP32-pair with the quintic kernel 25.7 ->
// 9.0 ms, 30,000 FP64 1.78 -> 1.10 ms; the launch without such a leaf costs each
// loop 3-5 us.  From 256 leaves on the force loop of the first took 2.6 instead of
// 1.3 ms (too many leaves for that many waves each), from 768 the density loops 3
// and 15 % more.  The h solve leaves a leaf at whichever pass its reaches have grown
// so far, and the next launch begins it anew; and however many leaves it leaves,
// their particles have a wave each: guesses of h three times too large make all
// leaves of 150,000 particles heavy (FP64 70 ms when leaves without end shared the
// waves of small sets' rule, one particle per wave 15 ms, no second launch 55),
// guesses of a tenth to five times 60,000 with five far away (FP32-pair 125, 24, 63).
constexpr int kHeavyLeaves = 384;
template <class Args>
__device__ inline bool left_over(const Args &A, int split, const WalkResult &wr, int64_t leaf)
{
    if (!A.heavy || split > 0 || (wr.lev == 0 && wr.n <= kHeavyLeaves)) return false;
    if ((threadIdx.x & (kWave - 1)) == 0) A.heavy[atomicAdd(A.heavy_count, 1u)] = (uint32_t)leaf;
    wave_lds_sync();   // the home table is rewritten for the next leaf
    return true;
}

// Whether a node's box is within reach of some home particle that takes part (a
// bit of `part`): its own squared reach in H or lim2, whichever is larger.  The
// relative slack covers the rounding of the differently formed distances
// (FP32-pair separations carry single-precision error).
template <int G, int PREC>
__device__ inline bool node_in_reach(const HomeTab<G, PREC> &H, uint64_t part, const Node &nd, const Box &bx,
                                     double lim2)
{
    constexpr double slack = PREC == SPH_FP64 ? 1.0 + 1e-6 : 1.0 + 1e-4;
    bool any = false;
    for (; part; part &= part - 1) {
        const HomeRow h = H.d[__builtin_ctzll(part)];
        const double c[3] = {h.x, h.y, h.z};
        double d2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            double d = fabs(c[a] - nd.c[a]);
            if (bx.periodic) d = fmin(d, fabs(bx.len[a] - d));
            const double g = fmax(d - nd.e[a], 0.0);
            d2 += g * g;
        }
        any = any || d2 <= fmax(h.thr, lim2) * slack;
    }
    return any;
}

// The lanes' flags (the same on all of a particle's `lpp` lanes) as a bit per
// particle.
__device__ inline uint64_t particle_bits(bool flag, int lpp)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int src = lane * lpp;
    return __ballot(__shfl(flag ? 1 : 0, src & (kWave - 1)) != 0 && src < kWave);
}

// The next group of at most `depth` candidate leaves of a walk's result
// (0: none left): a slice of the list, or, where the walk was truncated, the
// leaves under the listed nodes that pass the test, up to 64 of them collected
// in wb.tmp.
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
    int have = 0;
    wave_lds_sync();   // the last group's readers of wb.tmp
    while (pos < total) {
        const int64_t t = pos + lane;
        const int64_t c = t < total ? ((int64_t)wr.list[t >> sh] << sh) + (t & ((1ll << sh) - 1)) : L;
        const bool pass = c < L && test(load_global(nodes + c));
        const uint64_t mask = __ballot(pass);
        const int n = (int)__popcll(mask);
        if (have + n > kGroup) break;   // the next group starts with these
        if (pass) wb.tmp[have + rank_of(mask)] = (uint32_t)c;
        have += n;
        pos += kWave;
    }
    wave_lds_sync();
    leaves = wb.tmp;
    return have;
}

// Rows of 64 candidates whose bits a word holds, candidate slots per word, and
// the places of a home particle's list (at least a word's slots).
template <int G>
struct Words {
    static constexpr int rows = G == 32 ? 1 : 2;
    static constexpr int slots = rows * kWave;
    static constexpr int cap = G == 32 ? 64 : 128;
    static constexpr int tiles = (G + 15) / 16;   // of 16 home particles
    static_assert(cap >= slots, "a list takes a word's hits");
};

// Leaves per group of a list of n: groups of equal size (whole words, so the
// words hold the same candidates whatever the size), at most `most`.
template <int G>
__device__ inline int group_depth(int n, int most)
{
    constexpr int LPW = Words<G>::slots / G;
    const int groups = (n + most - 1) / most;
    const int d = groups > 0 ? (n + groups - 1) / groups : most;
    const int r = (d + LPW - 1) / LPW * LPW;
    return r < most ? r : most;
}

// Set up a group (lane l: leaf leaves[l]).  hcov < 0: symmetric force criterion
// (reach R max(h) over both leaves).  Returns how separations see the box.
// near (when not null): per home particle that takes part (a bit of takes_part),
// the leaves whose box is within its reach.
template <int G, int PREC, int K>
__device__ inline int open_group(const uint32_t *leaves, int count, const uint32_t *__restrict__ lstart,
                                 const Node *__restrict__ nodes, const Node &home, const Box &bx,
                                 double hcov, LeafTab<PREC> &tab, const HomeTab<G, PREC> &H,
                                 uint64_t takes_part, uint64_t *near)
{
    constexpr double RK = Kern<K>::R;
    const int lane = threadIdx.x & (kWave - 1);
    bool per_pair = false, shifted = false, spans = false;
    uint2 jm{0u, 0u};
    // the leaf's box as the home particles see it (a missing one is far away,
    // one with pair-by-pair images is near to all)
    double c[3] = {1e150, 0.0, 0.0}, e[3] = {0.0, 0.0, 0.0};
    if (lane < count) {
        const uint32_t leaf = leaves[lane];
        const uint32_t j0 = as_global(lstart)[leaf];
        jm.x = j0;
        jm.y = as_global(lstart)[leaf + 1] - j0;
        const Node cand = load_global(nodes + leaf);
        const double reach = RK * (hcov < 0.0 ? fmax(home.hmax, cand.hmax) : hcov);
        const Shift sh = leaf_shift(home, cand, bx, reach);
        per_pair = sh.per_pair;
#pragma unroll
        for (int a = 0; a < 3; a++) {
            shifted = shifted || sh.s[a] != 0.0;
            if (per_pair) spans = spans || !(reach + home.e[a] < 0.49 * bx.len[a]);
            if constexpr (PREC == SPH_FP64)
                jm.y |= (sh.s[a] > 0.0 ? 1u : (sh.s[a] < 0.0 ? 2u : 0u)) << (8 + 2 * a);
            else
                tab.o[a][lane] = (float)((home.c[a] - cand.c[a]) + (per_pair ? 0.0 : sh.s[a]));
            c[a] = cand.c[a] - sh.s[a];
            // (the slack is far above the rounding of the distances)
            e[a] = per_pair ? INFINITY : cand.e[a] + 1e-6 * reach;
        }
    }
    tab.jm[lane] = jm;
    const int img = __ballot(spans) ? kImgWide
                    : __ballot(per_pair) ? kImgPair
                                         : (__ballot(shifted) ? kImgShift : kImgNone);
    if (near) {
#pragma unroll
        for (int p = 0; p < G; p++) {
            uint64_t m = 0;
            if ((takes_part >> p) & 1) {
                const HomeRow h = H.d[p];
                const double dx = fmax(fabs(h.x - c[0]) - e[0], 0.0);
                const double dy = fmax(fabs(h.y - c[1]) - e[1], 0.0);
                const double dz = fmax(fabs(h.z - c[2]) - e[2], 0.0);
                m = __ballot((dx * dx + dy * dy) + dz * dz <= h.thr);
            }
            near[p] = m;   // (every lane stores the same value)
        }
    }
    wave_lds_sync();
    return img;
}

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

// r^2 of home particle (hx, hy, hz) and candidate j of leaf k of the open
// group, and the separation; w: what the candidate's position record carries
// besides.
template <int PREC, class T>
__device__ inline T group_separation(const LeafTab<PREC> &tab, int img, const Box &bx, T hx, T hy, T hz,
                                     int k, uint2 jm, uint32_t j, const Pos4 *__restrict__ pos,
                                     const Off4 *__restrict__ off, T &dx, T &dy, T &dz, T &w)
{
    if constexpr (PREC == SPH_FP64) {
        const auto *o = as_global((const double *)(pos + j));
        const double x = o[0], y = o[1], z = o[2];
        w = o[3];
        if (img == kImgNone)
            return separation<PREC, kImgNone, T>(bx, hx, hy, hz, x, y, z, 0.0, 0.0, 0.0, dx, dy, dz);
        if (img == kImgShift)
            return separation<PREC, kImgShift, T>(bx, hx, hy, hz, x, y, z, shift_of(jm.y, 0, bx),
                                                  shift_of(jm.y, 1, bx), shift_of(jm.y, 2, bx), dx, dy, dz);
        return separation<PREC, kImgPair, T>(bx, hx, hy, hz, x, y, z, 0.0, 0.0, 0.0, dx, dy, dz);
    } else {
        const auto *o = as_global((const float *)(off + j));
        const float x = o[0], y = o[1], z = o[2];
        w = o[3];
        if (img < kImgPair)
            return separation<PREC, kImgNone, T>(bx, hx, hy, hz, x, y, z, tab.o[0][k], tab.o[1][k], tab.o[2][k],
                                                 dx, dy, dz);
        return separation<PREC, kImgPair, T>(bx, hx, hy, hz, x, y, z, tab.o[0][k], tab.o[1][k], tab.o[2][k], dx,
                                             dy, dz);
    }
}

// The density loop in FP64 tests candidates lane by lane (in FP32-pair mode some
// groups, lanewise_density): a lane holds a
// candidate of each of kRows rows of 64 slots (slot s = particle s % G of leaf
// s / G), the home particle is the same for all lanes, a test is ten
// instructions for 64 candidates and its result a ballot, whose bits rank the
// hits; r^2 of a hit goes straight to the home particle's list.  Rows none of
// whose leaves are near the home particle are skipped.  Measured against the
// products below (which find the pairs faster, but whose readers then have to
// fetch each candidate again): 2.1M particles, M4 2.26 against 2.30 ms, 262,144
// with the quintic kernel 0.97 against 1.39 ms.
//
// near (lane p): what is left of home particle p's near leaves in the open
// group; cnt (lane p): the hits its list holds, at most `cap`.  Returns the home
// particle whose list is full: the caller empties it, sets cnt to match and
// calls again to go on; -1 when the group is done.  What a list holds when it
// is full depends on the particle and the rows alone.
constexpr int kRows = 4;
template <int G, int PREC, int IMG, int NR, class Mass, class Put>
__device__ inline int test_rows(const LeafTab<PREC> &tab, const HomeTab<G, PREC> &H, int count,
                                const Box &bx, const Pos4 *__restrict__ pos, const Off4 *__restrict__ off,
                                uint64_t &near, int &cnt, int cap, Mass mass, Put put)
{
    constexpr bool F64 = PREC == SPH_FP64;
    using T = std::conditional_t<F64, double, float>;
    constexpr int LPR = kWave / G;                      // leaves per row
    constexpr uint32_t RM = (1u << LPR) - 1;            // one row's leaves
    constexpr uint32_t BM = (uint32_t)((1ull << (NR * LPR)) - 1);
    static_assert(NR * LPR <= 32, "a block's leaves fit 32 bits");
    const int lane = threadIdx.x & (kWave - 1);
    const int nrows = (count + LPR - 1) / LPR;
    for (int r0 = 0; r0 < nrows; r0 += NR) {
        // home particles with a near leaf among these rows
        const uint32_t here = (uint32_t)(near >> (r0 * LPR)) & BM;
        uint64_t todo = __ballot(here != 0);
        if (todo == 0) continue;
        T x[NR], y[NR], z[NR], ox[NR], oy[NR], oz[NR];
        double w[NR];
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const int s = (r0 + r) * kWave + lane;
            const int slot = s % G;
            const uint2 jm = tab.jm[s / G];
            const bool ok = slot < (int)(jm.y & 255u);
            const uint32_t j = jm.x + (ok ? slot : 0);   // (a missing leaf's entry is particle 0)
            const auto *q = as_global(F64 ? (const T *)(pos + j) : (const T *)(off + j));
            x[r] = ok ? q[0] : (T)INFINITY;   // an empty slot is far away
            y[r] = q[1];
            z[r] = q[2];
            w[r] = mass(j);
            if constexpr (!F64) {
                ox[r] = tab.o[0][s / G];
                oy[r] = tab.o[1][s / G];
                oz[r] = tab.o[2][s / G];
            } else if constexpr (IMG == kImgShift) {
                ox[r] = shift_of(jm.y, 0, bx);
                oy[r] = shift_of(jm.y, 1, bx);
                oz[r] = shift_of(jm.y, 2, bx);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        do {
            const int p = (int)__builtin_ctzll(todo);
            todo &= todo - 1;
            T hx, hy, hz, thr;
            if constexpr (F64) {
                const HomeRow h = H.d[p];
                hx = h.x;
                hy = h.y;
                hz = h.z;
                thr = h.thr;
            } else {
                const HomeRowF h = H.f[p];
                hx = h.x;
                hy = h.y;
                hz = h.z;
                thr = (float)H.d[p].thr;
            }
            const uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)here, p);
            int have = __builtin_amdgcn_readlane(cnt, p);
            int full = -1;
#pragma unroll
            for (int r = 0; r < NR; r++) {
                if (!((bits >> (r * LPR)) & RM)) continue;
                T dx, dy, dz;
                const T r2 = separation<PREC, IMG, T>(bx, hx, hy, hz, x[r], y[r], z[r], ox[r], oy[r], oz[r], dx, dy,
                                                      dz);
                const uint64_t m = __ballot(r2 < thr);
                const int to = have + (int)__popcll(m);
                if (to > cap) {
                    full = r;
                    goto filled;
                }
                if (__builtin_amdgcn_inverse_ballot_w64(m)) put((uint32_t)(p * cap + have) + rank_of(m), r2, w[r]);
                have = to;
            }
        filled:
            cnt = lane == p ? have : cnt;
            if (full >= 0) {
                // what is done leaves the masks: these rows of the particles
                // before p, and of p the rows before the full one
                const uint32_t mine = lane < p ? BM : (lane == p ? (1u << (full * LPR)) - 1u : 0u);
                near &= ~((uint64_t)mine << (r0 * LPR));
                return p;
            }
        } while (todo);
        // these rows are done for every home particle
        near &= ~((uint64_t)BM << (r0 * LPR));
    }
    return -1;
}

using Half2 = _Float16 __attribute__((ext_vector_type(2)));
using Half4 = _Float16 __attribute__((ext_vector_type(4)));
using Float4 = float __attribute__((ext_vector_type(4)));

// Rounded towards zero.
__device__ inline Half2 to_halves(float a, float b)
{
    return __builtin_bit_cast(Half2, __builtin_amdgcn_cvt_pkrtz(a, b));
}

// What the halves leave open.  A coordinate X rounds by at most 2^-10 |X| (or
// 2^-14 where it has no normal half), so two points at distance r <= T of each
// other and |X_i| <= H of the home centre come out at most 2^-10 (2 H + T) +
// 2^-12 further apart; |x_j|^2 rounds downwards, which only adds hits; the sums
// are single precision, each wrong by up to a unit in the last place, which counts
// where H is a hundred times T.  kHalfRel and kHalfAbs hold these with a third to
// spare.  Beyond kHalfFar reaches nothing is tested: every candidate is listed.
constexpr float kHalfRel = 1.4e-3f, kHalfAbs = 4e-4f, kHalfFar = 150.f, kHalfTop = 65504.f;

// The home leaf as the product's second operand, per home particle: (-2 x_i, 1)
// as halves and the constants |x_i|^2 - T_i^2 and |x_i|^2 (1e30: takes no part).
// It stays in LDS: held in registers it displaced what the pair terms need.
struct alignas(16) HomeCol {
    Half4 b;
    float c, n;
};
template <int G>
struct HomeOp {
    HomeCol col[16 * Words<G>::tiles];
};
template <>
struct HomeOp<0> {};   // (not used)

// Units of the product's coordinates: 1 / unit length, the largest |x_i| (in
// units), and whether every candidate is listed.  Lengths are brought to these
// units in double precision: in single precision the square of a length leaves the
// range at some 1e-20 and 1e19 of the caller's units (and the force loop of
// 2,097,152 particles in FP64 took 1.68 ms; this takes 1.61).
struct HomeUnits {
    double scale;
    float extent;
    bool wide;
};

// thr: the home particles' squared reaches in H (< 0: takes no part), unit: the
// unit length (about the reach over R).
template <int G, int PREC>
__device__ inline HomeUnits home_operand(const HomeTab<G, PREC> &H, const Node &home, double unit, HomeOp<G> &O)
{
    const int lane = threadIdx.x & (kWave - 1);
    const double s = 1.0 / unit;
    HomeUnits U;
    U.scale = s;
    U.extent = (float)(sqrt((home.e[0] * home.e[0] + home.e[1] * home.e[1]) + home.e[2] * home.e[2]) * s);
    bool far = false;
    if (lane < 16 * Words<G>::tiles) {
        const bool in = lane < G;
        const HomeRow h = H.d[in ? lane : 0];
        const bool part = in && h.thr >= 0.0;
        float X, Y, Z;
        if constexpr (PREC == SPH_FP64) {
            X = (float)((h.x - home.c[0]) * s);
            Y = (float)((h.y - home.c[1]) * s);
            Z = (float)((h.z - home.c[2]) * s);
        } else {
            const HomeRowF f = H.f[in ? lane : 0];
            X = (float)(f.x * s);
            Y = (float)(f.y * s);
            Z = (float)(f.z * s);
        }
        const Half2 xy = to_halves(X, Y), z0 = to_halves(Z, 0.f);
        const float n = __builtin_amdgcn_fdot2(xy, xy, __builtin_amdgcn_fdot2(z0, z0, 0.f, false), false);
        const float T = __builtin_amdgcn_sqrtf((float)((h.thr * s) * s));
        const float Tw = T * (1.f + kHalfRel) + 2.f * kHalfRel * U.extent + kHalfAbs;
        far = part && !(U.extent + T <= kHalfFar);
        HomeCol c;
        c.b = part ? Half4{(_Float16)-2 * xy.x, (_Float16)-2 * xy.y, (_Float16)-2 * z0.x, (_Float16)1}
                   : Half4{0, 0, 0, 0};
        c.c = part ? n - Tw * Tw : 1e30f;
        c.n = part ? n : 1e30f;
        O.col[lane] = c;
    }
    U.wide = __ballot(far) != 0ull;
    // every candidate is a hit of the particles that take part, whatever their
    // halves came to (beyond their range, or not a number)
    if (U.wide && lane < 16 * Words<G>::tiles) {
        const float c = lane < G && H.d[lane].thr >= 0.0 ? -1.f : 1e30f;
        O.col[lane] = HomeCol{Half4{0, 0, 0, 1}, c, c};   // (empty slots still miss)
    }
    wave_lds_sync();
    return U;
}

// Sum over the four lanes l % 16, l % 16 + 16, + 32, + 48 of a lane and of
// those before it.
__device__ inline void column_scan(uint32_t v, uint32_t &before, uint32_t &total)
{
    const int row = (int)(threadIdx.x & (kWave - 1)) / 16;
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);   // rows 0 0 2 2, rows 1 1 3 3
    const uint32_t pair = a[0] + a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(pair, pair, false, false);
    before = ((row & 1) ? a[0] : 0u) + ((row & 2) ? b[0] : 0u);
    total = b[0] + b[1];
}

// The open group's pairs.  Every candidate within reach of a home particle
// (FORCE: or the home particle within its reach, which the position records
// carry squared) is listed for it: ids holds Words<G>::cap slots of the group
// per home particle, and use(n) is called with this lane's home particle's
// number n (p: that particle) whenever a list might overflow and at the
// group's end.  A list's order depends on the particle and the candidates alone.
template <int G, int PREC, bool FORCE, class Use>
__device__ inline void group_pairs(int p, const LeafTab<PREC> &tab, const Node &home, const Box &bx, int count, int img,
                                   const HomeOp<G> &op, const HomeUnits &U, const Pos4 *__restrict__ pos,
                                   const Off4 *__restrict__ off, uint16_t *ids, Use use)
{
    using W = Words<G>;
    constexpr bool F64 = PREC == SPH_FP64;
    using T = std::conditional_t<F64, double, float>;
    constexpr int NT = W::tiles;
    const int lane = threadIdx.x & (kWave - 1);
    const int words = (count * G + W::slots - 1) / W::slots;
    // the slot of this lane's candidate in row r of a word, so that a result's
    // bits, in the order t, v within a row, are consecutive slots
    const int sub = ((lane >> 2) & 3) * (16 * W::rows) + (lane >> 4) * 4 + (lane & 3);
    const bool wide = U.wide || img == kImgWide;
    const float scale = F64 ? 0.f : (float)U.scale;
    struct Raw {
        T x, y, z, w;
        uint32_t meta;
        int k;
        bool ok;
    };
    auto load = [&](int word, Raw (&c)[W::rows]) {
#pragma unroll
        for (int r = 0; r < W::rows; r++) {
            const int s = word * W::slots + r * 16 + sub;
            c[r].k = s / G;
            const uint2 jm = tab.jm[c[r].k];
            const int slot = s % G;
            c[r].ok = slot < (int)(jm.y & 255u);
            c[r].meta = jm.y;
            const uint32_t j = jm.x + (c[r].ok ? slot : 0);   // (a missing leaf's entry is particle 0)
            const auto *q = as_global(F64 ? (const T *)(pos + j) : (const T *)(off + j));
            c[r].x = q[0];
            c[r].y = q[1];
            c[r].z = q[2];
            if constexpr (FORCE) c[r].w = q[3];
        }
    };
    uint32_t held[NT] = {};
    __builtin_amdgcn_s_setprio(2);
    for (int word = 0;; word++) {
        uint32_t bits[NT] = {}, before[NT] = {}, total[NT] = {};
        bool over = false;
        if (word < words) {
            Raw raw[W::rows];
            load(word, raw);
            HomeCol col[NT];
#pragma unroll
            for (int u = 0; u < NT; u++) col[u] = op.col[lane % 16 + 16 * u];
#pragma unroll
            for (int r = 0; r < W::rows; r++) {
                float X, Y, Z;
                if constexpr (F64) {
                    double cx = home.c[0], cy = home.c[1], cz = home.c[2];
                    if (img == kImgShift) {
                        cx += shift_of(raw[r].meta, 0, bx);
                        cy += shift_of(raw[r].meta, 1, bx);
                        cz += shift_of(raw[r].meta, 2, bx);
                    }
                    double dx = raw[r].x - cx, dy = raw[r].y - cy, dz = raw[r].z - cz;
                    if (img == kImgPair) {
                        dx = min_image(dx, bx.len[0], bx.half[0]);
                        dy = min_image(dy, bx.len[1], bx.half[1]);
                        dz = min_image(dz, bx.len[2], bx.half[2]);
                    }
                    X = (float)(dx * U.scale);
                    Y = (float)(dy * U.scale);
                    Z = (float)(dz * U.scale);
                } else {
                    X = raw[r].x - tab.o[0][raw[r].k];
                    Y = raw[r].y - tab.o[1][raw[r].k];
                    Z = raw[r].z - tab.o[2][raw[r].k];
                    if (img == kImgPair) {
                        X = min_image_f(X, (float)bx.len[0], (float)bx.half[0]);
                        Y = min_image_f(Y, (float)bx.len[1], (float)bx.half[1]);
                        Z = min_image_f(Z, (float)bx.len[2], (float)bx.half[2]);
                    }
                    X *= scale;
                    Y *= scale;
                    Z *= scale;
                }
                Half2 xy = to_halves(X, Y);
                const Half2 z0 = to_halves(Z, 0.f);
                float n = __builtin_amdgcn_fdot2(xy, xy, __builtin_amdgcn_fdot2(z0, z0, 0.f, false), false);
                // an empty slot, or a candidate out of reach by far, hits nothing
                float z = Z, nf = 0.f;
                bool ok = raw[r].ok;
                if (!wide) ok = ok && n <= 4e4f;
                if constexpr (FORCE) {
                    // |x_j|^2 - T_j^2, rounded downwards; a reach beyond the halves'
                    // range takes everything
                    const float Tj = __builtin_amdgcn_sqrtf(
                        F64 ? (float)((raw[r].w * U.scale) * U.scale) : (float)((raw[r].w * scale) * scale));
                    const float Tw = Tj * (1.f + 2.f * kHalfRel) + 2.f * kHalfRel * U.extent + kHalfAbs;
                    const bool big = raw[r].ok && !(U.extent + Tw <= kHalfFar);
                    nf = n - Tw * Tw * (1.f + kHalfRel);
                    nf = ok ? nf : kHalfTop;
                    nf = big ? -kHalfTop : nf;
                    ok = ok && !big;
                }
                if (wide) {
                    n = 0.f;
                    nf = 0.f;
                    z = 0.f;
                    ok = raw[r].ok;
                    xy = Half2{0, 0};
                    if (!ok) nf = kHalfTop;
                }
                if (!ok) {
                    xy = Half2{0, 0};
                    z = 0.f;
                    n = kHalfTop;
                }
                const Half2 zn = to_halves(z, n);
                const Half4 a{xy.x, xy.y, zn.x, zn.y};
                Half4 af = a;
                if constexpr (FORCE) af.w = to_halves(nf, 0.f).x;
#pragma unroll
                for (int u = 0; u < NT; u++) {
                    const float c = wide ? (col[u].c < 1e29f ? -1.f : 1e30f) : col[u].c;
                    const float cn = wide ? c : col[u].n;
                    const Float4 C{c, c, c, c}, CN{cn, cn, cn, cn};
                    const Half4 zero{0, 0, 0, 0};
#pragma unroll
                    for (int t = 0; t < 4; t++) {
                        const Half4 b = lane / 16 == t ? col[u].b : zero;
                        const Float4 D = __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, C, 0, 0, 0);
                        Float4 E = D;
                        if constexpr (FORCE) E = __builtin_amdgcn_mfma_f32_16x16x16f16(af, b, CN, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; v++) {
                            const float d = D[v], e = E[v];
                            const uint32_t sign = __builtin_bit_cast(uint32_t, d) | __builtin_bit_cast(uint32_t, e);
                            bits[u] = __builtin_amdgcn_alignbit(bits[u], sign, 31);
                        }
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < NT; u++) {
                column_scan((uint32_t)__popc(bits[u]), before[u], total[u]);
                over = over || held[u] + total[u] > (uint32_t)W::cap;
            }
        }
        if (word == words || __ballot(over) != 0ull) {
            __builtin_amdgcn_s_setprio(0);
            wave_lds_sync();
            int n = __shfl((int)held[0], p % 16);
            if constexpr (NT == 2) {
                const int n1 = __shfl((int)held[1], p % 16);
                n = p < 16 ? n : n1;
            }
            use(n);
            wave_lds_sync();
#pragma unroll
            for (int u = 0; u < NT; u++) held[u] = 0;
            if (word == words) break;
            __builtin_amdgcn_s_setprio(2);
        }
        // this lane's hits to its home particle's list
#pragma unroll
        for (int u = 0; u < NT; u++) {
            const int i = lane % 16 + 16 * u;
            uint16_t *to = ids + (i < G ? i : 0) * W::cap + held[u] + before[u];
            const int last = word * W::slots + (lane >> 4) * (16 * W::rows) + 16 * W::rows - 1;
            for (uint32_t m = bits[u]; m; m &= m - 1) *to++ = (uint16_t)(last - __builtin_ctz(m));
            held[u] += total[u];
        }
    }
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


constexpr int log2_of(int v) { return v > 1 ? 1 + log2_of(v / 2) : 0; }

// Home leaves of a request, and log2 of the waves that share one.
template <class Args>
__device__ inline uint32_t home_leaves(const Args &A)
{
    return A.leaf_count ? *A.leaf_count : (uint32_t)A.tree->cnt[0];
}
template <int G, class Args>
__device__ inline int home_split(const Args &A, bool splits)
{
    if (!splits) return 0;
    if (A.leaf_count && A.leaf_count == A.heavy_count) return log2_of(G);   // heavy leaves
    const int all = split_of(A.n, G), some = split_of((int64_t)home_leaves(A) * G, G);
    return all > some ? all : some;
}

template <int G, class Args, class Splits>
__device__ inline void batch_prefix(const Batch<Args> &B, uint32_t *pre, Splits splits)
{
    // the host keeps the total leaf count (<= total particles) below 2^32
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        pre[0] = 0;
        for (int r = 0; r < B.nreq; r++) {
            acc += home_leaves(*B.req[r]) << home_split<G>(*B.req[r], splits(*B.req[r]));
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
// polynomial in x.  Of D1 the sum of q f' is kept (D1 = N D0 - it): Omega is that
// sum over D0, and where the particle itself is nearly all of D0 it would be lost
// in the difference.
template <int K>
struct Sums {
    double d0 = 0.0, s2 = 0.0;             // sum m f, sum m q f' (M4, FP64: a third of it)
    double d2 = 0.0;
    double wn = 0.0;                       // D3 of unequal masses, quintic's D3
    double edge = 1e300;                   // smallest |q - knot| met
    int n = 0, n1 = 0;                     // entries inside R h, inside h
    static constexpr int N = K == SPH_KERNEL_QUINTIC ? 5 : 3;
};

// Sums of a particle whose list filled up and was started afresh.
struct PartSums {
    double d0, s2, d2, wn;
    int n, n1;
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
    if constexpr (!EQ) m = in ? m : 0.0;   // (infinity * 0 outside R h)
    if constexpr (K == SPH_KERNEL_QUINTIC) {
        const double t3 = 3.0 - q;
        const double a = fmax(t3, 0.0), b = fmax(2.0 - q, 0.0), c = fmax(1.0 - q, 0.0);
        s.edge = fmin(s.edge, fabs(t3));
        const double a2 = a * a, b2 = b * b, c2 = c * c;
        const double a3 = a2 * a, b3 = b2 * b, c3 = c2 * c;
        const double a4 = a2 * a2, b4 = b2 * b2, c4 = c2 * c2;
        const double e0 = a4 * a - 6.0 * (b4 * b) + 15.0 * (c4 * c);
        const double t = 30.0 * b4 - 5.0 * a4 - 75.0 * c4;
        const double e2 = 90.0 * a3 - 240.0 * b3 + 150.0 * c3;
        const double e3 = 270.0 * a2 - 480.0 * b2 + 150.0 * c2;
        if constexpr (EQ) {
            s.d0 += e0;
            s.s2 = fma(q, t, s.s2);
            s.d2 += e2;
            s.wn += e3;
        } else {
            s.d0 += m * e0;
            s.s2 = fma(m * q, t, s.s2);
            s.d2 += m * e2;
            s.wn += m * e3;
        }
    } else {
        const double t2 = 2.0 - q, t1 = 1.0 - q;
        const double a = fmax(t2, 0.0), b = fmax(t1, 0.0);
        s.edge = fmin(fmin(s.edge, fabs(t2)), fabs(t1));
        const double a2 = a * a, b2 = b * b;
        const double e0 = (0.25 * a2) * a - b2 * b;
        const double t = b2 - 0.25 * a2;     // x 3
        const double e2 = a - b;             // x 3
        const bool in1 = t1 > 0.0;
        if constexpr (EQ) {
            s.d0 += e0;
            s.s2 = fma(q, t, s.s2);
            s.d2 += e2;
            s.n1 += in1 ? 1 : 0;
        } else {
            s.d0 += m * e0;
            s.s2 = fma(m * q, t, s.s2);
            s.d2 += m * e2;
            s.wn += m * ((in ? 2.0 : 0.0) - (in1 ? 1.0 : 0.0));
        }
    }
}

// A tight tolerance: the result then does not depend on how the root was
// approached, and the polynomial above may stand in for a pass.  With a loose
// one (the paper's 1 %) the solve stops at whatever h meets it, so it keeps to
// the plain Newton path.
constexpr double kTightTol = 1e-9;

// r^2 of the places that fill an FP64 list up to a whole step.
constexpr double kPadding = 1e300;

// The polynomial stands for the kernel sum near h: further away neighbours cross
// the kernel's knots, and the quintic's lacks its last two terms, while Newton on
// F(h) is exact where the density is uniform.  Up to a change of h of a half, cold
// quintic solves took up to 15 passes instead of Newton's 9 (cluster in a void, mean
// 3.42; with a tenth at most 8, mean 3.22, density of 80,000 particles 10.9 -> 6.4
// ms, with a fifth 10.9 again).  M4: guesses three times too large 5.70 passes, with
// a fifth 3.98 and a tenth 4.01 (80,000: 2.57 and 1.90 ms); 2,097,152 particles with
// the benchmark's guesses 2.31 ms up to a half or a fifth, 2.37 with a tenth.
template <int K>
constexpr double kPolyStep = K == SPH_KERNEL_QUINTIC ? 0.1 : 0.2;

// LW: the launch holds FP32-pair sets whose wide groups are tested lane by lane
// (DensArgs::lanewise).
template <int G, int PREC, int K, bool LW>
__global__ __launch_bounds__(kWave, pair_waves_per_simd<PREC>()) void k_density(Batch<DensArgs> B)
{
    constexpr int L0 = kWave / G;   // lanes per home particle of a whole leaf
    constexpr double RK = Kern<K>::R, SIG = Kern<K>::sigma;
    constexpr bool F64 = PREC == SPH_FP64;
    static_assert(Kern<K>::list % (4 * L0) == 0, "lists hold whole steps of four entries per lane");
    __shared__ WalkBuf wb;
    __shared__ TreeInfo T;
    __shared__ LeafTab<PREC> tab;
    __shared__ union {
        uint16_t id[F64 ? 1 : G * Words<G>::cap];   // FP32-pair: pairs of each home particle
        uint32_t walk_spare[kFront];                // lent to walks, which run between sweeps
    } S;
    __shared__ HomeTab<G, PREC> H;
    __shared__ HomeOp<F64 ? 0 : G> op;
    __shared__ uint64_t near_of[G];
    __shared__ PartSums part[G];
    __shared__ double part_edge[F64 ? G : 1];
    __shared__ uint32_t pre[kMaxBatch + 1];
    auto splits = [](const DensArgs &A) { return splits_density(PREC, A.box.periodic); };
    batch_prefix<G>(B, pre, splits);
    const int lane = threadIdx.x;
    // Candidate lists of this block: for every home particle up to KP entries
    // (r^2, and m unless all masses are equal) of the candidates within R Rc
    // of it, in the order a sweep meets them, one particle after the other.
    // FP32-pair forms every r^2 in single precision, so its list holds them
    // as floats (half the bytes, the same values); FP64 lists hold doubles.
    // A particle's lanes read 64 consecutive bytes of its list per load.
    using ListR2 = std::conditional_t<F64, double, float>;
    const int slice = (Kern<K>::list * G) >> B.split;
    double *const cslice = B.cache + (size_t)blockIdx.x * (2 * slice);
    ListR2 *const cr2 = reinterpret_cast<ListR2 *>(cslice);
    double *const cm = cslice + slice;
    // the request's counters, lane k for counts[k] (no scalar registers)
    int64_t tally = 0;
    auto count_up = [&](int k, int v) { tally += lane == k ? v : 0; };
    int cur = -1, split = 0;
    const __attribute__((address_space(4))) DensArgs *Ap = nullptr;
    // flushed when the wave moves to another request
    auto flush_counts = [&]() {
        if (cur >= 0 && tally != 0) {
            unsigned long long *to = (unsigned long long *)&Ap->counts[blockIdx.x % kCountRows * kCountWords + lane];
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
            split = __builtin_amdgcn_readfirstlane(home_split<G>(*B.req[r], splits(*B.req[r])));
        }
        const auto &A = *Ap;
        const int64_t item = gleaf - (int64_t)__builtin_amdgcn_readfirstlane(pre[r]);
        const int64_t li = item >> split;
        const int64_t leaf = A.leaf_list ? (int64_t)as_const(A.leaf_list)[li] : li;
        if (A.leaf_act && as_const(A.leaf_act)[leaf] == 0) return;   // no active particle
        // this wave's share of the leaf, and the lanes of each of its particles
        const int share = G >> split, LPP = L0 << split;
        const int p = lane >> (log2_of(L0) + split), q = lane & (LPP - 1);
        const int64_t first = (int64_t)as_const(A.lstart)[leaf] + (item & ((1 << split) - 1)) * share;
        const int nhome = (int)((int64_t)as_const(A.lstart)[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome && (!A.active || as_global(A.active)[i] != 0);
        if (__ballot(active) == 0ull) return;
        const int64_t ii = active ? i : first;
        const double mi = as_global(A.m)[ii];
        const double mu = as_const(A.mrange)[0];
        const bool equal_m = mu == as_const(A.mrange)[1];
        const bool tight = F64 && A.h_rtol <= kTightTol;
        // entries that a step of a particle's lanes reads, and a list's (whole
        // steps): the scratch holds an r^2 and a mass per entry as doubles, so equal
        // masses leave room for twice as many, four times with single-precision r^2
        // (a list that fills up is summed up in every pass instead of once: 12,167
        // particles FP32-pair 160 -> 104 us)
        const int more = (split - slice_split(A.n, G, splits(*B.req[r]))) + (equal_m ? (F64 ? 1 : 2) : 0);
        const int CHUNK = 4 * LPP, KP = (Kern<K>::list << more) & -CHUNK;
        double h = as_global((const double *)A.h)[ii];
        double lo_b = 0.0, hi_b = INFINITY;
        bool conv = !active;
        double h_out = h, rho_out = 0.0, om_out = 1.0;
        int n_out = 0;
        if (split > 0 && lane < G) H.d[lane].thr = -1.0;
        wave_lds_sync();
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
        // A node can hold neighbours if its box is within R hcov of the home leaf's
        // box, and (`close`) within R hw of some home particle, hw the walk's
        // margin over its h
        bool close = false;
        double hw = hcov;
        auto near_home = [&](const Node &home, const Box &bx, uint64_t part) {
            const double R = RK * hcov * (1.0 + 1e-10);
            const double R2 = R * R;
            const bool cl = close;
            return [&bx, &home, R2, part, cl](const Node &nd) {
                return box_gap2(home, nd, bx) < R2 && (!cl || node_in_reach<G, PREC>(H, part, nd, bx, -1.0));
            };
        };
        WalkResult wr{0, 0, nullptr};
        bool walked = false;
        int iter = 0;
        int evals_leaf = 0;   // this lane's density pairs evaluated for this leaf
        // list state of this particle: `cached` = the list holds every
        // candidate within R Rc; valid while h <= Rc.  count: its entries.
        bool cached = false;
        double Rc = 0.0;
        int count = 0;
        for (;;) {
            if (!walked) {
                // the walk and the candidate loads are chains of dependent loads:
                // the wave issues them at raised priority, ahead of waves in their
                // arithmetic (measured: the force loop 1 % faster, the density
                // loop unchanged)
                __builtin_amdgcn_s_setprio(2);
                const Node home = load_const(reload(A.nodes) + leaf);
                const Box bx = load_const(&reload(B.req[r])->box);
                const uint64_t part = particle_bits(!conv, LPP);
                close = false;
                hw = hcov;
                for (;;) {
                    wr = walk(T, A.nodes, near_home(home, bx, part), wb, S.walk_spare);
                    count_up(kCntDensWalks, close ? 0 : 1);
                    if (!close && wr.lev) count_up(kCntDensOverflows, 1);
                    if (close || (wr.lev == 0 && wr.n <= kManyLeaves)) break;
                    close = true;
                    hw = A.walk_margin * h;
                    if (q == 0) H.d[p].thr = (RK * hw) * (RK * hw);
                    wave_lds_sync();
                }
                __builtin_amdgcn_s_setprio(0);
                if (close && left_over(A, split, wr, leaf)) return;
                walked = true;
            }
            const double hinv = 1.0 / h;
            // (an infinite guess reaches every particle, but not the lists' padding)
            double h2x4 = (RK * h) * (RK * h);
            h2x4 = h2x4 > kPadding ? kPadding : h2x4;
            uint64_t emptied = 0;   // bit p: home particle p's list was, in this sweep
            // the pair terms of one entry (eq: all masses are equal, m not used)
            auto add = [&](Sums<K> &sm, auto eq, ListR2 r2, double m, double hinv, double h2x4) {
                constexpr bool EQ = decltype(eq)::value;
                if constexpr (F64) {
                    add_entry<K, EQ>(sm, r2, m, hinv, h2x4);
                } else {
                    // branch-free: an entry outside R h adds 0 * f, whatever it holds
                    // (padding, a position that is not finite: f and f' are zero, q
                    // f' is not a number)
                    const bool in = r2 < (float)h2x4;
                    const double mj = in ? (EQ ? mu : m) : 0.0;
                    float f, df;
                    const float qq = sqrtf(r2) * (float)hinv;
                    kern<K>(qq, f, df);
                    sm.d0 += mj * (double)f;
                    sm.s2 += mj * (double)(in ? qq * df : 0.f);
                    sm.n += in ? 1 : 0;
                }
            };
            // the pair terms of this particle's list entries [0, n), its lanes
            // sharing them four at a time; entries past n up to a whole step
            // are far away and add nothing
            auto eval_list = [&](Sums<K> &sm, int n) {
                const auto *l = as_global(cr2 + p * KP);
                const auto *lm = as_global(cm + p * KP);
                auto sums = [&](auto eq) {
                    constexpr bool EQ = decltype(eq)::value;
                    if constexpr (F64) {
                        using D2 = double __attribute__((ext_vector_type(2)));
                        using P2 = const __attribute__((address_space(1))) D2 *;
                        for (int e = 2 * q; e < n; e += CHUNK) {
                            const D2 u = *(P2)(l + e), v = *(P2)(l + e + 2 * LPP);
                            D2 mu2{}, mv2{};
                            if constexpr (!EQ) {
                                mu2 = *(P2)(lm + e);
                                mv2 = *(P2)(lm + e + 2 * LPP);
                            }
                            add(sm, eq, u.x, mu2.x, hinv, h2x4);
                            add(sm, eq, u.y, mu2.y, hinv, h2x4);
                            add(sm, eq, v.x, mv2.x, hinv, h2x4);
                            add(sm, eq, v.y, mv2.y, hinv, h2x4);
                        }
                    } else {
                        using F4 = float __attribute__((ext_vector_type(4)));
                        using D4 = double __attribute__((ext_vector_type(4)));
                        for (int e = 4 * q; e < n; e += CHUNK) {
                            const F4 u = *(const __attribute__((address_space(1))) F4 *)(l + e);
                            D4 mw{};
                            if constexpr (!EQ) mw = *(const __attribute__((address_space(1))) D4 *)(lm + e);
#pragma unroll
                            for (int k = 0; k < 4; k++) add(sm, eq, u[k], mw[k], hinv, h2x4);
                        }
                    }
                };
                if (equal_m) sums(std::true_type{});
                else sums(std::false_type{});
            };
            // entries [n, whole step) of this particle's list: far away
            auto pad_list = [&](int n) {
                const int end = (n + CHUNK - 1) & -CHUNK;
                for (int e = n + q; e < end; e += LPP) {
                    cr2[p * KP + e] = F64 ? (ListR2)kPadding : (ListR2)INFINITY;
                    if (!equal_m) cm[p * KP + e] = 0.0;
                }
                wave_mem_sync();
            };
            // the n entries of home particle pp's list, which is full, added to its
            // sums by the whole wave; the list starts afresh
            auto empty_list = [&](int pp, int n) {
                Sums<K> t;
                const double hv = readlane_d(hinv, pp * LPP), hh = readlane_d(h2x4, pp * LPP);
                wave_mem_sync();
                for (int e = lane; e < n; e += kWave) {
                    const ListR2 r2 = as_global(cr2)[pp * KP + e];
                    if (equal_m) add(t, std::true_type{}, r2, 0.0, hv, hh);
                    else add(t, std::false_type{}, r2, as_global(cm)[pp * KP + e], hv, hh);
                }
                const bool first_time = !((emptied >> pp) & 1);
                count_up(kCntDensListOverflows, first_time ? 1 : 0);
                emptied |= 1ull << pp;
                const double d0 = wave_sum(t.d0), s2 = wave_sum(t.s2), d2 = wave_sum(t.d2), wn = wave_sum(t.wn);
                const int n0 = (int)wave_sum_int(t.n), n1 = (int)wave_sum_int(t.n1);
                const PartSums c = first_time ? PartSums{} : part[pp];
                wave_lds_sync();
                const double edge = F64 ? -wave_max(-t.edge) : 0.0;
                if (lane == 0) {
                    part[pp] = PartSums{c.d0 + d0, c.s2 + s2, c.d2 + d2, c.wn + wn, c.n + n0, c.n1 + n1};
                    if constexpr (F64) part_edge[pp] = first_time ? edge : fmin(part_edge[pp], edge);
                }
                wave_lds_sync();
            };
            if (__ballot(!conv && !cached) != 0ull) {
                // sweep: every particle still iterating rebuilds its list
                // around its current h.  A list that fills up is added to the
                // particle's sums and started afresh; it cannot serve later
                // steps then
                double rc2 = -1.0;
                if (!conv) {
                    Rc = fmin(kCacheGrow * h, hw);
                    rc2 = (RK * Rc) * (RK * Rc);
                }
                wave_lds_sync();
                if (q == 0) H.d[p].thr = rc2;
                wave_lds_sync();
                const auto &Q = *reload(Ap);
                const Node home = load_const(reload(A.nodes) + leaf);
                const Box bx = load_const(&reload(B.req[r])->box);
                HomeUnits units{};
                if constexpr (!F64) units = home_operand<G, PREC>(H, home, hcov, op);
                const uint64_t takes_part = particle_bits(!conv, LPP);
                // (whole rows, so that a list that fills up does so at the same
                // row whatever the depth)
                constexpr int LPR = kWave / G;
                const int depth = group_depth<G>(wr.n, B.stage > 0 ? (B.stage * G / 2 + LPR - 1) / LPR * LPR : kGroup);
                count = 0;
                int held = 0;              // FP64: entries of home particle `lane`'s list
                int64_t at = 0;
                const uint32_t *leaves = nullptr;
                auto test = near_home(home, bx, takes_part);
                for (;;) {
                    const int ng = next_group(T, Q.nodes, wr, test, wb, depth, at, leaves);
                    if (ng == 0) break;
                    const int img = open_group<G, PREC, K>(leaves, ng, Q.lstart, Q.nodes, home, bx, hcov, tab, H,
                                                           takes_part, F64 ? near_of : nullptr);
                    count_up(kCntDensVisits, ng);
                    if (Q.count_tests) {
                        count_up(kCntDensBoxes, ng * (int)__popcll(takes_part));
                        count_up(kCntDensTests, ng * G * (int)__popcll(takes_part));
                    }
                    // FP32-pair groups whose every candidate the products would list
                    // are tested lane by lane too
                    if (F64 || (LW && (units.wide || img == kImgWide) && Q.lanewise)) {
                        uint64_t near = near_of[lane < G ? lane : 0];
                        if constexpr (!F64) {
                            near = ~0ull;
                            held = __shfl(count, (lane * LPP) & (kWave - 1));
                        }
                        if (lane >= G || !((takes_part >> lane) & 1)) near = 0;
                        auto mass = [&](uint32_t j) { return equal_m ? mu : as_global(Q.m)[j]; };
                        auto put = [&](uint32_t to, ListR2 r2, double m) {
                            // (fixed uniform base, 32-bit lane offset)
                            auto *list = (__attribute__((address_space(1))) char *)cr2;
                            *(__attribute__((address_space(1))) ListR2 *)(list + to * (uint32_t)sizeof(ListR2)) = r2;
                            if (!equal_m) {
                                auto *lm = (__attribute__((address_space(1))) char *)cm;
                                *(__attribute__((address_space(1))) double *)(lm + to * 8u) = m;
                            }
                        };
                        auto rows = [&](auto im, auto nr) {
                            constexpr int IM = decltype(im)::value, NR = decltype(nr)::value;
                            return test_rows<G, PREC, IM, NR>(tab, H, ng, bx, Q.pos, Q.off, near, held, KP, mass, put);
                        };
                        using None = std::integral_constant<int, kImgNone>;
                        using Shift = std::integral_constant<int, kImgShift>;
                        using Pair = std::integral_constant<int, kImgPair>;
                        using Full = std::integral_constant<int, kRows>;
                        using Half = std::integral_constant<int, kRows / 2>;
                        using One = std::integral_constant<int, 1>;
                        for (;;) {
                            int full;
                            if constexpr (F64) {
                                if (img == kImgNone) full = rows(None{}, Full{});
                                else if (img == kImgShift) full = rows(Shift{}, Half{});
                                else full = rows(Pair{}, Half{});
                            } else {
                                if (img < kImgPair) full = rows(None{}, One{});
                                else full = rows(Pair{}, One{});
                            }
                            if (full < 0) break;
                            empty_list(full, __builtin_amdgcn_readlane(held, full));
                            held = lane == full ? 0 : held;
                        }
                        if constexpr (!F64) count = __shfl(held, p);
                        wave_lds_sync();   // the next group rewrites the table
                    } else if constexpr (!F64) {
                        // r^2 of the pairs to the particle's list, its lanes taking
                        // them in turn, two at a time (both positions requested
                        // before either is used)
                        auto use = [&](int n) {
                            const HomeRowF hd = H.f[p];
                            const float hx = hd.x, hy = hd.y, hz = hd.z;
                            const uint16_t *id = S.id + p * Words<G>::cap;
                            int done = 0;
                            for (;;) {
                                const int m = n - done < KP - count ? n - done : KP - count;
                                auto *to = as_global_out(cr2 + p * KP + count);
                                auto *tm = as_global_out(cm + p * KP + count);
                                for (int e = q; e < m; e += 2 * LPP) {
                                    const bool two = e + LPP < m;
                                    const int sa = id[done + e], sb = id[done + (two ? e + LPP : e)];
                                    const uint2 ma = tab.jm[sa / G], mb = tab.jm[sb / G];
                                    const uint32_t ja = ma.x + (uint32_t)(sa % G), jb = mb.x + (uint32_t)(sb % G);
                                    ListR2 dx, dy, dz, w;
                                    const ListR2 ra = group_separation<PREC, ListR2>(
                                        tab, img, bx, hx, hy, hz, sa / G, ma, ja, Q.pos, Q.off, dx, dy, dz, w);
                                    const ListR2 rb = group_separation<PREC, ListR2>(
                                        tab, img, bx, hx, hy, hz, sb / G, mb, jb, Q.pos, Q.off, dx, dy, dz, w);
                                    to[e] = ra;
                                    if (two) to[e + LPP] = rb;
                                    if (!equal_m) {
                                        tm[e] = as_global(Q.m)[ja];
                                        if (two) tm[e + LPP] = as_global(Q.m)[jb];
                                    }
                                }
                                count += m;
                                done += m;
                                const bool full = done < n;
                                if (__ballot(full) == 0ull) break;
                                // full lists (KP entries, whatever the groups)
                                for (uint64_t f = __ballot(full && q == 0); f; f &= f - 1)
                                    empty_list((int)__builtin_ctzll(f) >> (log2_of(L0) + split), KP);
                                if (full) count = 0;
                            }
                        };
                        group_pairs<G, PREC, false>(p, tab, home, bx, ng, img, op, units, Q.pos, Q.off, S.id, use);
                    }
                }
                if constexpr (F64) {
                    const int mine = __shfl(held, p);   // every lane takes part
                    count = conv ? 0 : mine;
                }
                cached = !conv && !((emptied >> p) & 1);
                pad_list(count);
            }
            Sums<K> sm;
            eval_list(sm, conv ? 0 : count);
            if (((emptied >> p) & 1) && q == 0) {
                const PartSums &t = part[p];
                sm.d0 += t.d0;
                sm.s2 += t.s2;
                sm.d2 += t.d2;
                sm.wn += t.wn;
                if constexpr (F64) sm.edge = fmin(sm.edge, part_edge[p]);
                sm.n += t.n;
                sm.n1 += t.n1;
            }
            // one evaluation for every particle still iterating (uniform)
            count_up(kCntNrTotal, (int)__popcll(__ballot(!conv && q == 0)));
            const int cnt = lanes_sum<L0>(sm.n, LPP) - 1;   // without the particle itself
            double s0, s2;
            // x: relative change of h to the root (the polynomial's, where it
            // could be solved), b1: the polynomial's derivative there
            double x = 0.0, b1 = 0.0, edge = 0.0;
            bool poly = false;
            if constexpr (F64) {
                const double sc = equal_m ? mu : 1.0;
                const double f3 = K == SPH_KERNEL_QUINTIC ? 1.0 : 3.0;
                constexpr double N = Sums<K>::N;
                const double D0 = sc * lanes_sum<L0>(sm.d0, LPP);
                s2 = sc * (f3 * lanes_sum<L0>(sm.s2, LPP));
                const double D1 = N * D0 - s2;
                const double D2 = sc * (f3 * lanes_sum<L0>(sm.d2, LPP));
                double D3 = lanes_sum<L0>(sm.wn, LPP);
                if constexpr (K != SPH_KERNEL_QUINTIC) {
                    const int n1 = lanes_sum<L0>(sm.n1, LPP);
                    if (equal_m) D3 = (double)(2 * (cnt + 1) - n1);
                }
                D3 *= sc;
                edge = -lanes_max<L0>(-sm.edge, LPP);
                s0 = D0;
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
                        // (a lane whose solve leaves the range of use ends as not solved)
                        if (__ballot(!conv && fabs(st) > 1e-16 + 1e-15 * fabs(x) && fabs(x) < 0.5) == 0ull)
                            break;
                    }
                    // (a massless particle's relation has no root in h: plain Newton
                    // halves h until the particle is alone)
                    poly = kt > 0.0 && fabs(x) < kPolyStep<K> && fabs(st) <= 1e-15 + 1e-12 * fabs(x);
                    b1 = (3.0 * D3 * x + 2.0 * D2) * x + D1;
                }
            } else {
                s0 = lanes_sum<L0>(sm.d0, LPP);
                s2 = lanes_sum<L0>(sm.s2, LPP);
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
                    // rounding of q) and the pass has seen every neighbour there:
                    // the solve is done without another one
                    const bool exact = poly && inside && hn <= Rc &&
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
            if (__ballot(!conv && h > hw) != 0ull) {
                hcov = A.walk_margin * wave_max(conv ? 0.0 : h);
                walked = false;
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

// AC: the launch carries artificial conductivity (some set of the batch has
// alpha_AC > 0; a set with alpha_AC = 0 then adds exact zeros).
// SW: the launch carries per-particle alpha or the velocity divergence and
// curl (the artificial-viscosity switches); a set without them uses alpha_AV
// for every pair as the plain variant does.
template <int G, int PREC, bool AC, bool SW, int K>
__global__ __launch_bounds__(kWave, pair_waves_per_simd<PREC>()) void k_forces(Batch<ForceArgs> B)
{
    constexpr int L0 = kWave / G;   // lanes per home particle of a whole leaf
    constexpr bool F64 = PREC == SPH_FP64;
    __shared__ WalkBuf wb;
    __shared__ TreeInfo T;
    __shared__ LeafTab<PREC> tab;
    __shared__ union {
        uint16_t id[G * Words<G>::cap];   // pairs of each home particle: slots of the open group
        uint32_t walk_spare[kFront];      // lent to walks, which run between groups
    } S;
    __shared__ HomeTab<G, PREC> H;
    __shared__ HomeOp<G> op;
    __shared__ uint32_t pre[kMaxBatch + 1];
    batch_prefix<G>(B, pre, [](const ForceArgs &) { return true; });
    const int lane = threadIdx.x;
    // the request's counters, lane k for counts[k] (no scalar registers)
    int64_t tally = 0;
    auto count_up = [&](int k, int v) { tally += lane == k ? v : 0; };
    int cur = -1, split = 0;
    const __attribute__((address_space(4))) ForceArgs *Fp = nullptr;
    auto flush_counts = [&]() {
        if (cur >= 0 && tally != 0)
            atomicAdd((unsigned long long *)&Fp->counts[blockIdx.x % kCountRows * kCountWords + lane],
                      (unsigned long long)tally);
        tally = 0;
    };
    for_each_home_leaf(pre[B.nreq], B.work, B.claim, [&](int64_t gleaf) {
        const int r = __builtin_amdgcn_readfirstlane(find_req(pre, B.nreq, gleaf));
        if (r != cur) {
            flush_counts();
            cur = r;
            Fp = as_const(B.req[r]);
            load_tree(Fp->tree, T);
            split = __builtin_amdgcn_readfirstlane(home_split<G>(*B.req[r], true));
        }
        const auto &F = *Fp;
        const int64_t item = gleaf - (int64_t)__builtin_amdgcn_readfirstlane(pre[r]);
        const int64_t li = item >> split;
        const int64_t leaf = F.leaf_list ? (int64_t)as_const(F.leaf_list)[li] : li;
        if (F.leaf_act && as_const(F.leaf_act)[leaf] == 0) return;   // no active particle
        const Box bx = load_const(&B.req[r]->box);
        const double alpha = F.alpha, beta = F.beta;
        const double *const alpha_p = SW ? F.alpha_p : nullptr;
        const double alpha_ac = AC ? F.alpha_ac : 0.0, u_per_c2 = AC ? F.u_per_c2 : 0.0;
        const double inv_gamma = AC ? F.inv_gamma : 0.0;
        const bool ac_price = AC && F.ac_price != 0;
        // this wave's share of the leaf, and the lanes of each of its particles
        const int share = G >> split, LPP = L0 << split;
        const int p = lane >> (log2_of(L0) + split), q = lane & (LPP - 1);
        const int64_t first = (int64_t)as_const(F.lstart)[leaf] + (item & ((1 << split) - 1)) * share;
        const int nhome = (int)((int64_t)as_const(F.lstart)[leaf + 1] - first);
        const int64_t i = first + p;
        const bool active = p < nhome && (!F.active || as_global(F.active)[i] != 0);
        if (__ballot(active) == 0ull) return;
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
        if (split > 0 && lane < G) H.d[lane].thr = -1.0;
        wave_lds_sync();
        if (q == 0) {
            H.d[p] = HomeRow{hx, hy, hz, active ? hi2x4 : -1.0};
            if constexpr (!F64) H.f[p] = HomeRowF{hfx, hfy, hfz, 0.f};
        }
        // symmetric criterion: a node can hold force neighbours of the home leaf
        // if its box is closer than R max(h over home, h over node), and (`close`)
        // of some home particle if it is closer than R max(h, h over node)
        const uint64_t part = particle_bits(active, LPP);
        bool close = false;
        auto test = [&](const Node &nd) {
            const double R = RK * fmax(home.hmax, nd.hmax) * (1.0 + 1e-10);
            const double hk = RK * nd.hmax;
            return box_gap2(home, nd, bx) < R * R &&
                   (!close || node_in_reach<G, PREC>(H, part, nd, bx, hk * hk));
        };
        // walk and candidate loads at raised priority, as in the density loop
        __builtin_amdgcn_s_setprio(2);
        WalkResult wr;
        for (;;) {
            wr = walk(T, F.nodes, test, wb, S.walk_spare);
            if (!close && wr.lev) count_up(kCntForceOverflows, 1);
            if (close || (wr.lev == 0 && wr.n <= kManyLeaves)) break;
            close = true;
        }
        __builtin_amdgcn_s_setprio(0);
        if (close && left_over(F, split, wr, leaf)) return;

        double axi = 0.0, ayi = 0.0, azi = 0.0, dui = 0.0, vs_max = -INFINITY;
        double dvs = 0.0, cxs = 0.0, cys = 0.0, czs = 0.0;   // div v, curl v sums (SW)
        int cnt = 0;
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
        const HomeUnits units = home_operand<G, PREC>(H, home, home.hmax, op);
        const Real reach2 = (Real)hi2x4;
        const int depth = group_depth<G>(wr.n, B.stage > 0 ? B.stage * G / 2 : kGroup);
        int64_t at = 0;
        const uint32_t *leaves = nullptr;
        for (;;) {
            const int ng = next_group(T, F.nodes, wr, test, wb, depth, at, leaves);
            if (ng == 0) break;
            const int img = open_group<G, PREC, K>(leaves, ng, F.lstart, F.nodes, home, bx, -1.0, tab, H, 0, nullptr);
            if (F.count_tests) {
                count_up(kCntForceBoxes, ng);
                count_up(kCntForceTests, ng * G * (int)__popcll(__ballot(active && q == 0)));
            }
            // the pairs this particle's list holds, its lanes sharing them
            // round-robin: those within its own or the neighbour's reach, except
            // the particle itself
            auto use = [&](int n) {
                const uint32_t self = (uint32_t)i;
                const uint16_t *id = S.id + p * Words<G>::cap;
                for (int e = q; e < n; e += LPP) {
                    const int s = id[e];
                    const uint2 jm = tab.jm[s / G];
                    const uint32_t j = jm.x + (uint32_t)(s % G);
                    Real dx, dy, dz, w;
                    JData d;
                    if constexpr (F64) d = load_global(F.rec + j);
                    else d = load_global(F.rec32 + j);
                    const Real r2 = group_separation<PREC, Real>(
                        tab, img, bx, F64 ? (Real)hx : (Real)hfx, F64 ? (Real)hy : (Real)hfy,
                        F64 ? (Real)hz : (Real)hfz, s / G, jm, j, F.pos, F.off, dx, dy, dz, w);
                    if ((r2 < reach2 || r2 < w) && j != self) {
                        cnt++;
                        limiter(j);
                        pair_terms(j, d, dx, dy, dz, r2);
                    }
                }
            };
            group_pairs<G, PREC, true>(p, tab, home, bx, ng, img, op, units, F.pos, F.off, S.id, use);
        }
        axi = lanes_sum<L0>(axi, LPP);
        ayi = lanes_sum<L0>(ayi, LPP);
        azi = lanes_sum<L0>(azi, LPP);
        dui = lanes_sum<L0>(dui, LPP);
        vs_max = lanes_max<L0>(vs_max, LPP);
        cnt = lanes_sum<L0>(cnt, LPP);
        if (F.lev) lmx_l = lanes_max_int<L0>(lmx_l, LPP);
        if constexpr (SW) {
            dvs = lanes_sum<L0>(dvs, LPP);
            cxs = lanes_sum<L0>(cxs, LPP);
            cys = lanes_sum<L0>(cys, LPP);
            czs = lanes_sum<L0>(czs, LPP);
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
void launch_density(hipStream_t st, int G, int prec, bool lanewise, unsigned grid, const Batch<DensArgs> &B)
{
    auto go = [&](auto g) {
        constexpr int GG = decltype(g)::value;
        if (prec == SPH_FP32_PAIR && lanewise)
            hipLaunchKernelGGL((k_density<GG, SPH_FP32_PAIR, K, true>), dim3(grid), dim3(kWave), 0, st, B);
        else if (prec == SPH_FP32_PAIR)
            hipLaunchKernelGGL((k_density<GG, SPH_FP32_PAIR, K, false>), dim3(grid), dim3(kWave), 0, st, B);
        else
            hipLaunchKernelGGL((k_density<GG, SPH_FP64, K, false>), dim3(grid), dim3(kWave), 0, st, B);
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
