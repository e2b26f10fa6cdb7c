// Neighbour-search structure: bounding box, Hilbert or Morton keys, LSD radix sort,
// gathers into sorted order, leaf boxes and the 8-ary box tree above them.
//
// The paper builds a balanced KD-tree by median splits with N_LEAF particles
// per leaf and propagates each cell's smoothing-sphere extent box upwards
// (section 4.2).  On the GPU the same role is played by a sort along a
// space-filling curve (one radix sort instead of a recursive median selection, which the paper
// names as its tree-build scaling bottleneck, section 5.2.1) followed by
// leaves of leaf_size consecutive sorted particles; every leaf and node keeps
// the bounding box of its particles and their largest h.
#include "sph_internal.hpp"

#include <algorithm>

namespace sph {

namespace {

constexpr int kBoxThreads = 256;
constexpr int kRsThreads = 256;
// Bits per axis of the key, by set size: at least 64 cells per mean
// particle spacing along an axis (particles sharing a cell keep their input
// order: the sort is stable), rounded up to what a number of 8-bit passes
// holds: 10 bits (4 passes) up to 2^12 particles, 13 (5 passes) up to 2^21,
// else 16 (6 passes).  The sort and the segment rule use the same count.
constexpr int key_bits(int64_t n)
{
    return n <= (int64_t(1) << 12) ? 10 : (n <= (int64_t(1) << 21) ? 13 : 16);
}
static_assert(kRsTile == kRsThreads * kRsItems && kRsTileSmall == kRsThreads * kRsItemsSmall,
              "radix tiles are 256 threads wide");

__device__ inline void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(kBoxThreads) void k_box_partial(int64_t n, const double *__restrict__ x,
                                                             const double *__restrict__ y,
                                                             const double *__restrict__ z,
                                                             double *__restrict__ part)
{
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x) {
        double v[3] = {x[k], y[k], z[k]};
        for (int a = 0; a < 3; a++) { mn[a] = fmin(mn[a], v[a]); mx[a] = fmax(mx[a], v[a]); }
    }
    __shared__ double sh[6][kBoxThreads];
    for (int a = 0; a < 3; a++) { sh[a][threadIdx.x] = mn[a]; sh[3 + a][threadIdx.x] = mx[a]; }
    __syncthreads();
    for (int s = kBoxThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            for (int a = 0; a < 3; a++) {
                sh[a][threadIdx.x] = fmin(sh[a][threadIdx.x], sh[a][threadIdx.x + s]);
                sh[3 + a][threadIdx.x] = fmax(sh[3 + a][threadIdx.x], sh[3 + a][threadIdx.x + s]);
            }
        }
        __syncthreads();
    }
    if (threadIdx.x < 6) part[blockIdx.x * 6 + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(64) void k_box_final(int nb, const double *__restrict__ part,
                                                  double *__restrict__ box)
{
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int b = threadIdx.x; b < nb; b += 64)
        for (int a = 0; a < 3; a++) {
            mn[a] = fmin(mn[a], part[b * 6 + a]);
            mx[a] = fmax(mx[a], part[b * 6 + 3 + a]);
        }
    for (int o = 32; o > 0; o >>= 1)
        for (int a = 0; a < 3; a++) {
            mn[a] = fmin(mn[a], __shfl_xor(mn[a], o));
            mx[a] = fmax(mx[a], __shfl_xor(mx[a], o));
        }
    if (threadIdx.x == 0)
        for (int a = 0; a < 3; a++) { box[a] = mn[a]; box[3 + a] = mx[a]; }
}

__device__ inline uint64_t spread3(uint64_t v)
{
    v &= 0x1fffffull;
    v = (v | v << 32) & 0x1f00000000ffffull;
    v = (v | v << 16) & 0x1f0000ff0000ffull;
    v = (v | v << 8) & 0x100f00f00f00f00full;
    v = (v | v << 4) & 0x10c30c30c30c30c3ull;
    v = (v | v << 2) & 0x1249249249249249ull;
    return v;
}

// Hilbert curve: the digit of an octant and the orientation below it, by the
// orientation above (Hamilton, "Compact Hilbert Indices", 2006: an orientation
// is an entry corner e and a direction d; the octant, seen from there, is the
// Gray code of its digit).  Entry [8 (3 e + d) + octant] holds the digit and the
// new 3 e + d times 8.
//
// Why: a run of 16 particles along the Morton curve straddles its jumps, so the
// leaf boxes are larger than the particles need and a home leaf has 81 candidate
// leaves on C1-like sets (181 on a Plummer sphere's 500,000 particles, whose
// outer leaves reach across it); along the Hilbert curve 57 (68).  2,097,152
// particles in FP64: 6.10 -> 5.16 ms per evaluation, keys 21.5 -> 24 us.
// FP32-pair keeps the Morton order: its separations are differences of offsets
// rounded against the leaf centres, so other leaves would change results in
// their seventh digit.  So do resident states: the neighbour counts of
// particles that a sub-step leaves inactive stay at their place in the order
// when it changes, so another order would hand them to other particles, and a
// full sub-step gives the bits of a global step.
struct HilbertTable {
    uint8_t v[24 * 8];
};
constexpr int rot3(int x, int k)   // rotate 3 bits to the left by k (0..2)
{
    return ((x << k) | (x >> (3 - k))) & 7;
}
constexpr HilbertTable hilbert_table()
{
    HilbertTable t{};
    for (int e = 0; e < 8; e++)
        for (int d = 0; d < 3; d++)
            for (int octant = 0; octant < 8; octant++) {
                const int gray = rot3(octant ^ e, (3 - (d + 1) % 3) % 3);
                const int digit = gray ^ (gray >> 1) ^ (gray >> 2);
                // entry corner and direction of the digit's subcube
                const int below = digit == 0 ? 0 : ((digit - 1) / 2) * 2;
                const int entry = below ^ (below >> 1);
                // (trailing set bits of the digit, or of the one before it)
                const int odd = digit % 2 ? digit : digit - 1;
                int ones = 0;
                for (int b = digit == 0 ? 0 : odd; b & 1; b >>= 1) ones++;
                const int ne = e ^ rot3(entry, (d + 1) % 3);
                const int nd = (d + (digit == 0 ? 0 : ones % 3) + 1) % 3;
                t.v[8 * (3 * e + d) + octant] = (uint8_t)(digit | (3 * ne + nd) << 3);
            }
    return t;
}
__constant__ const HilbertTable kHilbert = hilbert_table();

// Position along the Hilbert curve from the interleaved octants of `bits`
// levels (a Morton key): consecutive positions are neighbouring cells, so runs
// of particles have compact boxes.  tab: the table in LDS.
__device__ inline uint64_t hilbert_key(uint64_t morton, int bits, const uint8_t *tab)
{
    uint64_t key = 0;
    uint32_t state = 0;
    for (int b = 3 * (bits - 1); b >= 0; b -= 3) {
        const uint32_t v = tab[(state & 0xf8u) | ((uint32_t)(morton >> b) & 7u)];
        key = (key << 3) | (v & 7u);
        state = v;
    }
    return key;
}

// Keys in the box stored at `box` (the bounding box a reduction wrote there),
// or, with fb.fixed (periodic sets), in the given box, which the first thread
// also stores at `box` for the kernels after this one (one launch fewer).
struct FixedBox {
    int fixed;
    double lo[3], hi[3];
};

// The box's corners, from either place.
__device__ inline void key_box(const double *box, const FixedBox &fb, double b[6])
{
    for (int a = 0; a < 3; a++) {
        b[a] = fb.fixed ? fb.lo[a] : box[a];
        b[3 + a] = fb.fixed ? fb.hi[a] : box[3 + a];
    }
}

__device__ inline uint64_t position_key(const double b[6], double x, double y, double z, int bits, int hilbert,
                                        const uint8_t *tab)
{
    double ext = fmax(fmax(b[3] - b[0], b[4] - b[1]), b[5] - b[2]);
    double cells = (double)(1u << bits);
    double scale = ext > 0.0 ? cells / ext : 0.0;
    double top = cells - 1.0;
    double q[3] = {(x - b[0]) * scale, (y - b[1]) * scale, (z - b[2]) * scale};
    uint64_t key = 0;
    for (int a = 0; a < 3; a++) {
        double c = floor(q[a]);
        c = c < 0.0 ? 0.0 : (c > top ? top : c);
        if (c != c) c = 0.0;   // NaN position: any key; flagged by the density loop
        key |= spread3((uint64_t)c) << a;
    }
    return hilbert ? hilbert_key(key, bits, tab) : key;
}

__global__ __launch_bounds__(256) void k_keys(int64_t n, const double *__restrict__ x,
                                              const double *__restrict__ y,
                                              const double *__restrict__ z, double *box,
                                              FixedBox fb, int bits, int hilbert,
                                              uint64_t *__restrict__ keys,
                                              uint32_t *__restrict__ vals)
{
    __shared__ uint8_t tab[sizeof(HilbertTable)];
    if (threadIdx.x < sizeof(HilbertTable)) tab[threadIdx.x] = kHilbert.v[threadIdx.x];
    __syncthreads();
    int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= n) return;
    double b[6];
    key_box(box, fb, b);
    if (fb.fixed && k == 0)
        for (int a = 0; a < 6; a++) box[a] = b[a];
    keys[k] = position_key(b, x[k], y[k], z[k], bits, hilbert, tab);
    vals[k] = (uint32_t)k;
}

// ---- LSD radix sort, 8-bit digits ------------------------------------------

// Block-wide exclusive scan (sum or max, of values that are 0 or above) of one
// value per thread, WAVES waves; total: over all threads.  Shuffles inside the
// waves and one exchange of their totals: with a barrier pair for each doubling
// of the distance instead, the two scans of a radix scatter block took longer
// than the rest of it.  sh: WAVES words.
template <bool MAX, int WAVES>
__device__ inline uint32_t block_scan(uint32_t v, uint32_t *sh, uint32_t &total)
{
    auto op = [](uint32_t a, uint32_t b) { return MAX ? (a > b ? a : b) : a + b; };
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t s = v;
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = __shfl_up(s, d);
        if (lane >= d) s = op(s, o);
    }
    if (lane == kWave - 1) sh[w] = s;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int k = 0; k < WAVES; k++) {
        const uint32_t o = sh[k];
        before = k < w ? op(before, o) : before;
        total = op(total, o);
    }
    __syncthreads();   // sh is free again
    const uint32_t prev = __shfl_up(s, 1);
    return lane > 0 ? op(before, prev) : before;
}

template <int ITEMS>
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(int64_t n, const uint64_t *__restrict__ keys,
                                                        int shift, uint32_t *__restrict__ hist,
                                                        int64_t ntiles)
{
    constexpr int64_t TILE = (int64_t)kRsThreads * ITEMS;
    __shared__ uint32_t cnt[256];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    int64_t base = blockIdx.x * TILE;
    for (int it = 0; it < ITEMS; it++) {
        int64_t k = base + it * kRsThreads + threadIdx.x;
        if (k < n) atomicAdd(&cnt[(keys[k] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[threadIdx.x * ntiles + blockIdx.x] = cnt[threadIdx.x];
}

// Per digit (one block each): exclusive scan over the tiles of that digit's
// counts, in place, 256 tiles at a time; the digit's total goes to totals[d].
// The digits' own offsets (a scan of the 256 totals) are formed by every
// scatter block.
__global__ __launch_bounds__(256) void k_rs_digit_scan(uint32_t *__restrict__ hist, int64_t ntiles,
                                                       uint32_t *__restrict__ totals)
{
    __shared__ uint32_t sh[4];
    uint32_t *a = hist + (int64_t)blockIdx.x * ntiles;
    uint32_t run = 0;
    for (int64_t b0 = 0; b0 < ntiles; b0 += 256) {
        const int64_t k = b0 + threadIdx.x;
        const uint32_t v = k < ntiles ? a[k] : 0u;
        uint32_t sum;
        const uint32_t before = block_scan<false, 4>(v, sh, sum);
        if (k < ntiles) a[k] = run + before;
        run += sum;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = run;
}

// Stable scatter.  Wave w of the block owns keys [tile + w*64*ITEMS, +64*ITEMS)
// and walks them in ITEMS rounds of 64 in index order; equal digits within a round
// are ranked with 8 ballots, across rounds with per-wave LDS counters, and
// across waves by an exclusive prefix of those counters.  raw = 0: offs holds
// k_rs_digit_scan's per-digit scans over the tiles and totals the digit
// totals; raw = 1 (few tiles): offs holds k_rs_hist's counts as they are and
// each block forms both itself (one thread per digit summing that digit's
// counts over the tiles), which saves the scan's launch.
template <int ITEMS>
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(int64_t n, const uint64_t *__restrict__ kin,
                                                           const uint32_t *__restrict__ vin,
                                                           uint64_t *__restrict__ kout,
                                                           uint32_t *__restrict__ vout, int shift,
                                                           const uint32_t *__restrict__ offs,
                                                           int64_t ntiles,
                                                           const uint32_t *__restrict__ totals,
                                                           int raw)
{
    __shared__ uint32_t wcnt[kRsThreads / kWave][256];
    __shared__ uint32_t dbase[256];
    __shared__ uint32_t sums[kRsThreads / kWave];
    __shared__ uint32_t tbase[256];            // first slot of each digit in the tile
    constexpr int TILE = kRsThreads * ITEMS;
    __shared__ uint64_t skey[TILE];            // the tile in digit order
    __shared__ uint32_t sval[TILE];
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    for (int k = threadIdx.x; k < (kRsThreads / kWave) * 256; k += kRsThreads)
        (&wcnt[0][0])[k] = 0;
    // this digit's keys in the tiles before this one, and in all tiles
    static_assert(kRsThreads == 256, "one thread per digit");
    uint32_t before_tile, digit_total;
    if (raw) {
        const uint32_t *h = offs + (int64_t)threadIdx.x * ntiles;
        before_tile = 0u;
        digit_total = 0u;
        for (int64_t t = 0; t < ntiles; t++) {
            const uint32_t v = h[t];
            before_tile += t < (int64_t)blockIdx.x ? v : 0u;
            digit_total += v;
        }
    } else {
        before_tile = offs[threadIdx.x * ntiles + blockIdx.x];
        digit_total = totals[threadIdx.x];
    }
    // first position of each digit: exclusive scan of the digit totals
    uint32_t all;
    dbase[threadIdx.x] = block_scan<false, kRsThreads / kWave>(digit_total, sums, all);
    __syncthreads();
    const uint64_t lt = __lanemask_lt();
    const int64_t base = blockIdx.x * (int64_t)TILE + w * (ITEMS * kWave);
    uint64_t key[ITEMS];
    uint32_t val[ITEMS];
    uint32_t rank[ITEMS];
    for (int r = 0; r < ITEMS; r++) {
        int64_t k = base + r * kWave + lane;
        bool valid = k < n;
        key[r] = valid ? kin[k] : 0ull;
        val[r] = valid ? vin[k] : 0u;
        uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
        uint64_t mask = __ballot(valid);
        for (int b = 0; b < 8; b++) {
            uint64_t bb = __ballot((d >> b) & 1u);
            mask &= ((d >> b) & 1u) ? bb : ~bb;
        }
        uint32_t before = valid ? wcnt[w][d] : 0u;
        uint32_t prior = (uint32_t)__popcll(mask & lt);
        rank[r] = before + prior;
        wave_lds_sync();
        bool leader = valid && prior == 0;
        if (leader) wcnt[w][d] = before + (uint32_t)__popcll(mask);
        wave_lds_sync();
    }
    __syncthreads();
    // per digit (one thread each): the waves' offsets inside the tile's run
    // of that digit, then the run's first slot in the tile
    uint32_t run = 0;
    for (int ww = 0; ww < kRsThreads / kWave; ww++) {
        uint32_t v = wcnt[ww][threadIdx.x];
        wcnt[ww][threadIdx.x] = run;
        run += v;
    }
    tbase[threadIdx.x] = block_scan<false, kRsThreads / kWave>(run, sums, all);
    __syncthreads();
    // stage the tile in digit order (stable: wave, then item, then lane)
    for (int r = 0; r < ITEMS; r++) {
        int64_t k = base + r * kWave + lane;
        if (k < n) {
            uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
            uint32_t lp = tbase[d] + wcnt[w][d] + rank[r];
            skey[lp] = key[r];
            sval[lp] = val[r];
        }
    }
    __syncthreads();
    // slot i of the tile goes to (global start of its digit's run in this tile)
    // + (i - tile start of that run); dbase + offs >= tbase, so no wrap
    dbase[threadIdx.x] += before_tile - tbase[threadIdx.x];
    __syncthreads();
    const int64_t left = n - blockIdx.x * (int64_t)TILE;   // >= 1
    const int tile_n = left < TILE ? (int)left : TILE;
    for (int i = threadIdx.x; i < tile_n; i += kRsThreads) {
        const uint64_t kk = skey[i];
        const uint32_t d = (uint32_t)(kk >> shift) & 255u;
        const uint32_t pos = dbase[d] + (uint32_t)i;
        kout[pos] = kk;
        vout[pos] = sval[i];
    }
}

// Up to kSmallSet particles: keys and all passes of the sort in one block of 16
// waves, the keys in LDS.  Wave w holds `rounds` x 64 consecutive keys; ranks as in
// k_rs_scatter, so the sort is stable and its order the same.  What this saves is
// launches: 4,096 keys took nine of them, 47 us, and this takes 28 us (1,000: 43 and
// 11 us).
constexpr int kSmallSet = 4096;

__global__ __launch_bounds__(1024) void k_sort_small(int n, const double *__restrict__ x,
                                                     const double *__restrict__ y,
                                                     const double *__restrict__ z, double *box, FixedBox fb,
                                                     int bits, int hilbert, uint64_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals)
{
    constexpr int W = 16, R = kSmallSet / (W * kWave);
    __shared__ uint64_t skey[kSmallSet];
    __shared__ uint16_t sval[kSmallSet];
    __shared__ uint16_t wcnt[W][256];
    __shared__ uint16_t dbase[256];
    __shared__ uint32_t sums[W];
    __shared__ uint8_t tab[sizeof(HilbertTable)];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t / kWave;
    if (t < (int)sizeof(HilbertTable)) tab[t] = kHilbert.v[t];
    __syncthreads();
    double b[6];
    key_box(box, fb, b);
    if (fb.fixed && t == 0)
        for (int a = 0; a < 6; a++) box[a] = b[a];
    const int rounds = (n + W * kWave - 1) / (W * kWave);
    const int base = w * rounds * kWave + lane;
    const uint64_t lt = __lanemask_lt();
    uint64_t key[R];
    uint32_t val[R], rank[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int k = base + r * kWave;
        // past the end: the largest key, which stays behind all others
        key[r] = ~0ull;
        val[r] = 0u;
        if (r < rounds && k < n) {
            key[r] = position_key(b, x[k], y[k], z[k], bits, hilbert, tab);
            val[r] = (uint32_t)k;
        }
    }
    for (int shift = 0; shift < 3 * bits; shift += 8) {
        for (int k = t; k < W * 256; k += 1024) (&wcnt[0][0])[k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (r >= rounds) break;
            const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
            uint64_t mask = ~0ull;
            for (int k = 0; k < 8; k++) {
                const uint64_t bb = __ballot((d >> k) & 1u);
                mask &= ((d >> k) & 1u) ? bb : ~bb;
            }
            const uint32_t before = wcnt[w][d], prior = (uint32_t)__popcll(mask & lt);
            rank[r] = before + prior;
            wave_lds_sync();
            if (prior == 0) wcnt[w][d] = (uint16_t)(before + (uint32_t)__popcll(mask));
            wave_lds_sync();
        }
        __syncthreads();
        // per digit (one thread each): the waves' offsets, then the digit's first slot
        uint32_t run = 0, all;
        if (t < 256)
            for (int k = 0; k < W; k++) {
                const uint32_t v = wcnt[k][t];
                wcnt[k][t] = (uint16_t)run;
                run += v;
            }
        const uint32_t first = block_scan<false, W>(run, sums, all);
        if (t < 256) dbase[t] = (uint16_t)first;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (r >= rounds) break;
            const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
            const uint32_t to = dbase[d] + wcnt[w][d] + rank[r];
            skey[to] = key[r];
            sval[to] = (uint16_t)val[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; r++) {
            if (r >= rounds) break;
            key[r] = skey[base + r * kWave];
            val[r] = sval[base + r * kWave];
        }
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        const int k = base + r * kWave;
        if (r < rounds && k < n) {
            keys[k] = key[r];
            vals[k] = val[r];
        }
    }
}

// ---- gathers ------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_gather(int64_t n, const uint32_t *__restrict__ perm,
                                                GatherList g, int identity)
{
    int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= n) return;
    int64_t src = identity ? k : (int64_t)perm[k];
    copy_listed(g, src, k);
}

__global__ void k_iota(int64_t n, uint32_t *__restrict__ v)
{
    int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k < n) v[k] = (uint32_t)k;
}

// ---- leaves and tree -------------------------------------------------------------
//
// Leaves are runs of at most G consecutive sorted particles that never cross
// the boundary of a cell of the curve about 4 h wide: a new segment starts between
// sorted particles k-1 and k when their keys differ above the level whose
// cell edge is the largest power-of-two fraction of the box not below
// 4 max(h_k-1, h_k).  Without this rule a run of G particles can straddle a
// jump of the curve and get a box as large as the domain.

constexpr int kScanTile = 1024;     // particles per block in the leaf scans
constexpr int kScanThreads = 256;   // 4 particles per thread

__device__ inline bool seg_break(int64_t k, const uint64_t *__restrict__ keys,
                                 const double *__restrict__ h, double ext, int bits)
{
    if (k == 0) return true;
    double hm = fmax(h[k - 1], h[k]);
    int T = 1;
    if (hm > 0.0 && ext > 0.0) {
        double t = floor(log2(ext / (4.0 * hm)));
        T = t < 1.0 ? 1 : (t > (double)bits ? bits : (int)t);
    }
    int sh = 3 * (bits - T);
    return (keys[k - 1] >> sh) != (keys[k] >> sh);
}

// per tile: break flags and the largest segment start inside the tile
__global__ __launch_bounds__(kScanThreads) void k_seg_tiles(int64_t n, const uint64_t *__restrict__ keys,
                                                            const double *__restrict__ h,
                                                            const double *__restrict__ box,
                                                            int bits, uint32_t *__restrict__ flag,
                                                            uint32_t *__restrict__ tmax)
{
    __shared__ uint32_t sh[kScanThreads / kWave];
    const double ext = fmax(fmax(box[3] - box[0], box[4] - box[1]), box[5] - box[2]);
    const int64_t base = blockIdx.x * (int64_t)kScanTile + threadIdx.x * 4;
    uint32_t mx = 0;
    for (int e = 0; e < 4; e++) {
        int64_t k = base + e;
        if (k < n) {
            bool b = seg_break(k, keys, h, ext, bits);
            flag[k] = b ? 1u : 0u;
            if (b) mx = (uint32_t)k;
        }
    }
    uint32_t top;
    block_scan<true, kScanThreads / kWave>(mx, sh, top);
    if (threadIdx.x == 0) tmax[blockIdx.x] = top;
}

// exclusive scan over the tile values, one block (max or sum); copy (when not
// null) receives the values as they were
template <bool MAX>
__global__ __launch_bounds__(1024) void k_scan_tiles(uint32_t *__restrict__ a, int64_t ntile,
                                                     uint32_t *__restrict__ copy)
{
    __shared__ uint32_t sums[16];
    const int t = threadIdx.x;
    const int64_t chunk = (ntile + 1023) / 1024;
    const int64_t s0 = t * chunk, s1 = s0 + chunk < ntile ? s0 + chunk : ntile;
    uint32_t s = 0;
    for (int64_t k = s0; k < s1; k++) s = MAX ? (a[k] > s ? a[k] : s) : s + a[k];
    uint32_t all;
    uint32_t run = block_scan<MAX, 16>(s, sums, all);
    for (int64_t k = s0; k < s1; k++) {
        uint32_t v = a[k];
        if (copy) copy[k] = v;
        a[k] = run;
        run = MAX ? (v > run ? v : run) : run + v;
    }
}

// per tile: segment start of every particle, leaf-start flags, leaf count
__global__ __launch_bounds__(kScanThreads) void k_seg_apply(int64_t n, int G,
                                                            uint32_t *__restrict__ flag,
                                                            const uint32_t *__restrict__ tmax,
                                                            uint32_t *__restrict__ tcnt)
{
    __shared__ uint32_t sh[kScanThreads / kWave];
    const int64_t base = blockIdx.x * (int64_t)kScanTile + threadIdx.x * 4;
    uint32_t loc[4];
    uint32_t mx = 0;
    for (int e = 0; e < 4; e++) {
        int64_t k = base + e;
        loc[e] = (k < n && flag[k]) ? (uint32_t)k : 0u;
        mx = loc[e] > mx ? loc[e] : mx;
    }
    uint32_t all;
    const uint32_t prev = block_scan<true, kScanThreads / kWave>(mx, sh, all);
    uint32_t seg = prev > tmax[blockIdx.x] ? prev : tmax[blockIdx.x];
    uint32_t count = 0;
    for (int e = 0; e < 4; e++) {
        int64_t k = base + e;
        if (k >= n) break;
        if (flag[k]) seg = (uint32_t)k;
        uint32_t ls = ((uint32_t)(k - seg) % (uint32_t)G) == 0u ? 1u : 0u;
        flag[k] = ls;
        count += ls;
    }
    block_scan<false, kScanThreads / kWave>(count, sh, all);
    if (threadIdx.x == 0) tcnt[blockIdx.x] = all;
}

// per tile: the first particle of every leaf
__global__ __launch_bounds__(kScanThreads) void k_leaf_starts(int64_t n, const uint32_t *__restrict__ flag,
                                                           const uint32_t *__restrict__ toff,
                                                           uint32_t *__restrict__ lstart)
{
    __shared__ uint32_t sh[kScanThreads / kWave];
    const int64_t base = blockIdx.x * (int64_t)kScanTile + threadIdx.x * 4;
    uint32_t cnt = 0;
    for (int e = 0; e < 4; e++) {
        int64_t k = base + e;
        if (k < n) cnt += flag[k];
    }
    uint32_t all;
    // leaf starts before this thread's items
    uint32_t run = toff[blockIdx.x] + block_scan<false, kScanThreads / kWave>(cnt, sh, all);
    for (int e = 0; e < 4; e++) {
        int64_t k = base + e;
        if (k >= n) break;
        if (flag[k]) {
            lstart[run] = (uint32_t)k;
            run++;
        }
        if (k == n - 1) lstart[run] = (uint32_t)n;
    }
}

// tree levels from the leaf count (one thread)
__device__ inline void tree_levels(int64_t n, int G, int64_t L, TreeInfo *__restrict__ T)
{
    T->leaf_size = G;
    T->n = n;
    int64_t cnt = L, off = 0;
    int lev = 0;
    for (; lev < kMaxLevels; lev++) {
        T->off[lev] = off;
        T->cnt[lev] = cnt;
        off += cnt;
        if (cnt <= 1) { lev++; break; }
        cnt = (cnt + 7) / 8;
    }
    T->nlev = lev;
    for (int l = lev; l < kMaxLevels; l++) { T->off[l] = off; T->cnt[l] = 0; }
}

__global__ void k_tree_info(int64_t n, int G, const uint32_t *__restrict__ toff,
                            const uint32_t *__restrict__ tcnt, int64_t ntile,
                            TreeInfo *__restrict__ T)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    tree_levels(n, G, (int64_t)toff[ntile - 1] + tcnt[ntile - 1], T);
}

// Up to kSmallSet particles: segments, leaf starts and tree levels in one block
// (the six launches above took 22 us for 1,000 particles; this takes 6 us, and 9 us
// for 4,096).
__global__ __launch_bounds__(1024) void k_leaves_small(int n, int G, const uint64_t *__restrict__ keys,
                                                       const double *__restrict__ h,
                                                       const double *__restrict__ box, int bits,
                                                       uint32_t *__restrict__ lstart, TreeInfo *__restrict__ T)
{
    constexpr int E = kSmallSet / 1024;   // consecutive particles per thread
    __shared__ uint32_t sh[16];
    const double ext = fmax(fmax(box[3] - box[0], box[4] - box[1]), box[5] - box[2]);
    const int base = threadIdx.x * E;
    bool brk[E];
    uint32_t mx = 0, all;
    for (int e = 0; e < E; e++) {
        brk[e] = base + e < n && seg_break(base + e, keys, h, ext, bits);
        if (brk[e]) mx = (uint32_t)(base + e);
    }
    uint32_t seg = block_scan<true, 16>(mx, sh, all);
    uint32_t starts = 0;   // bit e: a leaf starts at item e
    for (int e = 0; e < E; e++) {
        if (brk[e]) seg = (uint32_t)(base + e);
        if (base + e < n && ((uint32_t)(base + e) - seg) % (uint32_t)G == 0u) starts |= 1u << e;
    }
    uint32_t run = block_scan<false, 16>((uint32_t)__popc(starts), sh, all);
    for (int e = 0; e < E; e++)
        if ((starts >> e) & 1u) lstart[run++] = (uint32_t)(base + e);
    if (threadIdx.x == 0) {
        lstart[all] = (uint32_t)n;
        tree_levels(n, G, all, T);
    }
}

__device__ inline Node merge_children(const Node *__restrict__ child, int64_t c0, int64_t c1)
{
    Node nd;
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    nd.hmax = 0.0;
    nd.pad = 0.0;
    for (int64_t c = c0; c < c1; c++) {
        const Node &ch = child[c];
        for (int a = 0; a < 3; a++) {
            lo[a] = fmin(lo[a], ch.c[a] - ch.e[a]);
            hi[a] = fmax(hi[a], ch.c[a] + ch.e[a]);
        }
        nd.hmax = fmax(nd.hmax, ch.hmax);
    }
    set_box(nd, lo, hi);
    return nd;
}

// Leaf boxes and largest h: 16 lanes per leaf read its (consecutive)
// particles together, then reduce with shuffles inside their 16-lane group.
// The same pass writes the candidate positions of the pair loops.
constexpr int kLeafLanes = 16;

__global__ __launch_bounds__(256) void k_leaves(const TreeInfo *__restrict__ T,
                                                const uint32_t *__restrict__ lstart,
                                                const double *__restrict__ x,
                                                const double *__restrict__ y,
                                                const double *__restrict__ z,
                                                const double *__restrict__ h,
                                                Node *__restrict__ nodes,
                                                Pos4 *__restrict__ pos, Off4 *__restrict__ off)
{
    const int64_t L = T->cnt[0];
    const int q = threadIdx.x % kLeafLanes;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kLeafLanes);
    // the 16 lanes of a group share l, so they take the same trips
    for (int64_t l = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kLeafLanes; l < L; l += stride) {
        double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
        double hm = 0.0;
        for (int64_t k = lstart[l] + q; k < (int64_t)lstart[l + 1]; k += kLeafLanes) {
            const double v[3] = {x[k], y[k], z[k]};
            for (int a = 0; a < 3; a++) { lo[a] = fmin(lo[a], v[a]); hi[a] = fmax(hi[a], v[a]); }
            hm = fmax(hm, h[k]);
            if (pos) pos[k] = Pos4{v[0], v[1], v[2], 0.0};
        }
        for (int o = kLeafLanes / 2; o > 0; o >>= 1) {
            for (int a = 0; a < 3; a++) {
                lo[a] = fmin(lo[a], __shfl_xor(lo[a], o));
                hi[a] = fmax(hi[a], __shfl_xor(hi[a], o));
            }
            hm = fmax(hm, __shfl_xor(hm, o));
        }
        if (q == 0) {
            Node nd;
            set_box(nd, lo, hi);
            nd.hmax = hm;
            nd.pad = 0.0;
            nodes[l] = nd;
        }
        // FP32-pair mode: single-precision offsets from the centre of the box
        if (off)
            for (int64_t k = lstart[l] + q; k < (int64_t)lstart[l + 1]; k += kLeafLanes)
                off[k] = Off4{(float)(x[k] - 0.5 * (lo[0] + hi[0])), (float)(y[k] - 0.5 * (lo[1] + hi[1])),
                              (float)(z[k] - 0.5 * (lo[2] + hi[2])), 0.0f};
    }
}

// The leaves' largest h after the h solve changed h (boxes are unchanged), by the
// grid's 16-lane groups.
__device__ inline void leaf_hmax(const TreeInfo *__restrict__ T, const uint32_t *__restrict__ lstart,
                                 const double *__restrict__ h, Node *__restrict__ nodes)
{
    const int64_t L = T->cnt[0];
    const int q = threadIdx.x % kLeafLanes;
    const int64_t stride = (int64_t)gridDim.x * (blockDim.x / kLeafLanes);
    for (int64_t l = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kLeafLanes; l < L; l += stride) {
        double hm = 0.0;
        for (int64_t k = lstart[l] + q; k < (int64_t)lstart[l + 1]; k += kLeafLanes) hm = fmax(hm, h[k]);
        for (int o = kLeafLanes / 2; o > 0; o >>= 1) hm = fmax(hm, __shfl_xor(hm, o));
        if (q == 0) nodes[l].hmax = hm;
    }
}

__global__ __launch_bounds__(256) void k_leaf_hmax(const TreeInfo *__restrict__ T,
                                                   const uint32_t *__restrict__ lstart,
                                                   const double *__restrict__ h,
                                                   Node *__restrict__ nodes)
{
    leaf_hmax(T, lstart, h, nodes);
}

constexpr int64_t kSmallLevel = 4096;   // children per level handled by one block
constexpr int kBigLevels = 4;           // levels built grid-wide at most

// level `lev` from level lev-1, grid-wide, when the child level is large
__global__ __launch_bounds__(256) void k_tree_level_big(const TreeInfo *__restrict__ T,
                                                        Node *__restrict__ nodes, int lev)
{
    if (lev >= T->nlev || T->cnt[lev - 1] <= kSmallLevel) return;
    const Node *child = nodes + T->off[lev - 1];
    Node *par = nodes + T->off[lev];
    const int64_t nchild = T->cnt[lev - 1], npar = T->cnt[lev];
    for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < npar;
         p += (int64_t)gridDim.x * blockDim.x) {
        int64_t c1 = 8 * p + 8 < nchild ? 8 * p + 8 : nchild;
        par[p] = merge_children(child, 8 * p, c1);
    }
}

// all remaining (small) levels by one block, level after level
__global__ __launch_bounds__(1024) void k_tree_level_small(const TreeInfo *__restrict__ T,
                                                           Node *__restrict__ nodes)
{
    const int nlev = T->nlev;
    for (int lev = 1; lev < nlev; lev++) {
        if (lev <= kBigLevels && T->cnt[lev - 1] > kSmallLevel) continue;
        const Node *child = nodes + T->off[lev - 1];
        Node *par = nodes + T->off[lev];
        const int64_t nchild = T->cnt[lev - 1], npar = T->cnt[lev];
        for (int64_t p = threadIdx.x; p < npar; p += blockDim.x) {
            int64_t c1 = 8 * p + 8 < nchild ? 8 * p + 8 : nchild;
            par[p] = merge_children(child, 8 * p, c1);
        }
        __syncthreads();
    }
}

// Force record of particle k: A_k = P_k / (Omega_k rho_k^2),
// c_k = sqrt(gamma P_k / rho_k), 1/h_k, v_k, m_k, rho_k with
// P_k = (gamma - 1) rho_k u_k.  Also (R h_k)^2 into the position records and,
// with a tree, its leaves' largest h (the same h, one launch fewer).
__global__ __launch_bounds__(256) void k_force_prep(int64_t n, double gamma,
                                                    const double *__restrict__ rho,
                                                    const double *__restrict__ omega,
                                                    const double *__restrict__ u,
                                                    const double *__restrict__ h,
                                                    const double *__restrict__ m,
                                                    const double *__restrict__ vx,
                                                    const double *__restrict__ vy,
                                                    const double *__restrict__ vz,
                                                    ForceRec *__restrict__ rec,
                                                    ForceRec32 *__restrict__ rec32, double support,
                                                    Pos4 *__restrict__ pos, Off4 *__restrict__ off,
                                                    const TreeInfo *__restrict__ T,
                                                    const uint32_t *__restrict__ lstart,
                                                    Node *__restrict__ nodes)
{
    if (T) leaf_hmax(T, lstart, h, nodes);
    int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (k >= n) return;
    const double r = rho[k];
    const double P = (gamma - 1.0) * r * u[k];
    ForceRec f;
    f.c = sqrt(gamma * P / r);
    f.hinv = 1.0 / h[k];
    f.vx = vx[k];
    f.vy = vy[k];
    f.vz = vz[k];
    f.m = m[k];
    f.A = P / (omega[k] * r * r);
    f.rho = r;
    rec[k] = f;
    const double reach = support * h[k];
    if (pos) pos[k].reach2 = reach * reach;
    if (rec32) {
        off[k].reach2 = (float)(reach * reach);
        ForceRec32 g;
        g.c = (float)f.c;
        g.hinv = (float)f.hinv;
        g.vx = (float)f.vx;
        g.vy = (float)f.vy;
        g.vz = (float)f.vz;
        g.m = (float)f.m;
        g.A = (float)f.A;
        g.rho = (float)f.rho;
        rec32[k] = g;
    }
}

} // namespace

// nodes of the tree over at most n leaves (every leaf holds >= 1 particle)
int64_t node_count_bound(int64_t n)
{
    int64_t cnt = std::max<int64_t>(n, 1), tot = 0;
    while (true) {
        tot += cnt;
        if (cnt <= 1) break;
        cnt = ceil_div(cnt, 8);
    }
    return tot;
}

static inline unsigned grid_for(int64_t n, int threads)
{
    return (unsigned)((n + threads - 1) / threads);
}

sph_status build_order(sph_ctx *c, int64_t n, const double *x, const double *y, const double *z,
                       bool state)
{
    if (n == 0) return SPH_OK;
    const sph_params &p = c->p;
    FixedBox fb{};
    if (p.periodic) {
        // k_keys takes the box by value and stores it for the later kernels
        fb.fixed = 1;
        for (int a = 0; a < 3; a++) { fb.lo[a] = p.box_lo[a]; fb.hi[a] = p.box_hi[a]; }
    } else {
        int nb = (int)std::min<int64_t>(1024, ceil_div(n, kBoxThreads));
        hipLaunchKernelGGL(k_box_partial, dim3(nb), dim3(kBoxThreads), 0, c->stream, n, x, y, z,
                           c->d_part);
        hipLaunchKernelGGL(k_box_final, dim3(1), dim3(64), 0, c->stream, nb, c->d_part, c->d_box);
    }
    const int bits = key_bits(n);
    const int hilbert = p.precision == SPH_FP64 && !state ? 1 : 0;
    if (n <= kSmallSet) {
        hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(1024), 0, c->stream, (int)n, x, y, z, c->d_box, fb, bits,
                           hilbert, c->keys[0], c->vals[0]);
        c->perm = c->vals[0];
        c->skeys = c->keys[0];
        c->scratch_u32 = (uint32_t *)c->keys[1];
        c->tree_n = -1;
        return hip_check(c, hipGetLastError(), "build_order");
    }
    hipLaunchKernelGGL(k_keys, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, n, x, y, z,
                       c->d_box, fb, bits, hilbert, c->keys[0], c->vals[0]);
    // (a stable sort's result does not depend on the tiling)
    const bool small = n <= kRsSmallMax;
    const int64_t ntiles = small ? rs_small_tiles(n) : ceil_div(n, kRsTile);
    // more counts than c->hist holds: the gather's destination, idle until the sort ends
    uint32_t *hist = c->hist;
    int64_t room = c->hist_cap;
    if (256 * ntiles + 256 > room) {
        hist = (uint32_t *)c->t.x;
        room = 2 * c->ncap;
    }
    if (!hist || 256 * ntiles + 256 > room) return fail(c, SPH_ENOMEM, "radix count capacity");
    const int passes = (3 * bits + 7) / 8;
    const int raw = ntiles <= kRsRawMax ? 1 : 0;
    int cur = 0;
    for (int ps = 0; ps < passes; ps++) {
        int shift = 8 * ps;
        if (small)
            hipLaunchKernelGGL(k_rs_hist<kRsItemsSmall>, dim3((unsigned)ntiles), dim3(kRsThreads), 0,
                               c->stream, n, c->keys[cur], shift, hist, ntiles);
        else
            hipLaunchKernelGGL(k_rs_hist<kRsItems>, dim3((unsigned)ntiles), dim3(kRsThreads), 0,
                               c->stream, n, c->keys[cur], shift, hist, ntiles);
        if (!raw)
            hipLaunchKernelGGL(k_rs_digit_scan, dim3(256), dim3(256), 0, c->stream, hist, ntiles,
                               hist + 256 * ntiles);
        if (small)
            hipLaunchKernelGGL(k_rs_scatter<kRsItemsSmall>, dim3((unsigned)ntiles), dim3(kRsThreads),
                               0, c->stream, n, c->keys[cur], c->vals[cur], c->keys[cur ^ 1],
                               c->vals[cur ^ 1], shift, hist, ntiles, hist + 256 * ntiles, raw);
        else
            hipLaunchKernelGGL(k_rs_scatter<kRsItems>, dim3((unsigned)ntiles), dim3(kRsThreads), 0,
                               c->stream, n, c->keys[cur], c->vals[cur], c->keys[cur ^ 1],
                               c->vals[cur ^ 1], shift, hist, ntiles, hist + 256 * ntiles, raw);
        cur ^= 1;
    }
    c->perm = c->vals[cur];
    c->skeys = c->keys[cur];
    c->scratch_u32 = (uint32_t *)c->keys[cur ^ 1];
    c->tree_n = -1;
    return hip_check(c, hipGetLastError(), "build_order");
}

sph_status gather(sph_ctx *c, int64_t n, const GatherList &g, bool identity_src_index)
{
    if (n == 0 || g.count == 0) return SPH_OK;
    hipLaunchKernelGGL(k_gather, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, n, c->perm, g,
                       identity_src_index ? 1 : 0);
    return hip_check(c, hipGetLastError(), "gather");
}

// nodes above the leaves, merged level by level.  A grid-wide level is
// launched only where its children can outnumber what the one-block kernel
// takes (kSmallLevel): level l has at most ceil(n / 8^(l-1)) children (a leaf
// holds at least one particle), and a launch with fewer would return at once,
// so small sets skip those launches.
static void upper_levels(sph_ctx *c, int64_t n)
{
    int64_t children = n;
    for (int l = 1; l <= kBigLevels; l++) {
        const int64_t parents = ceil_div(children, 8);
        if (children > kSmallLevel)
            hipLaunchKernelGGL(k_tree_level_big, dim3(grid_for(parents, 256)), dim3(256), 0,
                               c->stream, c->d_tree, c->nodes, l);
        children = parents;
    }
    hipLaunchKernelGGL(k_tree_level_small, dim3(1), dim3(1024), 0, c->stream, c->d_tree, c->nodes);
}

sph_status build_tree(sph_ctx *c, int64_t n)
{
    c->tree_n = -1;
    if (n == 0) return SPH_OK;
    const int G = c->p.leaf_size;
    const bool f32 = c->p.precision == SPH_FP32_PAIR;
    if (!c->skeys || !c->scratch_u32 || !c->lstart || !c->d_tree || !c->nodes)
        return fail(c, SPH_ESTATE, "build_tree: order not built");
    const int64_t ntile = ceil_div(n, kScanTile);
    if (2 * ntile > c->hist_cap) return fail(c, SPH_ENOMEM, "scan tile capacity");
    if (c->node_cap < node_count_bound(n)) return fail(c, SPH_ENOMEM, "node capacity");
    uint32_t *tmax = c->hist, *tcnt = c->hist + ntile;
    uint32_t *flag = c->scratch_u32;
    if (n <= kSmallSet) {
        hipLaunchKernelGGL(k_leaves_small, dim3(1), dim3(1024), 0, c->stream, (int)n, G, c->skeys, c->s.h,
                           c->d_box, key_bits(n), c->lstart, c->d_tree);
    } else {
        hipLaunchKernelGGL(k_seg_tiles, dim3((unsigned)ntile), dim3(kScanThreads), 0, c->stream, n,
                           c->skeys, c->s.h, c->d_box, key_bits(n), flag, tmax);
        hipLaunchKernelGGL((k_scan_tiles<true>), dim3(1), dim3(1024), 0, c->stream, tmax, ntile,
                           (uint32_t *)nullptr);
        hipLaunchKernelGGL(k_seg_apply, dim3((unsigned)ntile), dim3(kScanThreads), 0, c->stream, n, G,
                           flag, tmax, tcnt);
        // tcnt -> exclusive offsets in place; the counts themselves go to tmax
        // for the total
        hipLaunchKernelGGL((k_scan_tiles<false>), dim3(1), dim3(1024), 0, c->stream, tcnt, ntile,
                           tmax);
        hipLaunchKernelGGL(k_tree_info, dim3(1), dim3(64), 0, c->stream, n, G, tcnt, tmax, ntile,
                           c->d_tree);
        hipLaunchKernelGGL(k_leaf_starts, dim3((unsigned)ntile), dim3(kScanThreads), 0, c->stream, n,
                           flag, tcnt, c->lstart);
    }
    hipLaunchKernelGGL(k_leaves, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, c->d_tree,
                       c->lstart, c->s.x, c->s.y, c->s.z, c->s.h, c->nodes,
                       f32 ? nullptr : c->s.pos(), f32 ? c->s.off : nullptr);
    upper_levels(c, n);
    sph_status st = hip_check(c, hipGetLastError(), "build_tree");
    if (st == SPH_OK) c->tree_n = n;
    return st;
}

sph_status refresh_hmax(sph_ctx *c, int64_t n)
{
    if (n == 0) return SPH_OK;
    if (c->tree_n != n) return fail(c, SPH_ESTATE, "refresh_hmax: tree not built");
    hipLaunchKernelGGL(k_leaf_hmax, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, c->d_tree,
                       c->lstart, c->s.h, c->nodes);
    upper_levels(c, n);
    return hip_check(c, hipGetLastError(), "refresh_hmax");
}

sph_status force_prep(sph_ctx *c, int64_t n, const double *u_sorted, const double *vx,
                      const double *vy, const double *vz, bool hmax)
{
    if (n == 0) return SPH_OK;
    if (hmax && c->tree_n != n) return fail(c, SPH_ESTATE, "force_prep: tree not built");
    const bool f32 = c->p.precision == SPH_FP32_PAIR;
    hipLaunchKernelGGL(k_force_prep, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, n,
                       c->p.gamma, c->s.rho, c->s.omega, u_sorted, c->s.h, c->s.m, vx, vy, vz,
                       c->s.frec, f32 ? c->s.frec32 : nullptr, kern_support(c->p.kernel),
                       f32 ? nullptr : c->s.pos(), f32 ? c->s.off : nullptr,
                       hmax ? c->d_tree : nullptr, c->lstart, c->nodes);
    if (hmax) upper_levels(c, n);
    return hip_check(c, hipGetLastError(), "force_prep");
}

sph_status iota(sph_ctx *c, int64_t n, uint32_t *v)
{
    if (n == 0) return SPH_OK;
    hipLaunchKernelGGL(k_iota, dim3(grid_for(n, 256)), dim3(256), 0, c->stream, n, v);
    return hip_check(c, hipGetLastError(), "iota");
}

} // namespace sph
