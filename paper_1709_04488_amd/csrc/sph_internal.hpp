// Internal definitions shared by the HIP translation units of libsph.
// Device code targets gfx950 (CDNA4, wave64) only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string>
#include <vector>

#include "../../include/sph.h"

namespace sph {

// Smoothing kernels (section 2), W(r, h) = sigma h^-3 f(r/h) with compact
// support R h:
//   M4 cubic spline, R = 2, sigma = 1/pi, in B-spline form
//     f(q) = (2-q)_+^3 / 4 - (1-q)_+^3
//   (1 - 3/2 q^2 + 3/4 q^3 on [0,1), (2-q)^3/4 on [1,2));
//   quintic spline (Morris 1996), R = 3, sigma = 1/(120 pi),
//     f(q) = (3-q)_+^5 - 6 (2-q)_+^5 + 15 (1-q)_+^5.
// list: density-loop candidate-list entries per particle (below).
template <int K>
struct Kern;
template <>
struct Kern<SPH_KERNEL_M4> {
    static constexpr double R = 2.0;
    static constexpr double sigma = 0.31830988618379067154;
    static constexpr int list = 160;
};
template <>
struct Kern<SPH_KERNEL_QUINTIC> {
    static constexpr double R = 3.0;
    static constexpr double sigma = 0.0026525823848649222;
    static constexpr int list = 480;
};
inline double kern_support(int k) { return k == SPH_KERNEL_QUINTIC ? 3.0 : 2.0; }
inline int kern_list(int k)
{
    return k == SPH_KERNEL_QUINTIC ? Kern<SPH_KERNEL_QUINTIC>::list : Kern<SPH_KERNEL_M4>::list;
}

constexpr int kWave = 64;
constexpr int kMaxLevels = 16;   // tree levels above the leaves (8-ary)
constexpr int kFront = 512;      // per-wave LDS capacity of a walk frontier / candidate list
constexpr int kXcds = 8;         // MI355X: 8 XCDs, blocks dispatched round-robin
constexpr int kMaxBatch = 128;   // particle sets per batched pair-kernel launch
constexpr int kArgBytes = 1024;  // device argument block of one pair-kernel launch

// Persistent pair-kernel grid: one wave per block, at most as many blocks as
// the GPU holds at once (256 CUs x 16 waves: the pair kernels run at 4 waves
// per SIMD), at least one block per 8 particles below that, a
// multiple of the XCD count.  Each block owns a slice of the density loop's
// candidate-list scratch, so the cap also bounds that scratch.
constexpr int64_t kMaxPairBlocks = 256 * 16;

// Radix sort tiles: 1024 keys (256 threads x 4) per block up to kRsSmallMax
// particles, 4096 (256 x 16) above.  A pass over a few hundred thousand keys is
// latency, not bandwidth: tiles of 4096 left 195,112 keys in 48 blocks on 256 CUs,
// 22.6 us per scatter (build of the order and tree: 209 -> 136 us with small
// tiles; 512,000: 233 -> 188; 1.7M: 390 -> 413, where the blocks suffice and the
// larger tiles write longer runs).  Up to kRsRawMax tiles the scatter blocks form
// the digit offsets from the raw counts themselves, one launch fewer per pass; each
// block reads all tiles' counts then, which at 63 tiles cost 64,000 particles 170
// against 120 us, and at 12 gained 12,167 as many as 12 us.  The counts take 256
// words per tile plus 256 digit totals; where that is more than hist_words, they
// stand in memory that the sort's successor fills (the budgets do not change).
constexpr int kRsItems = 16, kRsItemsSmall = 4;
constexpr int64_t kRsTile = 256 * kRsItems, kRsTileSmall = 256 * kRsItemsSmall;
constexpr int64_t kRsSmallMax = 1 << 20, kRsRawMax = 24;
constexpr int64_t kRsHistTiles = 64;   // small tiles that hist_words has room for
constexpr int64_t rs_small_tiles(int64_t n) { return (n + kRsTileSmall - 1) / kRsTileSmall; }
constexpr int64_t hist_words(int64_t cap)
{
    // the larger of the two tilings any n <= cap can use
    const int64_t big = (cap + kRsTile - 1) / kRsTile;
    const int64_t small = rs_small_tiles(cap) < kRsHistTiles ? rs_small_tiles(cap) : kRsHistTiles;
    return 256 * (big > small ? big : small) + 256;
}

// Active-leaf compaction of block time-steps: leaves per block, and the
// per-block counts (one more than the blocks, for the bound of n leaves)
constexpr int kActTile = 1024;
constexpr int64_t act_tiles(int64_t cap) { return (cap + kActTile - 1) / kActTile + 1; }
// Claim counters of the persistent loops: one per XCD, each in a memory channel
// of its own.  In one cache line all XCDs' claims took turns, some 15 ns each
// (195,112 particles FP64, 12,200 claims a loop: forces 290 -> 178 us, density
// 264 -> 215 us; 2.1M: forces 1.87 -> 1.76 ms).
constexpr int kWorkStride = 64;
// d_work: the claim counters of a loop's two launches, then the heavy leaves' counts
// of the density and the force loop.
constexpr int kWorkWords = (2 * kXcds + 2) * kWorkStride;
inline unsigned pair_grid(int64_t n)
{
    int64_t blocks = (n + 7) / 8;
    blocks = blocks < kXcds ? kXcds : (blocks > kMaxPairBlocks ? kMaxPairBlocks : blocks);
    blocks = ((blocks + kXcds - 1) / kXcds) * kXcds;
    return (unsigned)blocks;
}

// log2 of the waves that share a home leaf of a set of n particles.  A wave is
// latency-bound, and a small set has fewer leaves than the chip has SIMDs (1,024),
// so up to some 4,500 waves, four per SIMD, share the leaves of a set: with a
// quarter of the home particles a wave has a quarter of the tests and of the
// Newton steps' sums per lane, but its own walk and its own staging of the same
// candidate leaves.  Whole leaves against this rule (density + forces, us):
// 1,000 particles FP64 85 + 37 / 39 + 29 (16 waves per leaf); 8,000 quintic FP64
// 765 + 218 / 276 + 107; a Plummer sphere of 12,000 FP64 4,650 + 170 / 1,640 +
// 101; 24,389 FP32-pair, forces 99 / 78.  The line: at twice as many, 46,656
// particles gain a third, but 32,768 on a lattice take 81 + 74 instead of 58 + 44,
// and a batch, which fills the chip anyway and whose sets are split as each is
// alone, loses 20 %.
constexpr int64_t kSplitParticles = 49152;
__host__ __device__ inline int split_of(int64_t n, int G)
{
    int k = 0;
    while ((2 << k) <= G && (n << (k + 1)) <= kSplitParticles) k++;
    return k;
}

// Density loop: FP32-pair in a periodic box keeps whole leaves.  Where a
// candidate leaf's shift is ambiguous its pairs' separations take another
// rounding, and whether it is depends on the largest h of the home particles
// that the wave holds, so shares would change results in their eighth digit.
__host__ __device__ inline bool splits_density(int precision, int periodic)
{
    return precision == SPH_FP64 || !periodic;
}

// FP32-pair density: where a reach and a leaf span half the box, the image of a pair
// is not that of its leaf, the products of the search cannot be formed and list every
// candidate.  Such groups are tested lane by lane as in FP64; lists of all candidates
// overflowed, and every Newton step swept again (2,500 particles at random 1,285 us,
// lane by lane 290; 2,197 on a lattice with the quintic kernel 887 and 226).  The
// line: guesses of h three times too large make 10,000 particles such a set (6,970 and
// 1,740 us) and 40,000 not; the variant's registers cost 4,194,304 particles 2.5 %, and
// 12,167 nothing.
constexpr int64_t kLanewiseParticles = 32768;
inline bool lanewise_density(int64_t n, int precision, int periodic)
{
    return precision == SPH_FP32_PAIR && periodic && n <= kLanewiseParticles;
}

// Whether a loop leaves its heavy home leaves (kHeavyLeaves) to a second launch with
// a wave for each of their particles: isolated sets of whole leaves, whose outermost
// particles' supports can hold thousands of others.  Not in a periodic box, where
// the launch would cost each loop 3-5 us: its sets are mostly near their mean density
// throughout, and only a void's particles whose supports reach a cluster (25,000
// particles, sigma 0.02 of the box: 11,900 neighbours) would gain.  Not in sets whose
// leaves are shared, down to 2 of 16 particles per wave: they keep the tail that is
// left (12,000 Plummer FP64 1.4 ms against 1.1 ms of 30,000).
//
// kHeavyBlocks: two per SIMD.  One, two, four: 150,000 particles with guesses of h
// three times too large 23, 15, 11.5 ms; the forces of 150,000 quintic ones 1.92, 1.63,
// 1.53; sets without a heavy leaf 0, 0 and 3 us more per loop.
constexpr unsigned kHeavyBlocks = 2048;
inline bool second_launch(int64_t n, int G, int periodic)
{
    return !periodic && split_of(n, G) == 0;
}

// log2 of the blocks that share the density lists of a whole leaf: half as many
// as share the leaf, so that a list holds whole steps of 4 entries per lane (a
// particle of its own wave has all 64).
__host__ __device__ inline int slice_split(int64_t n, int G, bool splits)
{
    const int k = splits ? split_of(n, G) : 0;
    return k > 0 ? k - 1 : 0;
}

// Density-loop candidate lists: up to Kern<K>::list entries per home
// particle (160 for the M4, whose sphere of radius 2 Rc holds ~90 neighbours
// at eta = 1.2; 480 for the quintic's ~300 within 3 Rc), each an FP64 r^2 and
// an FP64 mass, for the candidates within R Rc, Rc = kCacheGrow h (capped by
// the walk radius), so that Newton steps within that bound reuse them.  A
// block holds the lists of one leaf's G particles; with equal masses the masses'
// places hold r^2 too.
constexpr double kCacheGrow = 1.15;
inline int64_t cache_bytes(int G, int kernel, int64_t blocks)
{
    return blocks * 2 * (int64_t)kern_list(kernel) * G * (int64_t)sizeof(double);
}

// Tree node: bounding box of the particles below it, as centre and half
// extents (what the distance tests take; the half extents are rounded up so
// that the box holds its particles), and their largest h.  64 bytes, so one
// node is half a 128-byte cache line.
struct alignas(64) Node {
    double c[3];
    double hmax;
    double e[3];
    double pad;
};

// The node of the box [lo, hi]: half extents to the farther side, with a few
// units in the last place of the coordinates on top.
__device__ inline void set_box(Node &nd, const double lo[3], const double hi[3])
{
    for (int a = 0; a < 3; a++) {
        nd.c[a] = 0.5 * (lo[a] + hi[a]);
        const double e = fmax(hi[a] - nd.c[a], nd.c[a] - lo[a]);
        nd.e[a] = e + 1e-15 * (fabs(nd.c[a]) + e);
        // a box of nothing (no finite position): infinitely far from anything,
        // and without effect on the box of its parent
        if (!(hi[a] >= lo[a])) {
            nd.c[a] = 0.0;
            nd.e[a] = -INFINITY;
        }
    }
}

// Tree description, written on the device by the build (the leaf count is
// data dependent) and read by every pair kernel.
struct TreeInfo {
    int32_t nlev;                  // levels including the leaf level (level 0)
    int32_t leaf_size;
    int64_t n;                     // particles
    int64_t off[kMaxLevels];       // first node of each level in the node array
    int64_t cnt[kMaxLevels];       // nodes per level (cnt[0] = leaves)
};
constexpr int kTreeWords = (int)(sizeof(TreeInfo) / 8);

struct Box {
    int32_t periodic;
    double lo[3];
    double len[3];                 // periodic box lengths
    double half[3];                // len / 2
};

// Device status word: [0] flags, [1] h solves not converged, [2] non-finite
// results, [3] periodic 2h >= L/2, [4] walk overflows (slow path taken),
// [5] max Newton-Raphson iterations, [6..7] spare.
enum : int32_t {
    kFlagNotConverged = 1,
    kFlagNonFinite = 2,
    kFlagStencil = 4,
    kFlagLevel = 8,     // block time-steps: a level deeper than the timeline allows
};
constexpr int kStatusWords = 8;

// Device counters of the last evaluation.  [0, 1] are written by the
// conserved-quantity reduction; the density loop zeroes and fills
// [kCntDensFirst, kCntDensFirst + kCntDensWords), the force loop
// [kCntForceFirst, kCntForceFirst + kCntForceWords).  They stand in kCountRows
// rows that different blocks add to, and a counter is the rows' sum (the
// largest of them for kCntNrMax): atomics on one cache line take turns, and each
// block ends with about ten (1,000 particles as 1,008 waves: density 53 -> 37 us
// with 64 rows, forces 36 -> 30 us).
enum : int {
    kCntNngb = 0,            // sum of density neighbour counts
    kCntNforce = 1,          // sum of force neighbour counts
    kCntDensEvals = 2,       // density pairs evaluated, all Newton-Raphson iterations
    kCntNrMax = 3,           // largest Newton-Raphson iteration count of a wave
    kCntDensOverflows = 4,   // density walks that overflowed the LDS frontier
    kCntDensVisits = 5,      // candidate leaves staged by density sweeps
    kCntDensWalks = 6,       // density tree walks
    kCntNrTotal = 7,         // density evaluations summed over particles
    kCntDensTests = 8,       // particle-candidate distance tests, density
    kCntDensBoxes = 9,       // particle-leaf box tests, density
    kCntForceEvals = 10,     // force pairs evaluated
    kCntForceOverflows = 11, // force walks that overflowed the LDS frontier
    kCntForceTests = 12,     // particle-candidate distance tests, force
    kCntForceBoxes = 13,     // particle-leaf box tests, force
    kCntDensListOverflows = 14, // particles whose candidate list outgrew its capacity in a sweep
    kCountWords = 16,
    kCountRows = 64,
    kCntDensFirst = kCntDensEvals,
    kCntDensWords = kCntDensBoxes - kCntDensEvals + 1,
    kCntForceFirst = kCntForceEvals,
    kCntForceWords = kCntForceBoxes - kCntForceEvals + 1,
};

// What the force loop reads of every neighbour j, in one 64-byte line:
// c_j, 1/h_j, v_j, m_j, A_j = P_j / (Omega_j rho_j^2) and rho_j.
struct alignas(64) ForceRec {
    double c, hinv, vx, vy, vz, m, A, rho;
};

// FP32-pair mode: the same record rounded to single precision (32 bytes), so
// the force loop's pair terms read half the bytes and convert nothing.  The
// home particle's values are rounded the same way, so the (j, i) pair sees
// exactly the values of the (i, j) pair.
struct alignas(32) ForceRec32 {
    float c, hinv, vx, vy, vz, m, A, rho;
};

// A particle's position as the pair loops' candidate loads read it: FP64, or
// in FP32-pair mode the single-precision offset from the centre of its leaf.
// One record per particle, which also carries the squared gather reach (R h)^2
// once the force records are written.
struct alignas(32) Pos4 {
    double x, y, z, reach2;
};
struct alignas(16) Off4 {
    float x, y, z, reach2;
};
static_assert(sizeof(Pos4) == sizeof(ForceRec32), "they share memory");

// Arrays in sorted order (along the Hilbert or Morton curve).
struct Sorted {
    double *x = nullptr, *y = nullptr, *z = nullptr;
    double *vx = nullptr, *vy = nullptr, *vz = nullptr;
    double *m = nullptr, *u = nullptr, *h = nullptr;
    double *rho = nullptr, *omega = nullptr;
    ForceRec *frec = nullptr;                  // force record
    ForceRec32 *frec32 = nullptr;              // its single-precision copy (FP32-pair)
    double *ax = nullptr, *ay = nullptr, *az = nullptr, *du = nullptr;
    double *vsig = nullptr, *dt = nullptr;
    int32_t *nngb = nullptr, *nforce = nullptr;
    uint32_t *id = nullptr;                    // original (caller) index
    // resident-state integration arrays
    double *vpx = nullptr, *vpy = nullptr, *vpz = nullptr, *up = nullptr;
    // artificial-viscosity switches: alpha (state), its predictor and rate
    // (MM97), div v of the previous step (CD10); div v and |curl v| outputs
    double *al = nullptr, *alp = nullptr, *adot = nullptr, *dprev = nullptr;
    double *divv = nullptr, *curlv = nullptr;
    // block time-steps: level, step start and end (ticks), half-step v and u
    // (and alpha under MM97), the active flag and the limiter's neighbour
    // level and wake-up mark of the current sub-step
    int32_t *lev = nullptr;
    int64_t *ts = nullptr, *te = nullptr;
    double *vhx = nullptr, *vhy = nullptr, *vhz = nullptr, *uh = nullptr, *alh = nullptr;
    int32_t *act = nullptr, *lmx = nullptr, *mark = nullptr;
    // candidate positions of the pair loops, written by the tree build:
    // FP32-pair offsets, or FP64 positions, which share the memory of the
    // single-precision records (only FP32-pair mode has those)
    Off4 *off = nullptr;
    Pos4 *pos() const { return (Pos4 *)frec32; }
};

// Device clock of the block time-steps (one level-0 step = 2^lmax ticks).
struct BlockClock {
    int64_t T;          // current tick within the level-0 step
    int64_t Tn;         // tick of the sub-step in progress
    int64_t full;       // level-0 steps completed
    int64_t nsub;       // sub-steps taken
    int64_t active;     // active particles of the last sub-step
    int64_t updates;    // active particles summed over the sub-steps
    double tick;        // time per tick of the current level-0 step
    double tick_next;   // time per tick of the next one (set at a full sync)
    double time;        // elapsed time
    double dt_max;      // length of the current level-0 step
    double dt_max_next; // of the next one (set at a full sync)
    int64_t pad[5];
};

struct Timer {
    bool on = false;
    double ms[3] = {0, 0, 0};
    int64_t launches[3] = {0, 0, 0};
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pending[3];
    std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
};

} // namespace sph

struct sph_ctx {
    sph_params p{};
    hipStream_t stream = nullptr;
    int device = 0;
    size_t budget = 0;
    size_t bytes = 0;
    std::string err;

    // capacity of the per-particle buffers
    int64_t ncap = 0;
    int64_t n = 0;
    std::vector<void *> allocs;          // everything sized by ncap

    // build
    uint64_t *keys[2] = {nullptr, nullptr};
    uint32_t *vals[2] = {nullptr, nullptr};
    uint32_t *hist = nullptr;
    int64_t hist_cap = 0;
    uint32_t *perm = nullptr;            // sorted position -> source index
    double *d_box = nullptr;             // [lo0..2, hi0..2] on device
    double *d_part = nullptr;            // reduction partials
    sph::Node *nodes = nullptr;
    int64_t node_cap = 0;
    sph::TreeInfo *d_tree = nullptr;    // device-resident tree description
    uint32_t *lstart = nullptr;         // leaf -> first sorted particle, [L+1]
    uint32_t *d_work = nullptr;         // per-XCD claim counters of the pair kernels
    double *cache = nullptr;            // density-loop candidate lists, a slice per pair-kernel block
    int64_t cache_size = 0;             // its bytes (cache_bytes(G, 1) per block at leaf size G)
    void *d_dargs = nullptr;            // device argument block of the density loop
    void *d_fargs = nullptr;            // device argument block of the force loop
    uint64_t *skeys = nullptr;          // sorted keys of the last build
    uint32_t *scratch_u32 = nullptr;    // per-particle scratch (free sort buffer)
    int64_t tree_n = -1;                // n of the tree on the device (-1: none)
    sph::Box box{};

    sph::Sorted s;       // working / resident arrays
    sph::Sorted t;       // alternate buffers for re-sorting the resident state

    // identity of the arrays the current structure was built from
    const double *built_x = nullptr;
    int64_t built_n = -1;
    bool built = false;

    // resident state
    bool resident = false;
    bool res_alpha = false;     // the resident state carries per-particle alpha
    sph::BlockClock *d_clock = nullptr;   // block time-steps (device)
    int32_t *leaf_act = nullptr;     // active particles per leaf of the current sub-step
    // the leaves with an active particle, in leaf order, and their number (on
    // the device): the home leaves of the pair loops in a sub-step; per-tile
    // counts, then offsets, of the compaction that lists them
    uint32_t *act_list = nullptr, *act_tile = nullptr, *act_cnt = nullptr;
    double *d_scal = nullptr;   // [0] dt_next [1] dt_last [2] time [3] KE [4] TE [5..7] P
                                // [8] smallest, [9] largest mass of the last density pass
    // device counters, indexed by the kCnt* constants
    int64_t *d_counts = nullptr;
    double *h_scal = nullptr;   // pinned mirror
    int64_t *h_counts = nullptr;   // pinned mirror of d_counts
    sph::BlockClock *h_clock = nullptr; // pinned mirror of d_clock
    double *dt_used_out = nullptr;
    int64_t steps = 0;

    int32_t *d_status = nullptr;
    int32_t *h_status = nullptr;   // pinned mirror

    // captured pair of resident steps
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    double graph_dt = 0.0;

    sph::Timer timer;
    bool count_tests = false;   // pair loops also count box and candidate tests

    // per-call active set of the pair loops (block time-steps; nullptr: every
    // particle) and the force loop's limiter outputs
    const int32_t *f_act = nullptr;
    bool f_block = false;

    // per-call inputs of the force loop: the sorted per-particle alpha it
    // uses (nullptr: alpha_av for every pair), whether it writes div v and
    // |curl v| (set by the phase functions before forces_prepare)
    const double *f_alpha = nullptr;
    bool f_div = false;

    // this device's copy of the library's static scratch array (the
    // no-allocation entry point); nullptr if its address could not be taken
    void *static_scratch = nullptr;
    std::string static_err;
};

namespace sph {

// ---- host helpers (api.hip) --------------------------------------------------
sph_status fail(sph_ctx *c, sph_status s, const std::string &msg);
sph_status hip_check(sph_ctx *c, hipError_t e, const char *what);
sph_status ensure_capacity(sph_ctx *c, int64_t n);

// ---- build.hip ---------------------------------------------------------------
// Bounding box, keys, sort: fills c->perm (sorted -> source) for n positions.
// `state`: the positions of a resident state (they keep the Morton order).
sph_status build_order(sph_ctx *c, int64_t n, const double *x, const double *y,
                       const double *z, bool state);
// Gather `count` arrays through c->perm: dst[k] = src[perm[k]].
struct GatherList {
    int32_t count;
    int32_t kind[32];        // 0: 8-byte word, 1: uint32, 2: float
    const void *src[32];
    void *dst[32];
};
sph_status gather(sph_ctx *c, int64_t n, const GatherList &g, bool identity_src_index);
// Leaf boxes and tree over c->s.{x,y,z,h}; FP32 offsets when requested.
sph_status build_tree(sph_ctx *c, int64_t n);
// leaf and node hmax from the current sorted h (after the h solve), boxes kept
sph_status refresh_hmax(sph_ctx *c, int64_t n);
// Force records from rho, omega, h, m and the given sorted u and velocities; hmax:
// and the leaves' and nodes' largest h from the current h (after the h solve).
sph_status force_prep(sph_ctx *c, int64_t n, const double *u_sorted, const double *vx,
                      const double *vy, const double *vz, bool hmax);
sph_status iota(sph_ctx *c, int64_t n, uint32_t *v);
int64_t node_count_bound(int64_t n);

// ---- pairs.hip (dispatch) and pairs.hpp (kernels) -------------------------
sph_status run_density(sph_ctx *c, int64_t n);
sph_status run_forces(sph_ctx *c, int64_t n);
// batched pair loops: prepare writes each set's argument block on its
// stream; launch runs one persistent kernel over cs[0..count) (same stream,
// precision and leaf size)
sph_status density_prepare(sph_ctx *c, int64_t n);
sph_status forces_prepare(sph_ctx *c, int64_t n);
sph_status density_launch(sph_ctx *const *cs, int count, int64_t nmax);
sph_status forces_launch(sph_ctx *const *cs, int count, int64_t nmax);
// meshless finite-volume gradient matrix and gradients over the built tree,
// with h and the number density (c->s.rho) already solved; sorted arrays
sph_status run_mfv(sph_ctx *c, int64_t n, int nf, const double *const *f, double *const *B,
                   double *cond, double *const *grad);
sph_status run_neighbours(sph_ctx *c, int64_t n, int32_t mode, int64_t *counts_sorted,
                          const int64_t *offsets_sorted, int32_t *idx, int64_t cap);

// ---- step.hip ----------------------------------------------------------------
// scatter sorted arrays back to caller order through c->perm
struct ScatterList {
    int32_t count;
    int32_t kind[32];
    const void *src[32];
    void *dst[32];
};
sph_status scatter(sph_ctx *c, int64_t n, const ScatterList &s, const uint32_t *index);

// dst[a][to] = src[a][from] for every array of a Gather/ScatterList, copied as
// bits (8 bytes for kind 0, 4 otherwise).  Up to 16 loads are issued before
// their stores: the lists carry no no-alias guarantee, so a load after a store
// would wait for it, and a one-array-at-a-time loop runs ~10 dependent memory
// round trips per element.
template <class List>
__device__ inline void copy_listed(const List &L, int64_t from, int64_t to)
{
    constexpr int kChunk = 16;
    for (int a0 = 0; a0 < L.count; a0 += kChunk) {
        uint64_t v[kChunk];
#pragma unroll
        for (int j = 0; j < kChunk; j++) {
            const int a = a0 + j;
            if (a < L.count)
                v[j] = L.kind[a] == 0 ? ((const uint64_t *)L.src[a])[from]
                                      : (uint64_t)((const uint32_t *)L.src[a])[from];
        }
#pragma unroll
        for (int j = 0; j < kChunk; j++) {
            const int a = a0 + j;
            if (a < L.count) {
                if (L.kind[a] == 0) ((uint64_t *)L.dst[a])[to] = v[j];
                else ((uint32_t *)L.dst[a])[to] = (uint32_t)v[j];
            }
        }
    }
}
sph_status eos_scatter(sph_ctx *c, int64_t n, const uint32_t *index, const double *u_caller,
                       double *P, double *cs);
// scatter plus the equation of state (P, cs may be NULL) from sorted rho, u
sph_status scatter_eos(sph_ctx *c, int64_t n, const ScatterList &s, const uint32_t *index,
                       const double *u_sorted, double *P, double *cs);
sph_status kick_drift(sph_ctx *c, int64_t n, double dt_host);
sph_status closing_kick(sph_ctx *c, int64_t n, double dt_host);
// artificial-viscosity switches on the resident state: MM97 rate adot from
// the predicted alpha and the latest div v; CD10 update of alpha (and
// dprev = div v) with the step length on the device
sph_status av_rate(sph_ctx *c, int64_t n, const double *alpha_now);
sph_status av_cd10(sph_ctx *c, int64_t n, bool first);
sph_status fill(sph_ctx *c, int64_t n, double *v, double value);
// block time-steps on the resident state (step.hip)
sph_status block_next(sph_ctx *c, int64_t n);           // Tn = min te; drift every particle
sph_status block_predict(sph_ctx *c, int64_t n);        // predictors, active set, leaf counts
sph_status block_finish(sph_ctx *c, int64_t n, bool init);  // close, levels, limiter, open, clock
sph_status block_av(sph_ctx *c, int64_t n);             // switches of the active particles
// smallest and largest sorted mass per block -> d_part[2b], d_part[2b + 1]
sph_status reduce_mass_range(sph_ctx *c, int64_t n, int *blocks);
// conserved quantities and neighbour counts; with_dt: and min dt -> d_scal[0]
sph_status reduce_diag(sph_ctx *c, int64_t n, bool with_dt);
// zero the per-XCD claim counters of the persistent pair kernels
sph_status zero_work(sph_ctx *c);
// exclusive prefix sum in place over a[0..n], treating a[n] as 0 on input
sph_status scan_offsets(sph_ctx *c, int64_t n, int64_t *a);

// timing
void timer_begin(sph_ctx *c, int which, hipEvent_t *b, hipEvent_t *e);
void timer_end(sph_ctx *c, int which, hipEvent_t b, hipEvent_t e);

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

} // namespace sph
