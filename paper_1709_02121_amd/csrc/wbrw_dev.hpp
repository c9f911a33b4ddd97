// Device-side data layout of the WBRW library.
//
// Particles of all instances live in one structure of arrays; instance b owns
// the segment [base_b, base_b + cap_b).  Two such sets exist and annihilation
// writes the regenerated ensemble into the inactive one ("cur" flips).  All
// mutable bookkeeping (counts, tile plans, tickets, look-back status words,
// tallies, the step counter) is device resident, so a step or an epoch can be
// enqueued, or captured into a hipGraph, without host round trips.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace wbrw {

constexpr int kMaxM = 4;
constexpr int kThreads = 256;           // threads per block in every kernel
constexpr int kPPT = 8;                 // particles (or cells) per thread in the passes over all of them
constexpr int kTileA = kThreads * kPPT; // particles per tile of those passes
constexpr int kParents = 32;            // fewest event parents taken at a time (see Dev::ftile)
constexpr int kTileS = kThreads * kPPT; // cells per scan tile
constexpr int kSupGroup = 64;           // walk tiles per group sum of their counts
constexpr int kXcd = 8;                 // accelerator complexes (XCDs), each with its own L2
constexpr int kTileR = kThreads * 4;    // regenerated particles per tile
constexpr int kMaxDepth = 16;           // deepest family tree walked within one step
constexpr uint32_t kEventCap = 4096u;   // jumps per particle-step
constexpr int kXiN = 4096;              // xi(r) grid intervals (Alg. 4 sampler)
constexpr int kXiQ = 8192;              // quadrature nodes for xi(r)
constexpr uint32_t kRejectMax = 256u;   // rejection proposals per kick
constexpr int kChunk = 5;               // steps in one launch of k_walk, at most
constexpr int kClasses = 1 << kChunk;   // sets of steps in which an offspring and its ancestors were born
constexpr int kPend = 32;               // steps between materialisations of the positions, at most
constexpr int kRangeMin = 64;           // particles in a tile of k_walk, at least; a multiple of 64
constexpr int kRangeMax = 8192;         // particles in a tile of k_walk, at most
constexpr int kLocalBits = 4096;        // offspring of a tile whose event bits are kept in LDS
constexpr int kDirect = 23;             // pages of a tile's offspring that the tile itself lists
constexpr int kPages = kDirect + 1;     // their entries, and where the table of further pages starts
constexpr int kTableMin = 64;           // pages that such a table holds, at least
constexpr int kTableShare = kRangeMin / 8;  // entries of such tables for each possible tile
constexpr int kFewInst = 8;             // instances whose class totals are summed from the tiles'
constexpr int kMaxGrid = 8192;          // blocks of a persistent launch (per-block partials)
// 4D family kernels: the payloads of a tile's records beyond the block's LDS
// pool go to a per-block overflow area in HBM (kGPool records for each of the
// first kGPoolBlocks blocks).  Per record: eight doubles (x0, k0, x1, k1, w
// and three tangents), the id and the sign.
constexpr int kGPool = 1024;
constexpr int kGPoolBlocks = 1024;
constexpr size_t kGPoolBytes = (size_t)kGPool * (8 * 8 + 8 + 1);

enum : uint32_t { kErrCapacity = 1u, kErrDepth = 2u, kErrRange = 4u };

// tally slots per instance
enum : int {
    kTalEvents = 0, kTalPairs, kTalKilled, kTalEscaped, kTalMaxDepth, kTalEventCap,
    kTalSplus, kTalSminus, kTalNplus, kTalNminus, kTalPSteps, kTalAnn, kTalTrig, kTalCount = 16
};

// ticket counters of the persistent passes
enum : int {
    kPassFamily = 1, kPassFamilyG = 3, kPassGhost = 7, kPassCount = 8
};

struct InstParam {
    double gamma0;
    double thr_lo, thr_hi;          // certain-jump / certain-no-jump band on the first uniform
    uint32_t ib_lo, ib_hi;          // the same on its high word: jump if below ib_lo, none above ib_hi
    int32_t wr, gwr;                // most particles (ghosts) in a tile of k_walk
    int32_t wt, gwt;                // tiles to cut the instance into where that leaves fewer
    double c[kMaxM];                // xi_m / (2 gamma0)
    double sq[kMaxM];               // Gaussian kick std 1/(2w)
    double H[kMaxM], width[kMaxM];  // Gaussian parameters (tangent scores)
    double center[kMaxM];           // centre of the kernel phase
    double sgnV[kMaxM];             // sign of F[V_m]
    double xi_h[kMaxM];             // Alg. 4 sampler: xi grid spacing in |x - x0|
    double ma[kMaxM], mb[kMaxM];    // time-varying height factor a + b cos(omega t + phase)
    double mw[kMaxM], mp[kMaxM];
    int64_t base, cap;              // particle segment
    int64_t gbase, gcap;            // ghost segment
    int64_t N0;                     // sample size N_alpha
    int64_t rbase, rtiles;          // this instance's slots in Dev::rstart
    uint32_t key;                   // Philox key word 1
    uint32_t pad;
};

// A bucket of a table's guide: the bins [lo, hi] that its draws can fall in
// and the cumulative sum at the start of bin lo + 1, which decides between
// two of them.
struct GuideEntry {
    int32_t lo, hi;
    double next;
};

struct Table {
    const double *cum;        // n + 1 cumulative sums of |F[V](2q_j)|
    const GuideEntry *guide;  // kg buckets: lo of bucket i is the last bin j < n with
                              // cum[j] <= (i / kg) cum[n] (as the sampler rounds it)
    int32_t n;
    int32_t kg;               // guide buckets, a power of two >= n
    double q_lo, dq;
    double total;             // cum[n]
};

struct Ens {
    double *x0, *x1, *k0, *k1;
    int8_t *sg;
    double *w;
    uint64_t *id;
    double *D;     // planar [3][cap_total]
};

struct Ctl {
    uint32_t step;             // steps completed (Philox counter word 2)
    uint32_t cur;              // active real buffer set
    uint32_t gcur;             // active ghost buffer set
    uint32_t err;              // sticky error bits
    uint32_t ann_seq;          // annihilations so far (look-back epoch of the scans)
    uint32_t ann_now;          // conditional annihilation: the one after this step runs
    uint32_t chunk;            // chunks of steps so far: its parity picks the tile plan and group sums
    uint32_t wpar;             // parity of the chunk that k_place closes
    uint32_t table[2];         // entries of ptx and ptxg handed out (zero between chunks)
    uint32_t fill[22];         // the counters below start a line of their own: their
                               // atomics do not hold up the reads of the words above
    uint32_t ticket[kPassCount];   // zero between launches (see next_tile)
};

struct Dev {
    const Dev *self;            // a copy of this structure in device memory
    // sizes and constants
    int32_t B, dim, M, strategy, tangent;
    int32_t tdep;               // some Gaussian height varies in time
    // conditional annihilation (wbrw_run_adaptive): the step's closing kernel
    // sets ctl->ann_now when the step count is a multiple of ann_every or an
    // instance holds more than ann_limit particles, and with cond_ann set the
    // annihilation kernels run only then
    int32_t cond_ann, ann_every;
    int64_t ann_limit;
    double hbar;
    int32_t nx, nk;
    uint32_t seed;
    int64_t Nh;                 // cells per instance
    int64_t cap_total, gcap_total;
    double dt, vfac;
    double x_lo, x_hi, k_lo, k_hi, dx, dk;
    double rdx, rdk;            // 1/dx and 1/dk, rounded (see axis_cell)
    int32_t kind[kMaxM], axis[kMaxM], sampler[kMaxM];
    int32_t ftile, gftile;      // event parents that k_walk takes at a time (particles, ghosts):
                                // as many as kThreads, fewer where their records (see
                                // Families) would not fit the pool or queue
    const double *xi_tab;       // [B][M][kXiN + 1] xi(r) tables of the Alg. 4 sampler
    Table tab[kMaxM];
    // buffers
    Ens ens[2], gens[2];
    const InstParam *ip;
    Ctl *ctl;
    int64_t *N, *NG, *Nnew, *NGnew;
    int64_t *Nbase;             // [2][B] counts at the start of the chunk (real, ghost): its records go after them
    int64_t *nstep;             // [2][B][kPend + 1] counts at the start of every step since the
                                // positions were materialised (real, ghost); entry 0 always holds
    int64_t *tileA;             // [2][B+1] plan of those tiles (real, ghost)
    int64_t *tileW;             // [2][2][B+1] walk-tile plan (parity; real, ghost)
    int64_t *wrange;            // [2][2][B][2] its particles per tile, and the binary logarithm
                                // of the slots of a page (see page_slot)
    uint64_t *wpool;            // [2][B] slots handed out as further pages (zero between chunks)
    uint32_t *ptab, *ptabg;     // per walk tile: its kPages entries (see page_slot)
    uint32_t *ptx, *ptxg;       // behind them: tables of the tiles with more than kDirect pages
    int64_t *tileR;             // [B+1] regeneration-tile plan
    int64_t *tileG;             // [B+1] ghost-regeneration plan
    int64_t *tally;             // [B][kTalCount]
    int64_t *fpart;             // [kMaxGrid][8]: instance and tallies of each walking block
    char *gpool;                // [gpool_blocks][kGPoolBytes] (4D only, else null)
    int32_t gpool_blocks;
    int64_t *rstart;            // first cell of every regeneration tile (written by k_scan)
    uint64_t *stS;              // scan-tile sums of |n_nu|, then their exclusive prefix
    uint64_t *stG;              // look-back status words of k_ghosts
    uint16_t *smask, *smaskg;           // per slot of the tiles' pages: the offspring's class, and
                                        // from bit kChunk on the chunk's steps in which it jumps
    uint32_t *wcnt, *wcntg;             // per walk tile: records of each class
    uint32_t *wsup, *wsupg;             // [2] (parity) per kSupGroup walk tiles: their sums
    int64_t wsup_g, wsup_gg;            // groups of one parity
    uint32_t *wtot;                     // [2][B][kClasses] records of each class (more than
                                        // kFewInst instances; zero between chunks)
    int32_t *cnt;               // [B][Nh] signed counts (sp1) / rounded counts (sp2)
    int32_t *cntx;              // partial counts of the blocks on the other XCDs (copy 0
                                // is the grid itself): sp1 [kXcd - 1][B][Nh] of cnt, sp2
                                // [kXcd - 1][2][B][Nh] of ntil; null when not used
    int64_t *off;               // [B][Nh] exclusive prefix of |n_nu|, bit 62 = negative cell
    int32_t *occ;               // [B][Nh] occupancy (tangents)
    int64_t *Tq;                // [B][Nh][6] tangent sums per cell in 32.32 fixed point
                                // (see fx_split), high and low words; a cell in one or two lines
    int32_t *occx;              // with tangents: [kXcd - 1][B][Nh] XCD copies of occ,
    int64_t *Tqx;               // and [kXcd - 1][B][Nh][6] of Tq (see cntx); else null
    int32_t *ntil;              // [2][B][Nh] sp2 bootstrap counts per class
    int64_t *dacc;              // [kXcd][B][max_bins] density accumulator, one per XCD
                                // (a block flushes into copy blockIdx mod kXcd)
    int64_t *dTq;               // [B][6][max_bins] tangent density sums (fixed point, as Tq)
    int32_t max_bins;
    // sp2 bootstrap scratch
    uint64_t *bA;               // [cap_total] quantised weight, then the residual
    int32_t *bcopies;           // [cap_total] copies per particle
    int8_t *bcls;               // [cap_total] class (0 +, 1 -, -1 none)
    int32_t *bcell;             // [cap_total] cell or -1
    uint64_t *bP;               // [2][cap_total] 128-bit residual prefix (lo, hi interleaved)
    uint64_t *bTile;            // [2][tiles] 128-bit tile sums
    int32_t *bG;                // [2][4 cap_total] draw guide per class, four
                                // slots per particle slot (sp2_guide_bits)
    int64_t *bcls_stat;         // [B][8]: N+, N-, S+, S-, sumk+, sumk-, Nr+, Nr-
    int64_t *tileD;             // [2][B+1] draw-tile plan (per class)
    int64_t *bscan_tiles;       // [B+1] tiles per instance for the residual scan
    int64_t tstride;            // tiles per class in bTile
};

// Pages.  A tile's offspring wait in the inactive buffer set for their places
// in pages of 2^sh slots, the largest power of two up to half a tile's range:
// tile tl of the instance has the page at tl 2^sh, and takes further ones
// from the slots behind all first pages as it grows.  T first pages take at
// most (N + R) / 2 slots, and a tile that takes further ones has fewer slots in
// them than offspring, so whatever the tiles' shares and however far they
// grow, the pages fit where the offspring will fit behind the N > R particles.
// A single tile has all slots.
//
// The first kDirect pages are listed with the tile, all others in a table of
// its own in ptx, which is replaced by one of twice the size when it is full.
// The tables that a tile has had are less than four entries for each of its
// pages, and pages have 32 slots or more: an eighth of the slots is room for
// all of them.
__host__ __device__ __forceinline__ int32_t page_bits(int64_t range, int64_t tiles)
{
    if (tiles <= 1) return 31;
    int32_t sh = 5;
    while ((int64_t)(4 << sh) <= range) ++sh;
    return sh;
}
// entries of the table of a tile with np pages
__host__ __device__ __forceinline__ uint32_t page_table(int np)
{
    if (np <= kDirect) return 0u;
    uint32_t n = kTableMin;
    while (n < (uint32_t)(np - kDirect)) n <<= 1;
    return n;
}
// slot (from the instance's first) of offspring l; more(): ptx or ptxg
template <class F>
__host__ __device__ __forceinline__ int64_t page_slot(const uint32_t *pages, int sh, uint32_t l, F more)
{
    const uint32_t p = l >> sh;
    uint32_t first = pages[p < (uint32_t)kDirect ? p : (uint32_t)kDirect];
    if (p >= (uint32_t)kDirect) first = more()[first + (p - (uint32_t)kDirect)];
    return first + (l - (p << sh));
}

// Particles in a tile of k_walk for an ensemble of n: an equal share of a
// whole multiple of `tiles` tiles, those of one round (see set_tiles), so that
// the blocks that run at once all take the same number of tiles; rounded up
// to kRangeMin, at most `most`.
__host__ __device__ __forceinline__ int64_t walk_range(int64_t n, int32_t tiles, int32_t most)
{
    const int64_t waves = (n + (int64_t)tiles * most - 1) / ((int64_t)tiles * most);
    const int64_t t = (waves < 1 ? 1 : waves) * tiles;
    const int64_t r = ((n + t - 1) / t + kRangeMin - 1) / kRangeMin * kRangeMin;
    return r < kRangeMin ? kRangeMin : (r > most ? most : r);
}
// Synchronises the block.  The wait is spelt out: a barrier at the top of a
// loop can lose the one that its fence asks for, where nothing is under way
// before the loop but LDS operations of the loop's end are (the pass that
// places waits drops it on its first visit and does not put it back when it
// comes round).  Wavefronts then read what others had yet to write: the cell
// pass lost a few hundred of 2e7 particles in one annihilation of fifty.
__device__ __forceinline__ void block_sync()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
}

// The same where only LDS is shared: stores to global memory may still be
// under way.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// An annihilation kernel enqueued after a step of wbrw_run_adaptive does
// nothing unless that step's closing kernel asked for the annihilation.
__device__ __forceinline__ bool ann_skipped(const Dev &d)
{
    return d.cond_ann && d.ctl->ann_now == 0u;
}

__device__ __forceinline__ Ens pick_set(const Dev &d, int ghost, uint32_t which)
{
    if (ghost) return which ? d.gens[1] : d.gens[0];
    return which ? d.ens[1] : d.ens[0];
}

// segment b with plan[b] <= t < plan[b+1]
__device__ __forceinline__ int segment_of(const int64_t *plan, int B, int64_t t)
{
    int lo = 0, hi = B - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (plan[mid] <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Tiles [a, c) as the tiles before the first whole group of kSupGroup, whole
// groups, and the tiles after the last: nh, ng and nt of them, from a, group
// ga / kSupGroup and gc on.
struct TileRange {
    int64_t a, ga, gc, nh, ng, nt;
    __device__ __forceinline__ TileRange(int64_t a_, int64_t c) : a(a_)
    {
        ga = (a + kSupGroup - 1) / kSupGroup * kSupGroup;
        gc = c / kSupGroup * kSupGroup;
        const bool groups = ga <= gc;
        nh = c <= a ? 0 : (groups ? ga - a : c - a);
        ng = groups ? (gc - ga) / kSupGroup : 0;
        nt = groups ? c - gc : 0;
    }
    __device__ __forceinline__ int64_t n() const { return nh + ng + nt; }
};

// ---- decoupled look-back (single-pass ordered scans) ----------------------
// status word: [epoch:30 | flag:2 | value:32]; flag 1 = tile aggregate, 2 = inclusive prefix
__device__ __forceinline__ void lb_publish(uint64_t *st, uint32_t epoch, uint32_t flag, uint32_t v)
{
    const uint64_t w = ((uint64_t)((epoch << 2) | flag) << 32) | (uint64_t)v;
    __hip_atomic_store(st, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wave-parallel look-back: the 64 lanes of one wavefront examine 64
// predecessors per round, wait until each has published, and sum back to the
// nearest inclusive prefix.  Returns the exclusive prefix to every lane.
__device__ __forceinline__ uint32_t lb_lookback_wave(uint64_t *st, int64_t t, int64_t first, uint32_t epoch)
{
    const int lane = threadIdx.x & 63;
    uint32_t excl = 0;
    for (int64_t top = t - 1; top >= first; top -= 64) {
        const int64_t p = top - lane;
        uint32_t flag = 2u, val = 0u;   // lanes past the segment start act as a zero prefix
        if (p >= first) {
            for (;;) {
                const uint64_t w = __hip_atomic_load(st + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t hi = (uint32_t)(w >> 32);
                if ((hi >> 2) == epoch && (hi & 3u) != 0u) {
                    flag = hi & 3u;
                    val = (uint32_t)w;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
            }
        }
        const uint64_t incl = __ballot(flag == 2u);
        const int stop = incl ? (__ffsll((unsigned long long)incl) - 1) : 64;
        uint32_t v = lane <= stop ? val : 0u;
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        excl += v;
        if (incl) break;
    }
    return excl;
}

// Publishes tile t's aggregate, looks back over its segment [first, t) and
// publishes its inclusive prefix.  Called by all lanes of wavefront 0.
__device__ __forceinline__ uint32_t tile_prefix(uint64_t *st, int64_t t, int64_t first, uint32_t epoch,
                                                uint32_t agg)
{
    const int lane = threadIdx.x & 63;
    if (t == first) {
        if (lane == 0) lb_publish(st + t, epoch, 2u, agg);
        return 0u;
    }
    if (lane == 0) lb_publish(st + t, epoch, 1u, agg);
    const uint32_t excl = lb_lookback_wave(st, t, first, epoch);
    if (lane == 0) lb_publish(st + t, epoch, 2u, excl + agg);
    return excl;
}

// Next tile of a persistent pass, for thread 0 of a block.  Every block
// draws until it gets a ticket >= ntiles, so one launch hands out exactly
// ntiles + gridDim.x tickets, and the block that draws the last of them
// clears the counter for the next launch (which sees it after the kernel
// boundary).  No block waits for the others at the end, and no device-wide
// fence is needed.  Work that needs every block's results runs in one extra
// block of the next launch.
__device__ __forceinline__ int64_t next_tile(uint32_t *ctr, int64_t ntiles)
{
    const uint32_t t = atomicAdd(ctr, 1u);
    if ((int64_t)t == ntiles + (int64_t)gridDim.x - 1)
        __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return (int64_t)t;
}

// The same dispenser with every block's first tile given statically (block
// b takes tile b): when the tiles are about as many as the blocks, every
// block starts at once instead of queueing behind one atomic on one line
// (some 11 ns each).  With no more tiles than blocks no ticket is drawn at
// all; otherwise the counter hands out tiles gridDim.x, ...: each of those
// tickets is drawn once and every block draws one ticket past the end, so the
// block that draws ticket ntiles - 1 clears the counter.  `first` is the
// caller's flag, true on its first call.
__device__ __forceinline__ int64_t next_tile_static_first(uint32_t *ctr, int64_t ntiles, bool &first)
{
    const int64_t G = (int64_t)gridDim.x;
    if (first) {
        first = false;
        return (int64_t)blockIdx.x;
    }
    if (ntiles <= G) return ntiles;
    const uint32_t u = atomicAdd(ctr, 1u);
    if ((int64_t)u == ntiles - 1) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return G + (int64_t)u;
}

// Exclusive scan of the per-tile counts cnt[0..T) into pre[0..T) by one
// block (pre may be cnt); returns the total to every thread.  Chunks of
// kThreads x P counts are loaded coalesced (all loads in flight together)
// into LDS, padded by one slot per P so that the per-thread runs below fall
// in different banks; every thread scans its own run of P, the run totals are
// scanned within each wavefront and across the four wavefronts, and the
// prefixes leave LDS coalesced.
constexpr int kScanP = 24;
template <int P>
__device__ __forceinline__ uint64_t scan_chunks(const uint64_t *cnt, uint64_t *pre, int64_t T,
                                                uint64_t *s_v, uint64_t *s_w)
{
    constexpr int C = kThreads * P, W = kThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int run0 = tid * (P + 1);
    uint64_t carry = 0;
    for (int64_t c0 = 0; c0 < T; c0 += C) {
        const int n = (int)min((int64_t)C, T - c0);
        block_sync();
        uint64_t v[P], acc = 0;
#pragma unroll
        for (int r = 0; r < P; ++r)   // clamped, unconditional: no branch between the loads
            v[r] = cnt[c0 + min(r * kThreads + tid, n - 1)];
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int i = r * kThreads + tid;
            s_v[i + i / P] = v[r];
        }
        block_sync();
#pragma unroll
        for (int r = 0; r < P; ++r) {
            v[r] = tid * P + r < n ? s_v[run0 + r] : 0ull;
            acc += v[r];
        }
        uint64_t incl = acc;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint64_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) s_w[wv] = incl;
        block_sync();
        uint64_t below = 0, chunk = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const uint64_t t = s_w[w];
            below += w < wv ? t : 0ull;
            chunk += t;
        }
        uint64_t run = carry + below + (incl - acc);
#pragma unroll
        for (int r = 0; r < P; ++r) {
            s_v[run0 + r] = run;
            run += v[r];
        }
        block_sync();
#pragma unroll
        for (int r = 0; r < P; ++r) {
            const int i = r * kThreads + tid;
            if (i < n) pre[c0 + i] = s_v[i + i / P];
        }
        carry += chunk;
    }
    block_sync();
    return carry;
}

__device__ __forceinline__ uint64_t scan_tile_counts(const uint64_t *cnt, uint64_t *pre, int64_t T)
{
    __shared__ uint64_t s_v[kThreads * (kScanP + 1)];
    __shared__ uint64_t s_w[kThreads / 64];
    // a short list takes one small chunk: fewer loads and LDS passes per thread
    if (T <= kThreads * 4) return scan_chunks<4>(cnt, pre, T, s_v, s_w);
    return scan_chunks<kScanP>(cnt, pre, T, s_v, s_w);
}

// plan[b] = sum_{b' < b} value(b'), plan[B] = total; one block.  Values are
// scanned within each wavefront, then across the four wavefronts.
template <class F>
__device__ __forceinline__ void block_prefix(int64_t *plan, int B, F value)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (B == 1) {
        if (tid == 0) {
            plan[1] = value(0);
            plan[0] = 0;
        }
        block_sync();
        return;
    }
    __shared__ int64_t s_w[kThreads / 64];
    int64_t carry = 0;
    for (int c0 = 0; c0 < B; c0 += kThreads) {
        const int b = c0 + tid;
        const int64_t v = b < B ? value(b) : 0;
        int64_t incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        block_sync();
        if (lane == 63) s_w[wv] = incl;
        block_sync();
        int64_t below = 0, chunk = 0;
#pragma unroll
        for (int w = 0; w < kThreads / 64; ++w) {
            const int64_t t = s_w[w];
            below += w < wv ? t : 0;
            chunk += t;
        }
        if (b < B) plan[b] = carry + below + incl - v;
        carry += chunk;
    }
    if (tid == 0) plan[B] = carry;
    block_sync();
}

// plan[b] = sum_{b' < b} ceil(cnt[b'] / tile), plan[B] = total; one block.
__device__ __forceinline__ void block_plan(int64_t *plan, const int64_t *cnt, int B, int64_t tile)
{
    block_prefix(plan, B, [&](int b) { return (cnt[b] + tile - 1) / tile; });
}

// The tile plan of k_walk at chunk parity `par` for counts n[b]; one block.
__device__ __forceinline__ void plan_walk(const Dev &d, uint32_t par, int ghost, const int64_t *n)
{
    const int64_t at = 2 * par + (uint32_t)ghost;
    block_prefix(d.tileW + at * (d.B + 1), d.B, [&](int b) {
        const InstParam &P = d.ip[b];
        const int64_t r = ghost ? walk_range(n[b], P.gwt, P.gwr) : walk_range(n[b], P.wt, P.wr);
        const int64_t t = (n[b] + r - 1) / r;
        d.wrange[2 * (at * d.B + b)] = r;
        d.wrange[2 * (at * d.B + b) + 1] = page_bits(r, t);
        return t;
    });
}

// Tangent sums over cells and bins are exact integer sums in 32.32 fixed
// point, so that no summation order is singled out: a component D enters as
// q = trunc(D 2^32), which needs |D| < 2^31 (else, or for a NaN, it adds
// nothing and false is returned), split as hi = floor(q / 2^32) and
// lo = q mod 2^32.  Over at most 2^31 particles the high words sum to less
// than 2^62 and the low words to less than 2^63, so two 64-bit sums per
// component are exact without carries.
__device__ __forceinline__ bool fx_split(double D, int64_t &hi, uint64_t &lo)
{
    if (!(fabs(D) < 2147483648.0)) {
        hi = 0;
        lo = 0;
        return false;
    }
    const int64_t q = (int64_t)(D * 4294967296.0);
    hi = q >> 32;
    lo = (uint64_t)q & 0xFFFFFFFFull;
    return true;
}

// value of the sum with high-word sum hs and low-word sum ls:
// (double)floor(Q / 2^32) + (double)(Q mod 2^32) 2^-32, Q = hs 2^32 + ls
__device__ __forceinline__ double fx_value(int64_t hs, uint64_t ls)
{
    const int64_t h = hs + (int64_t)(ls >> 32);
    return (double)h + (double)(ls & 0xFFFFFFFFull) * 0x1p-32;
}

}  // namespace wbrw
