// Time steps of the Wigner branching random walk (Alg. 1, Sec. 2).
//
// Up to kChunk steps run in two launches.  Particles do not interact, and
// every draw is keyed by the particle's lineage id and the step, so a block
// takes a range of consecutive particles of an instance (a tile) through all
// steps of the chunk by itself, with the offspring born on the way:
//
// k_walk    reads the ids of the range and decides for every particle and
//           step whether it jumps (exact clocks for a constant gamma0, Sec.
//           3.2.1), keeping one bit each in LDS.  Then, step by step, it
//           gathers the jumping particles of the range and of its offspring,
//           in order, and takes their jumps (wbrw_step.hpp); where there are
//           few, generation by generation: the range's jumps in all steps,
//           then those of their offspring, and so on, by step and in order.
//           Offspring go to pages of the inactive buffer set, in order.
// k_place   puts the offspring of all tiles behind the particles, in the
//           order of the whole ensemble's steps, and closes the chunk.
//
// Order.  A step appends its records in the order of their event parents in
// the array.  Give an offspring the set of steps (a bit mask, its class) in
// which its ancestors since the chunk's start and it were born.  The array
// sorts the chunk's offspring by step of birth, then by the parent's place:
// first by the parent's step of birth, and so on, which is the numeric order
// of the classes (the highest bit first); within a class by the range of the
// first ancestor; within a class and tile by the tile's own order.  So the
// place of a record is the sum of the lower classes, its class's records in
// earlier tiles, and its index within its class and tile, and no step waits
// for another tile.  Nor does a step wait for the one before: a particle goes
// on with its wave vector whatever it leaves behind, so all steps' jumps of
// the range can be one list, and the offspring of a generation, listed by step
// and parent, are class by class in the order of the steps one by one.  (Step
// by step a small ensemble's tile has a chain of five, each with a jump or
// two.)
//
// Positions.  A particle's x in the array is its position at the last
// materialisation (or at the end of the step of its birth, if later); its
// position at the start of a later step is reached by adding (hbar/m) k dt
// once per step, which are the additions that one step at a time would do.
// The last chunk of a call adds them up in the array (adv), unless an
// annihilation follows in the same call, whose cell pass does it instead.
#pragma once
#include "wbrw_dev.hpp"
#include "wbrw_math.hpp"
#include "wbrw_step.hpp"

namespace wbrw {

// The launch constants, read again from memory by scalar loads.  k_walk holds
// more of them than there are scalar registers; values read where a scope
// begins do not stay live across the loops around it.  (Kept in registers
// from the kernel's start, some 200 of them lived in lanes of vector
// registers.)  The copy in device memory is written once, at wbrw_init.
__device__ __forceinline__ const Dev &fresh(const Dev *self)
{
    uint64_t p = (uint64_t)self;
    asm volatile("" : "+s"(p));
    return *(const Dev *)(const __attribute__((address_space(4))) Dev *)p;
}

// Instance b's parameters (b uniform over the wavefront), which no kernel
// writes: read by scalar loads, also after stores to global memory.
__device__ __forceinline__ const InstParam &inst_param(const Dev &d, int b)
{
    return *(const InstParam *)(const __attribute__((address_space(4))) InstParam *)(uintptr_t)(d.ip + b);
}

// Birth index of instance-particle i: the number of entries of the table
// nst[0 .. pend] (counts at the start of the steps since the last
// materialisation) that are <= i.  Its first advance is that of step
// `birth`, so m steps after the materialisation it has taken m - birth.
__device__ __forceinline__ int birth_of(const uint32_t *nst, int pend, uint32_t i)
{
    int b = 0;
    for (int q = 0; q < pend; ++q) b += nst[q] <= i ? 1 : 0;
    return b;
}

__device__ __forceinline__ double advanced(double x, double c, int m)
{
    for (int q = 0; q < m; ++q) x = x + c;
    return x;
}

// The high word of the first uniform of particle `id` in step `step` (word 1
// of its clock draw, counter (id, step, 0)): the rounds of Philox4x32-10 as
// far as this word needs them, 15 products.  The first round's products of
// the id and the second round's product that follows from them do not depend
// on the step (Clock), those of the step not on the particle.
struct Clock {
    uint32_t id_hi, h1, l1, h2, l2;
};
__device__ __forceinline__ Clock clock_of(uint64_t id, uint32_t key)
{
    const uint64_t p0 = (uint64_t)(uint32_t)id * 0xD2511F53ull;
    const uint32_t c2 = (uint32_t)(p0 >> 32) ^ key;
    const uint64_t p1 = (uint64_t)c2 * 0xCD9E8D57ull;
    return {(uint32_t)(id >> 32), c2, (uint32_t)p0, (uint32_t)(p1 >> 32), (uint32_t)p1};
}
__device__ __forceinline__ uint32_t clock_word(const Dev &d, const Clock &c, uint32_t step, uint32_t key)
{
    uint32_t k0 = d.seed, k1 = key;
    const uint64_t ps = (uint64_t)step * 0xCD9E8D57ull;
    // round 1: c0 ^= ..., c1 = low word of the step's product, c2 = h1, c3 = l1
    uint32_t c0 = c.id_hi ^ ((uint32_t)(ps >> 32) ^ k0);
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
    // round 2
    uint64_t p0 = (uint64_t)c0 * 0xD2511F53ull;
    c0 = c.h2 ^ ((uint32_t)ps ^ k0);
    uint32_t c1 = c.l2, c2 = xor3((uint32_t)(p0 >> 32), c.l1, k1), c3 = (uint32_t)p0;
#pragma unroll
    for (int r = 3; r <= 8; ++r) {
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
        p0 = (uint64_t)c0 * 0xD2511F53ull;
        const uint64_t p1 = (uint64_t)c2 * 0xCD9E8D57ull;
        c0 = xor3((uint32_t)(p1 >> 32), c1, k0);
        c1 = (uint32_t)p1;
        c2 = xor3((uint32_t)(p0 >> 32), c3, k1);
        c3 = (uint32_t)p0;
    }
    k1 += 0xBB67AE85u;
    c2 = xor3(__umulhi(c0, 0xD2511F53u), c3, k1);   // round 9
    return c2 * 0xCD9E8D57u;                        // round 10
}

// Does the particle jump before the end of the step?  The whole test, where
// the high word of its first uniform does not decide.
__device__ __noinline__ bool clock_exact(uint64_t id, uint32_t step, uint32_t seed, uint32_t key, double thr_lo,
                                         double thr_hi, double g0, double dt)
{
    const W4 e = draw(id, step, kTagStep, 0u, 0u, seed, key);
    const double u = unit53(e.a, e.b);
    if (u < thr_lo) return true;
    if (!(u <= thr_hi)) return false;
    return -ln_series(1.0 - u) / g0 <= dt;
}
__device__ __forceinline__ bool clock_jumps(const Dev &d, const InstParam &P, const Clock &c, uint64_t id, uint32_t step)
{
    const uint32_t w = clock_word(d, c, step, P.key);
    bool j = w < P.ib_lo;
    if (!j && w <= P.ib_hi) j = clock_exact(id, step, d.seed, P.key, P.thr_lo, P.thr_hi, P.gamma0, d.dt);
    return j;
}

// Inclusive scan of v over the wavefront, by data-parallel moves within rows
// of 16 lanes and broadcasts of the rows' last lanes (all 64 lanes call).
__device__ __forceinline__ uint32_t wave_incl(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // row_bcast:15
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // row_bcast:31
    return v;
}

// Exclusive scan of v over the block's threads (s_w: kThreads / 64 slots, not
// in use by an earlier call without a barrier in between); tot: the sum.
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t *s_w, uint32_t &tot)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t incl = wave_incl(v);
    if (lane == 63) s_w[wv] = incl;
    lds_barrier();
    uint32_t excl = incl - v;
    tot = 0;
#pragma unroll
    for (int q = 0; q < kThreads / 64; ++q) {
        const uint32_t t = s_w[q];
        if (q < wv) excl += t;
        tot += t;
    }
    return excl;
}

// A value that is the same in all lanes, for scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v));
}

// What a block of k_walk keeps in LDS.
constexpr uint32_t kLocal = 0x80000000u;
struct WalkTile {
    int64_t i0, a0;              // first particle, pages' base
    uint32_t nl, q0;             // offspring so far, event parents of the list that are done
    uint32_t g0, g1;             // the list's offspring
    int s;                       // its step, or (merged) the generation
    bool merged;                 // lists by generation
    int b, nr, i00, sh;
};
template <int DIM, bool SP2, bool TAN>
struct WalkShared {
    static constexpr int kW0 = kRangeMax / 64;       // words of a step's bits of the range
    static constexpr int kWL = kLocalBits / 64;      // ... of the offspring
    Families<DIM, SP2, TAN> F;
    uint64_t ev[kChunk][kW0];
    unsigned long long evl[kChunk][kWL];
    int64_t tal[5];
    uint32_t limit, cap;          // offspring that the pages hold; the instance's slots
    uint32_t pool;                // ... and those of all first pages
    WalkTile rest;                // what k_walk leaves to walk_general, and gets back
    int32_t t;
    uint32_t wsum[2][4];
    uint32_t total;               // event parents of the range, all steps
    uint32_t item[kThreads];      // event parents: index in the range, or
                                  // kLocal | index among the offspring
    uint32_t ccnt[kClasses];      // records of each class
    uint32_t nst[kPend + 1];
    uint32_t page[kPages];
    int parents;                  // event parents taken at a time in this tile
    int npage;                    // the tile's pages (thread 0 adds to them)
    uint8_t cls[kThreads];        // the step of the chunk the event parents jump in and,
                                  // above its kStepBits, their classes
    static constexpr int kStepBits = 3;
    __device__ __forceinline__ int step(int slot) const { return cls[slot] & ((1 << kStepBits) - 1); }
    static_assert(kChunk <= (1 << kStepBits) && (kClasses << kStepBits) <= 256, "a byte");
};

// Takes the event parents of tile T from generation T.g0 .. T.g1 on, batch by
// batch (k_walk).  False where a path of a batch does not fit, or its records
// even with kParents of them, with what is left to do in W.rest.  With GENERAL
// the next kThreads event parents are taken, each family by the general walk of
// one lane.  (Such ensembles mostly have batches of kParents, which would leave
// seven of eight lanes idle: 1e5 particles, gamma0 dt = 1.2, 2200 us by batches
// of 32 and 1900 by 256.)
template <int DIM, bool SP2, bool TAN, bool ONE, bool GENERAL, bool MERGED>
__device__ __forceinline__ bool walk_steps(const Dev *self, int ghost, int S, int pend, uint32_t set, uint32_t step0,
                                           WalkTile &T, WalkShared<DIM, SP2, TAN> &W, uint32_t &err)
{
    using FT = Families<DIM, SP2, TAN>;
    FT &F = W.F;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int b = T.b, nr = T.nr, i00 = T.i00, sh = T.sh;
    const int64_t i0 = T.i0, a0 = T.a0;
    uint32_t nl = T.nl;                  // offspring of the tile so far
    auto barrier = [] { if (GENERAL) block_sync(); else lds_barrier(); };
    auto more = [&]() -> const uint32_t * { return ghost ? fresh(self).ptxg : fresh(self).ptx; };
    const int nw0 = (nr + 63) / 64;
    int s0 = T.s;
    uint32_t g0 = T.g0, g1 = T.g1, q0 = T.q0;
    // event parents taken at a time (a batch)
    auto parents = [&] { return GENERAL ? kThreads : __builtin_amdgcn_readfirstlane(W.parents); };
    for (;; q0 = 0u) {
        // the list: steps sa .. sz - 1, of each the range's bits (step by
        // step, or the first generation) and those of offspring g0 .. g1 - 1
        const uint32_t sa = MERGED ? 0u : (uint32_t)s0, sz = MERGED ? (uint32_t)S : sa + 1u;
        const uint32_t nr0 = MERGED && s0 > 0 ? 0u : (uint32_t)nw0;
        const uint32_t wa = g0 / 64u, nw = nr0 + (g1 + 63u) / 64u - wa;
        uint32_t np = 0;                 // event parents of the list
        for (;;) {
            // event parents [q0, q0 + FS) of the list, by step and in order
            if (GENERAL || g1 > (uint32_t)kLocalBits) block_sync(); else lds_barrier();
            const int FS = parents();
            uint32_t run = 0, s = sa, w = (uint32_t)tid;      // word w of step s
            for (uint32_t w0 = 0, it = 0; w0 < nw * (sz - sa); w0 += kThreads, w += kThreads, ++it) {
                if (MERGED)
                    for (; w >= nw && s < sz; w -= nw) ++s;
                const uint32_t wl = wa + w - nr0;
                const bool loc = w >= nr0;
                uint64_t m = 0;
                if (MERGED ? s < sz : w < nw) {
                    if (!loc) {
                        m = W.ev[s][w];
                    } else {
                        if (wl < (uint32_t)WalkShared<DIM, SP2, TAN>::kWL) m = W.evl[s][wl];
                        else             // past the bits kept in LDS
                            for (uint32_t q = 0; q < 64u && wl * 64u + q < g1; ++q)
                                m |= (uint64_t)(((ghost ? fresh(self).smaskg : fresh(self).smask)
                                                 [a0 + page_slot(W.page, sh, wl * 64u + q, more)] >> (kChunk + s)) & 1u) << q;
                        if (MERGED && wl == wa) m &= ~0ull << (g0 & 63u);
                        if (MERGED && wl == g1 / 64u) m &= (1ull << (g1 & 63u)) - 1ull;
                    }
                }
                uint32_t tot;
                uint32_t pos = run + block_excl((uint32_t)__popcll(m), W.wsum[it & 1], tot);
                if (pos >= q0 + (uint32_t)FS || pos + (uint32_t)__popcll(m) <= q0) m = 0;
                while (m) {
                    const int k = __builtin_ctzll(m);
                    m &= m - 1ull;
                    if (pos >= q0 && pos < q0 + (uint32_t)FS) {
                        W.item[pos - q0] = loc ? kLocal | (wl * 64u + (uint32_t)k) : w * 64u + (uint32_t)k;
                        if (MERGED) W.cls[pos - q0] = (uint8_t)s;
                    }
                    ++pos;
                }
                run += tot;
                if (run >= q0 + (uint32_t)FS && np > 0u) break;     // (np is known)
            }
            if (np == 0u) np = run;
            if (q0 >= np) break;
            if (tid == 0) {
                F.n = F.nq[0] = F.nq[1] = F.overflow = F.events = F.pairs = F.maxdepth = 0u;
                F.killed = 0;
            }
            F.cnt[tid] = 0u;
            F.head[tid] = kNone;
            block_sync();
            const bool live = tid < FS && q0 + (uint32_t)tid < np;
            // event parent ti at the start of the step
            auto load_root = [&](int ti) {
                const Dev &d = fresh(self);
                const int64_t dstride = ghost ? d.gcap_total : d.cap_total;
                const uint32_t it = W.item[ti];
                const int s = MERGED ? W.step(ti) : s0;
                const bool loc = (it & kLocal) != 0u;
                const uint32_t l = it & ~kLocal;
                const Ens *sets = ghost ? d.gens : d.ens;
                const Ens E = sets[set], A = sets[set ^ 1u], X = loc ? A : E;
                const int64_t pi = loc ? a0 + page_slot(W.page, sh, l, more) : i0 + (int64_t)l;
                Node root;
                root.x[0] = X.x0[pi];
                root.x[1] = DIM == 2 ? X.x1[pi] : 0.0;
                root.k[0] = X.k0[pi];
                root.k[1] = DIM == 2 ? X.k1[pi] : 0.0;
                root.t0 = 0.0;
                root.id = X.id[pi];
                root.w = SP2 ? X.w[pi] : 0.0;
                root.sg = SP2 ? 0 : (int32_t)X.sg[pi];
                root.D[0] = TAN ? X.D[pi] : 0.0;
                root.D[1] = TAN ? X.D[dstride + pi] : 0.0;
                root.D[2] = TAN ? X.D[2 * dstride + pi] : 0.0;
                int m;
                if (!loc) {
                    if (!MERGED) W.cls[ti] = 0;
                    m = pend + s - birth_of(W.nst, pend, (uint32_t)i00 + l);
                } else {                 // steps since that of its birth, the class's highest
                    const uint32_t cls = (ghost ? d.smaskg : d.smask)[pi] & (kClasses - 1);
                    W.cls[ti] = (uint8_t)((MERGED ? s : 0) | (cls << W.kStepBits));
                    m = s - 1 - (31 - __builtin_clz(cls));
                }
                root.x[0] = advanced(root.x[0], (d.vfac * root.k[0]) * d.dt, m);
                if (DIM == 2) root.x[1] = advanced(root.x[1], (d.vfac * root.k[1]) * d.dt, m);
                return root;
            };
            // 1. the parents' first jumps, then round by round those
            //    found.  Each wavefront takes 64 jumps; where there are
            //    few, two or four share the same ones, each with its
            //    share of their pair slots.
            Tally tal{0, 0, 0, 0, 0};
            if constexpr (!GENERAL) {
                const int slots = ONE && !TAN ? 1 : (TAN && fresh(self).tangent == 2 ? 2 : 1) * (ONE ? 1 : fresh(self).M);
                uint32_t nt = min((uint32_t)FS, np - q0);      // jumps of the round
                int share = slots == 1 || nt > 128u ? 1 : (nt > 64u ? 2 : 4);
                int ti = wv / share * 64 + lane, m0 = wv % share;
                Node cur;
                uint64_t key = 0ull;
                uint32_t rec = kNone, step = step0 + (uint32_t)s0;
                int slot = ti, lev = 0;
                bool act = false;
                if (ti < (int)nt && m0 < slots) {
                    cur = load_root(ti);
                    if (MERGED) step = step0 + W.step(ti);
                    const Dev &d = fresh(self);
                    const InstParam &P = inst_param(d, b);
                    const W4 r = draw(cur.id, step, kTagStep, 0u, 0u, d.seed, P.key);
                    cur.te = cur.t0 + (-ln_series(1.0 - unit53(r.a, r.b)) / P.gamma0);
                    cur.ua0 = unit53(r.c, r.d);
                    cur.e = 0u;
                    act = cur.te <= d.dt;
                }
                for (int round = 0;; ++round) {
                    const Dev &d = fresh(self);
                    const InstParam &P = inst_param(d, b);
                    if (act)
                        take_jump<DIM, SP2, TAN, ONE>(d, P, step, round, cur, key, lev, slot, rec, m0, share, F);
                    if (DIM == 2) block_sync(); else lds_barrier();   // 4D records may be in HBM
                    nt = F.nq[round & 1];
                    if (nt == 0u || F.overflow) break;
                    share = slots == 1 || nt > 128u ? 1 : (nt > 64u ? 2 : 4);
                    ti = wv / share * 64 + lane;
                    m0 = wv % share;
                    act = ti < (int)nt && m0 < slots;
                    if (act) {
                        rec = F.qrec[ti];
                        load_record<DIM, SP2, TAN>(d, F, rec, cur);
                        cur.x[0] = F.qx0[ti];
                        cur.x[1] = DIM == 2 ? F.qx1[ti] : 0.0;
                        cur.t0 = F.qt0[ti];
                        cur.te = F.qte[ti];
                        cur.ua0 = F.qua[ti];
                        cur.e = F.qe[ti];
                        key = F.key[rec];
                        slot = F.slot[rec];
                        if (MERGED) step = step0 + W.step(slot);
                        lev = key ? FT::kLevels - (__ffsll((unsigned long long)key) - 1) / 8 : 0;
                    }
                    if (tid == 0) F.nq[(round + 1) & 1] = 0u;
                    lds_barrier();
                }
            }
            if constexpr (!GENERAL) {
                if (__builtin_expect(F.overflow != 0u, 0)) {    // (uniform)
                    // Records or jumps than there is room for: half as
                    // many parents, for the rest of the tile.  (Ensembles
                    // crowded where |sin| is near 1 leave 1.57 times the
                    // records that Dev::ftile counts with.  7e5 particles,
                    // gamma0 dt = 0.3, two steps: 270 us so, 1550 with every
                    // such batch by the general walk.)
                    const int fs = parents();
                    if (F.overflow == 1u && fs > kParents) {
                        lds_barrier();
                        if (tid == 0) W.parents = max(kParents, fs / 2 / kParents * kParents);
                        continue;
                    }
                    if (tid == 0) {
                        W.rest = T;
                        W.rest.nl = nl;
                        W.rest.q0 = q0;
                        W.rest.g0 = g0;
                        W.rest.g1 = g1;
                        W.rest.s = s0;
                    }
                    return false;
                }
            } else if (live) {
                const Node root = load_root(tid);
                F.cnt[tid] = walk_family<DIM, SP2, TAN>(self, b, step0 + (uint32_t)(MERGED ? W.step(tid) : s0), &root, false, Ens{}, a0, 0, 0, W.page, more(), sh, 0, &tal, &err);
            }
            if (GENERAL) barrier();
            // 2. ordered exclusive scan of the families' record counts
            uint32_t agg;
            // (read before the barrier that thread 0 may change it after)
            const uint32_t room = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.limit);
            const uint32_t excl = block_excl(F.cnt[tid], W.wsum[0], agg);
            F.first[tid] = excl;
            if (__builtin_expect(nl + agg > room && sh < 31, 0)) {     // (uniform) further pages, as many as fit
                if (tid == 0) {
                    const Dev &d = fresh(self);
                    int q = W.npage;
                    const uint32_t want = ((nl + agg + ((1u << sh) - 1u)) >> sh) - (uint32_t)q;
                    const uint64_t from = W.pool +
                        atomicAdd((unsigned long long *)&d.wpool[(int64_t)ghost * d.B + b], (unsigned long long)want << sh);
                    const int np = q + (int)(from < W.cap ? min(want, (W.cap - (uint32_t)from) >> sh) : 0u);
                    const uint32_t old = W.page[kDirect], size = page_table(np);
                    uint32_t table = old, *tab = ghost ? d.ptxg : d.ptx;
                    if (size != page_table(q)) {
                        table = atomicAdd(&d.ctl->table[ghost], size);
                        for (int j = 0; j < q - kDirect; ++j) tab[table + j] = tab[old + j];
                        W.page[kDirect] = table;
                    }
                    uint32_t first = (uint32_t)from;
                    for (; q < min(np, kDirect); ++q, first += 1u << sh) W.page[q] = first;
                    for (; q < np; ++q, first += 1u << sh) tab[table + (q - kDirect)] = first;
                    W.npage = np;
                    W.limit = (uint32_t)np << sh;
                }
                block_sync();
            }
            barrier();
            // 3. records into the tile's area, each at its rank in its
            //    family, with its class and its own jumps in the chunk's
            //    later steps
            const Dev &d = fresh(self);
            const InstParam &P = inst_param(d, b);
            const Ens &A = (ghost ? d.gens : d.ens)[set ^ 1u];
            const uint32_t limit = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.limit);
            uint16_t *smask = ghost ? d.smaskg : d.smask;
            const int64_t dstride = ghost ? d.gcap_total : d.cap_total;
            auto close_record = [&](uint32_t li, int64_t o, uint64_t id, int slot) {
                const int s = MERGED ? W.step(slot) : s0;
                const uint32_t cls = (uint32_t)(W.cls[slot] >> W.kStepBits) | (1u << s);
                uint32_t ev = 0;
                const Clock c = clock_of(id, P.key);
                for (int q = MERGED ? 1 : s + 1; q < S; ++q)
                    if ((!MERGED || q > s) && clock_jumps(d, P, c, id, step0 + (uint32_t)q)) {
                        ev |= 1u << q;
                        if (li < kLocalBits) atomicOr(&W.evl[q][li >> 6], 1ull << (li & 63));
                    }
                smask[o] = (uint16_t)(cls | (ev << kChunk));
                atomicAdd(&W.ccnt[cls], 1u);
            };
            if constexpr (!GENERAL) {
                const uint32_t nrec = F.n;
                uint32_t deep = 0;
                for (uint32_t r = (uint32_t)tid; r < nrec; r += kThreads) {
                    const uint64_t key = F.key[r];
                    if (key == 0ull) continue;
                    const int slot = F.slot[r];
                    uint32_t rank = 0;
                    for (uint32_t q = F.head[slot]; q != kNone; q = F.next[q]) rank += F.key[q] < key ? 1u : 0u;
                    deep = max(deep, (uint32_t)(FT::kLevels - (__ffsll((unsigned long long)key) - 1) / 8));
                    const uint32_t li = nl + F.first[slot] + rank;
                    if (li >= limit) { err |= kErrCapacity; continue; }
                    const int64_t o = a0 + page_slot(W.page, sh, li, more);
                    Node nd;
                    load_record<DIM, SP2, TAN>(d, F, r, nd);
                    A.x0[o] = nd.x[0];
                    A.k0[o] = nd.k[0];
                    if (DIM == 2) {
                        A.x1[o] = nd.x[1];
                        A.k1[o] = nd.k[1];
                    }
                    if (SP2) A.w[o] = nd.w; else A.sg[o] = (int8_t)nd.sg;
                    A.id[o] = nd.id;
                    if (TAN) {
                        A.D[o] = nd.D[0];
                        A.D[dstride + o] = nd.D[1];
                        A.D[2 * dstride + o] = nd.D[2];
                    }
                    close_record(li, o, nd.id, slot);
                }
                // the wavefront's deepest level by ballots (an atomic
                // maximum of per-lane values takes the lanes one by one)
                uint32_t top = 0;
                while (__ballot(deep > top)) ++top;
                if (lane == 0) atomicMax(&F.maxdepth, top);
            } else {
                if (live) {
                    const Node root = load_root(tid);
                    Tally none{0, 0, 0, 0, 0};
                    const int64_t f = (int64_t)nl + (int64_t)excl;
                    const uint32_t c = walk_family<DIM, SP2, TAN>(self, b, step0 + (uint32_t)(MERGED ? W.step(tid) : s0), &root, true, A, a0, f, limit, W.page, more(), sh,
                                                                  dstride, &none, &err);
                    for (uint32_t r = 0; r < c && f + r < limit; ++r) {
                        const int64_t o = a0 + page_slot(W.page, sh, (uint32_t)(f + r), more);
                        close_record((uint32_t)(f + r), o, A.id[o], tid);
                    }
                }
                atomicAdd((unsigned long long *)&W.tal[0], (unsigned long long)tal.events);
                atomicAdd((unsigned long long *)&W.tal[1], (unsigned long long)tal.pairs);
                atomicAdd((unsigned long long *)&W.tal[2], (unsigned long long)tal.killed);
                atomicAdd((unsigned long long *)&W.tal[3], (unsigned long long)tal.cap);
                atomicMax((unsigned long long *)&W.tal[4], (unsigned long long)tal.maxdepth);
            }
            nl = min(nl + agg, limit);
            barrier();
            if (tid == 0 && !GENERAL) {
                W.tal[0] += F.events;
                W.tal[1] += F.pairs;
                W.tal[2] += F.killed;
                W.tal[4] = max(W.tal[4], (int64_t)F.maxdepth);
            }
            if constexpr (GENERAL) {
                T.nl = nl;
                T.q0 = q0 + (uint32_t)kThreads;
                return true;
            }
            q0 += (uint32_t)parents();
            if (q0 >= np) break;
        }
        ++s0;
        if (MERGED) g0 = g1;             // the next generation
        g1 = nl;
        if (s0 == S || (MERGED && g0 == g1)) break;
    }
    return true;
}

// Event parents whose families do not fit the pool.  A function of its own, called
// where k_walk holds nothing else: with the general walk's calls inside the
// steps the common path spilt 100 vector registers and took longer (256
// instances 8.95 ms a pass and 7.63 so, barrier of 1e7 2.32 and 2.12, of 1e4
// 1.02 and 0.88, weighted 1e7 1.78 and 1.52, 4D 12.3 and 11.2).
template <int DIM, bool SP2, bool TAN>
__device__ __noinline__ uint32_t walk_general(const Dev *self, int ghost, int S, int pend, uint32_t set, uint32_t step0,
                                           WalkShared<DIM, SP2, TAN> *W)
{
    const Dev *uniform = (const Dev *)uniform64((int64_t)self);
    WalkTile T = W->rest;
    T.b = __builtin_amdgcn_readfirstlane(T.b);
    uint32_t err = 0;
    if (DIM == 1 && T.merged) walk_steps<DIM, SP2, TAN, false, true, DIM == 1>(uniform, ghost, S, pend, set, step0, T, *W, err);
    else walk_steps<DIM, SP2, TAN, false, true, false>(uniform, ghost, S, pend, set, step0, T, *W, err);
    if (threadIdx.x == 0) W->rest = T;
    block_sync();
    return err;
}

template <int DIM, bool SP2, bool TAN, bool ONE>
__global__ __launch_bounds__(kThreads, (DIM == 2 || TAN) ? 3 : 4) void k_walk(const Dev *self, int ghost, int S,
                                                                             int pend, int adv)
{
    using WS = WalkShared<DIM, SP2, TAN>;
    constexpr int kWL = WS::kWL;
    __shared__ WS W;

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t err = 0, step0, par, set;
    int B;
    int64_t ntiles;
    {
        const Dev &d = fresh(self);
        Ctl *ctl = d.ctl;
        step0 = ctl->step;
        par = ctl->chunk & 1u;
        set = ghost ? ctl->gcur : ctl->cur;
        B = d.B;
        ntiles = d.tileW[(int64_t)(2 * par + ghost) * (B + 1) + B];
        // kept for k_place, whose closing block changes both
        if (blockIdx.x == 0) {
            const int64_t *Ncur = ghost ? d.NG : d.N;
            for (int b = tid; b < B; b += kThreads) d.Nbase[(int64_t)ghost * B + b] = Ncur[b];
            if (tid == 0) ctl->wpar = par;
        }
    }
    // Tallies stay in LDS while the block works on one instance; they go to
    // the instance's counters when the block moves on to another one, and the
    // last instance's share is left in the block's slot of fpart for the
    // closing block of the placement launch.  Per-tile atomics on one cache
    // line would serialise the whole grid.
    int cb = -1;
    bool first = true;
    if (tid < 5) W.tal[tid] = 0;
    for (;;) {
        if (tid == 0) {
            const Dev &d = fresh(self);
            W.t = (int32_t)next_tile_static_first(&d.ctl->ticket[ghost ? kPassFamilyG : kPassFamily], ntiles, first);
        }
        for (int q = tid; q < kChunk * kWL; q += kThreads) (&W.evl[0][0])[q] = 0ull;
        if (tid < kClasses) W.ccnt[tid] = 0u;
        if (tid == 0) W.total = 0u;
        lds_barrier();
        const int64_t t = __builtin_amdgcn_readfirstlane(W.t);
        if (t >= ntiles) break;
        // tile t is tile tl of instance b: its range of nr particles from i0
        // on; its offspring go to pages of 2^sh slots behind a0
        int b, nr, i00, sh;
        int64_t i0, a0;
        bool merged;
        {
            const Dev &d = fresh(self);
            const int64_t at = 2 * par + (uint32_t)ghost, *plan = d.tileW + at * (B + 1);
            b = B == 1 ? 0 : __builtin_amdgcn_readfirstlane(segment_of(plan, B, t));
            const InstParam &P = inst_param(d, b);
            const int64_t base = ghost ? P.gbase : P.base, n = (ghost ? d.NG : d.N)[b], tl = t - plan[b];
            const int64_t R = d.wrange[2 * (at * B + b)];
            sh = (int)d.wrange[2 * (at * B + b) + 1];
            i00 = (int)(tl * R);
            i0 = base + tl * R;
            nr = (int)min(R, n - tl * R);
            a0 = base;
            if (tid == 0) {
                W.page[0] = (uint32_t)(tl << (sh & 31));
                W.npage = 1;
                W.parents = ghost ? d.gftile : d.ftile;
                W.cap = (uint32_t)(ghost ? P.gcap : P.cap);
                W.limit = min(1u << sh, W.cap);
                W.pool = (uint32_t)(plan[b + 1] - plan[b]) << (sh & 31);
            }
        }
        if (b != cb) {
            const Dev &d = fresh(self);
            if (tid == 0 && cb >= 0) {
                int64_t *T = d.tally + (int64_t)cb * kTalCount;
                if (W.tal[0]) atomicAdd((unsigned long long *)&T[kTalEvents], (unsigned long long)W.tal[0]);
                if (W.tal[1]) atomicAdd((unsigned long long *)&T[kTalPairs], (unsigned long long)W.tal[1]);
                if (W.tal[2]) atomicAdd((unsigned long long *)&T[kTalKilled], (unsigned long long)W.tal[2]);
                if (W.tal[3]) atomicAdd((unsigned long long *)&T[kTalEventCap], (unsigned long long)W.tal[3]);
                if (W.tal[4]) atomicMax((unsigned long long *)&T[kTalMaxDepth], (unsigned long long)W.tal[4]);
                for (int q = 0; q < 5; ++q) W.tal[q] = 0;
            }
            cb = b;
            if (tid < pend) W.nst[tid] = (uint32_t)d.nstep[((int64_t)ghost * B + b) * (kPend + 1) + tid];
        }
        // the range's clocks, lanes on consecutive particles; the next ids
        // are loaded while the draws of the last ones run
        {
            const Dev &d = fresh(self);
            const InstParam &P = inst_param(d, b);
            const uint64_t *ids = (ghost ? d.gens : d.ens)[set].id + i0;
            uint64_t id = ids[min(tid, nr - 1)];
            uint32_t nev = 0;
            for (int j = 0; j * kThreads < nr; ++j) {
                const int li = j * kThreads + tid;
                const uint64_t cur = id;
                const Clock c = clock_of(cur, P.key);
                const uint64_t in = __ballot(li < nr);
                id = ids[min(li + kThreads, nr - 1)];
                for (int s = 0; s < S; ++s) {
                    const uint32_t w = clock_word(d, c, step0 + (uint32_t)s, P.key);
                    uint64_t m = __ballot(w < P.ib_lo);
                    const uint64_t band = __ballot(w <= P.ib_hi) ^ m;   // not decided by this word
                    if (band)
                        m |= band & __ballot(clock_exact(cur, step0 + (uint32_t)s, d.seed, P.key, P.thr_lo, P.thr_hi,
                                                         P.gamma0, d.dt));
                    m &= in;
                    nev += (uint32_t)__popcll(m);
                    if (lane == 0) W.ev[s][j * (kThreads / 64) + wv] = m;
                }
            }
            // Do all steps' jumps of the range fit one list?  (1e4 barrier: the
            // kernel takes 44.5 us step by step and 31.5 so, 2e5 cat state 61
            // and 45; at 1e7, whose tiles find 440 jumps for 256 threads,
            // lists of all steps took 284 us and single steps 264.  4D step by
            // step: its ensembles are large, and the second path alone cost
            // them 1 %.)
            merged = DIM == 1 && S > 1;
            if (merged) {
                if (lane == 0 && nev) atomicAdd(&W.total, nev);
                lds_barrier();
                merged = __builtin_amdgcn_readfirstlane((int)W.total) <= (ghost ? d.gftile : d.ftile);
            }
        }
        WalkTile T{i0, a0, 0u, 0u, 0u, 0u, 0, merged, b, nr, i00, sh};
        while (!(DIM == 1 && merged ? walk_steps<DIM, SP2, TAN, ONE, false, DIM == 1>(self, ghost, S, pend, set, step0, T, W, err)
                        : walk_steps<DIM, SP2, TAN, ONE, false, false>(self, ghost, S, pend, set, step0, T, W, err))) {
            block_sync();
            err |= walk_general<DIM, SP2, TAN>(self, ghost, S, pend, set, step0, &W);
            T.nl = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.rest.nl);
            T.q0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.rest.q0);
            T.g0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.rest.g0);
            T.g1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)W.rest.g1);
            T.s = __builtin_amdgcn_readfirstlane(W.rest.s);
        }
        lds_barrier();
        // the tile's counts per class, also summed over groups of tiles
        const Dev &d = fresh(self);
        if (tid < min(W.npage, kPages)) (ghost ? d.ptabg : d.ptab)[t * kPages + tid] = W.page[tid];
        if (tid < kClasses) {
            uint32_t *wcnt = ghost ? d.wcntg : d.wcnt;
            uint32_t *wsup = (ghost ? d.wsupg : d.wsup) + (int64_t)par * (ghost ? d.wsup_gg : d.wsup_g) * kClasses;
            const uint32_t c = W.ccnt[tid];
            wcnt[t * kClasses + tid] = tid ? c : (uint32_t)merged;      // (no class 0)
            if (c) atomicAdd(&wsup[(t / kSupGroup) * kClasses + tid], c);
            if (c && B > kFewInst) atomicAdd(&d.wtot[((int64_t)ghost * B + b) * kClasses + tid], c);
        }
        if (adv) {
            const Ens &E = (ghost ? d.gens : d.ens)[set];
            for (int li = tid; li < nr; li += kThreads) {
                const int64_t i = i0 + li;
                const int m = pend + S - birth_of(W.nst, pend, (uint32_t)(i00 + li));
                const double c0 = (d.vfac * E.k0[i]) * d.dt;
                __builtin_nontemporal_store(advanced(E.x0[i], c0, m), &E.x0[i]);
                if (DIM == 2) {
                    const double c1 = (d.vfac * E.k1[i]) * d.dt;
                    __builtin_nontemporal_store(advanced(E.x1[i], c1, m), &E.x1[i]);
                }
            }
        }
        lds_barrier();
    }
    if (tid == 0) {
        int64_t *T = fresh(self).fpart + (int64_t)blockIdx.x * 8;
        T[0] = cb;
        for (int q = 0; q < 5; ++q) T[1 + q] = W.tal[q];
    }
    if (err) atomicOr(&fresh(self).ctl->err, err);
}

// Per class c (threads tid mod kClasses = c; all threads of the block call):
// the records of tiles [a, m) and of [a, z), from the tiles' counts and
// their group sums.  s_red: 2 * kThreads words.
__device__ __forceinline__ void class_sums(const uint32_t *wcnt, const uint32_t *wsup, int64_t a, int64_t m, int64_t z,
                                           uint32_t *s_red, uint32_t &below, uint32_t &total)
{
    constexpr int kRows = kThreads / kClasses;
    const int tid = threadIdx.x, c = tid % kClasses, row = tid / kClasses;
    auto sum = [&](int64_t lo, int64_t hi) {
        const TileRange R(lo, hi);
        uint32_t v = 0;
        for (int64_t e = row; e < R.n(); e += kRows) {
            if (e < R.nh) v += wcnt[(R.a + e) * kClasses + c];
            else if (e < R.nh + R.ng) v += wsup[(R.ga / kSupGroup + (e - R.nh)) * kClasses + c];
            else v += wcnt[(R.gc + (e - R.nh - R.ng)) * kClasses + c];
        }
        return v;
    };
    const uint32_t v0 = sum(a, m), v1 = sum(m, z);
    block_sync();
    s_red[tid] = v0;
    s_red[kThreads + tid] = v1;
    block_sync();
    below = total = 0;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
        below += s_red[r * kClasses + c];
        total += s_red[kThreads + r * kClasses + c];
    }
    total += below;
}

__device__ void close_chunk(const Dev &d, int ghost, int S, int pend, int adv, int advance, int fgrid);

// The tiles' offspring go to their places behind the particles (see the
// order above).  A block takes a run of tiles.  Block 0 (dispatched first)
// closes the chunk.
template <int DIM, bool SP2, bool TAN>
__global__ __launch_bounds__(kThreads) void k_place(Dev d, int ghost, int S, int pend, int adv, int advance, int fgrid)
{
    if (blockIdx.x == 0) {
        close_chunk(d, ghost, S, pend, adv, advance, fgrid);
        return;
    }
    __shared__ uint32_t s_red[2 * kThreads];
    __shared__ uint32_t s_below[kClasses], s_tot[kClasses], s_own[kClasses], s_off[kClasses];
    __shared__ uint32_t s_page[kPages];
    Ctl *ctl = d.ctl;
    const int B = d.B;
    const uint32_t par = ctl->wpar;
    const int64_t *plan = d.tileW + (int64_t)(2 * par + ghost) * (B + 1);
    const int64_t ntiles = plan[B];
    const uint32_t set = ghost ? ctl->gcur : ctl->cur;
    const Ens E = pick_set(d, ghost, set);
    const Ens A = pick_set(d, ghost, set ^ 1u);
    const uint16_t *smask = ghost ? d.smaskg : d.smask;
    const uint32_t *ptab = ghost ? d.ptabg : d.ptab, *more = ghost ? d.ptxg : d.ptx;
    const uint32_t *wcnt = ghost ? d.wcntg : d.wcnt;
    const uint32_t *wsup = (ghost ? d.wsupg : d.wsup) + (int64_t)par * (ghost ? d.wsup_gg : d.wsup_g) * kClasses;
    const int64_t dstride = ghost ? d.gcap_total : d.cap_total;
    const int tid = threadIdx.x;
    const int64_t g = blockIdx.x - 1, G = gridDim.x - 1;
    const int64_t t0 = ntiles * g / G, t1 = ntiles * (g + 1) / G;
    uint32_t err = 0;
    int cb = -1;
    for (int64_t t = t0; t < t1; ++t) {
        const int b = __builtin_amdgcn_readfirstlane(segment_of(plan, B, t));
        if (b != cb) {
            uint32_t below, total;
            class_sums(wcnt, wsup, plan[b], t, plan[b + 1], s_red, below, total);
            if (tid < kClasses) {
                s_below[tid] = below;
                s_tot[tid] = total;
            }
            cb = b;
        } else if (tid < kClasses) {
            s_below[tid] += s_own[tid];
        }
        block_sync();
        if (tid < kClasses) s_own[tid] = wcnt[t * kClasses + tid];
        if (tid >= kThreads - kPages) s_page[tid - (kThreads - kPages)] = ptab[t * kPages + tid - (kThreads - kPages)];
        block_sync();
        const InstParam &P = d.ip[b];
        const int64_t base = ghost ? P.gbase : P.base;
        const int64_t cap = ghost ? P.gcap : P.cap;
        const int sh = (int)d.wrange[2 * ((int64_t)(2 * par + ghost) * B + b) + 1];
        if (tid < kClasses) {
            // lower classes, earlier tiles, less the class's start in the tile:
            // a tile holds its offspring by class, or (where k_walk merged the
            // steps, s_own[0]) by generation, then by class
            uint32_t o = s_below[tid];
            for (int c = 1; c < kClasses; ++c) {
                const int order = s_own[0] ? __popc(c) - __popc(tid) : 0;
                o += (c < tid ? s_tot[c] : 0u) - (order < 0 || (order == 0 && c < tid) ? s_own[c] : 0u);
            }
            s_off[tid] = o;
        }
        uint32_t nrec = 0;
        for (int c = 1; c < kClasses; ++c) nrec += s_own[c];
        block_sync();
        const int64_t n0 = d.Nbase[(int64_t)ghost * B + b];
        for (uint32_t r = (uint32_t)tid; r < nrec; r += kThreads) {
            const int64_t i = base + page_slot(s_page, sh, r, [&] { return more; });
            const uint32_t cls = smask[i] & (kClasses - 1);
            const int64_t dst = n0 + (int64_t)(uint32_t)(s_off[cls] + r);
            double x0 = A.x0[i], x1 = DIM == 2 ? A.x1[i] : 0.0;
            const double k0 = A.k0[i], k1 = DIM == 2 ? A.k1[i] : 0.0;
            const double w = SP2 ? A.w[i] : 0.0;
            const int8_t sg = SP2 ? (int8_t)0 : A.sg[i];
            const uint64_t id = A.id[i];
            double D[3];
            for (int c = 0; c < 3; ++c) D[c] = TAN ? A.D[c * dstride + i] : 0.0;
            if (dst >= cap) { err |= kErrCapacity; continue; }
            if (adv) {
                const int m = S - 1 - (31 - __builtin_clz(cls));   // born in the step of the highest bit
                x0 = advanced(x0, (d.vfac * k0) * d.dt, m);
                if (DIM == 2) x1 = advanced(x1, (d.vfac * k1) * d.dt, m);
            }
            const int64_t o = base + dst;
            E.x0[o] = x0;
            E.k0[o] = k0;
            if (DIM == 2) {
                E.x1[o] = x1;
                E.k1[o] = k1;
            }
            if (SP2) E.w[o] = w; else E.sg[o] = sg;
            E.id[o] = id;
            if (TAN)
                for (int c = 0; c < 3; ++c) E.D[c * dstride + o] = D[c];
        }
        block_sync();
    }
    if (err) atomicOr(&ctl->err, err);
}

// In the first block of the placement launch: the walking blocks' tallies,
// the new particle counts (also those at the start of every step of the
// chunk) with the capacity clamp, the next chunk's tile plan and that of the
// passes over the ensemble, the group sums the next chunk adds to, and the
// step counter.  Nothing here is read by the placing blocks.
__device__ void close_chunk(const Dev &d, int ghost, int S, int pend, int adv, int advance, int fgrid)
{
    Ctl *ctl = d.ctl;
    const int B = d.B;
    const int tid = threadIdx.x;
    const uint32_t step = ctl->step, par = ctl->wpar;
    int64_t *Ncur = ghost ? d.NG : d.N;
    const int64_t *plan = d.tileW + (int64_t)(2 * par + ghost) * (B + 1);
    int64_t *next = d.tileW + (int64_t)(2 * (par ^ 1u) + ghost) * (B + 1);
    const int64_t groups = ghost ? d.wsup_gg : d.wsup_g;
    const uint32_t *wcnt = ghost ? d.wcntg : d.wcnt;
    uint32_t *sup = ghost ? d.wsupg : d.wsup;
    {   // clear the other parity's group sums (the tiles of the chunk before)
        const int64_t used = (next[B] + kSupGroup - 1) / kSupGroup * kClasses;
        uint32_t *o = sup + (int64_t)(par ^ 1u) * groups * kClasses;
        for (int64_t q = tid; q < used; q += kThreads) o[q] = 0u;
    }
    const uint32_t *wsup = sup + (int64_t)par * groups * kClasses;
    // the walking blocks' last tallies, summed per instance in LDS when the
    // instances fit (global atomics from one block on one line serialise)
    constexpr int kLdsB = 256;
    __shared__ int64_t s_acc[5][kLdsB];
    __shared__ uint32_t s_red[2 * kThreads];
    __shared__ uint32_t s_tot[kClasses];
    const bool lds = B <= kLdsB;
    if (lds)
        for (int b = tid; b < B; b += kThreads)
            for (int q = 0; q < 5; ++q) s_acc[q][b] = 0;
    block_sync();
    for (int g = tid; g < fgrid; g += kThreads) {
        const int64_t *F = d.fpart + (int64_t)g * 8;
        if (F[0] < 0) continue;
        if (lds) {
            const int b = (int)F[0];
            for (int q = 0; q < 4; ++q)
                if (F[1 + q]) atomicAdd((unsigned long long *)&s_acc[q][b], (unsigned long long)F[1 + q]);
            if (F[5]) atomicMax((unsigned long long *)&s_acc[4][b], (unsigned long long)F[5]);
        } else {
            int64_t *T = d.tally + F[0] * kTalCount;
            if (F[1]) atomicAdd((unsigned long long *)&T[kTalEvents], (unsigned long long)F[1]);
            if (F[2]) atomicAdd((unsigned long long *)&T[kTalPairs], (unsigned long long)F[2]);
            if (F[3]) atomicAdd((unsigned long long *)&T[kTalKilled], (unsigned long long)F[3]);
            if (F[4]) atomicAdd((unsigned long long *)&T[kTalEventCap], (unsigned long long)F[4]);
            if (F[5]) atomicMax((unsigned long long *)&T[kTalMaxDepth], (unsigned long long)F[5]);
        }
    }
    block_sync();
    int over = 0;         // an instance of this thread holds more than ann_limit
    // counts from the class totals: by all threads from the tiles' counts
    // where there are few instances, else kept per instance by k_walk (whose
    // tiles of one instance are then few: their additions to its line of
    // totals do not queue up)
    auto finish = [&](int b, auto total) {   // total(c): the instance's records of class c
        int64_t *T = d.tally + (int64_t)b * kTalCount;
        if (lds) {
            T[kTalEvents] += s_acc[0][b];
            T[kTalPairs] += s_acc[1][b];
            T[kTalKilled] += s_acc[2][b];
            T[kTalEventCap] += s_acc[3][b];
            if (s_acc[4][b] > T[kTalMaxDepth]) T[kTalMaxDepth] = s_acc[4][b];
        }
        const int64_t cap = ghost ? d.ip[b].gcap : d.ip[b].cap;
        int64_t n = Ncur[b], ps = 0;
        int64_t *ns = d.nstep + ((int64_t)ghost * B + b) * (kPend + 1);
        for (int s = 0; s < S; ++s) {
            ps += n;
            for (int c = 1 << s; c < (2 << s); ++c) n += (int64_t)total(c);
            if (n > cap) {
                atomicOr(&ctl->err, kErrCapacity);
                n = cap;
            }
            if (!adv) ns[pend + s + 1] = n;
        }
        if (adv) ns[0] = n;
        d.wpool[(int64_t)ghost * B + b] = 0ull;
        if (!ghost) T[kTalPSteps] += ps;
        Ncur[b] = n;
        if (d.ann_limit > 0 && n > d.ann_limit) over = 1;
    };
    if (B <= kFewInst) {
        for (int b = 0; b < B; ++b) {
            uint32_t below, tot;
            class_sums(wcnt, wsup, plan[b], plan[b], plan[b + 1], s_red, below, tot);
            if (tid < kClasses) s_tot[tid] = tot;
            block_sync();
            if (tid == 0) finish(b, [&](int c) { return s_tot[c]; });
            block_sync();
        }
    } else {
        for (int b = tid; b < B; b += kThreads) {
            uint32_t *W = d.wtot + ((int64_t)ghost * B + b) * kClasses;
            finish(b, [&](int c) { return W[c]; });
            for (int c = 0; c < kClasses; ++c) W[c] = 0u;
        }
    }
    // conditional annihilation after this step (chunks of one step):
    // scheduled, or an instance about to outgrow the threshold (the real
    // ensemble's closing block)
    __shared__ int s_over;
    if (tid == 0) s_over = 0;
    block_sync();
    if (over) s_over = 1;
    block_sync();
    const int any_over = s_over;
    if (d.cond_ann && !ghost && tid == 0) {
        const bool sched = d.ann_every > 0 && (step + (uint32_t)S) % (uint32_t)d.ann_every == 0u;
        ctl->ann_now = (sched || any_over) ? 1u : 0u;
        if (any_over && !sched)
            for (int b = 0; b < B; ++b) d.tally[(int64_t)b * kTalCount + kTalTrig] += 1;
    }
    // the tile plans
    block_plan(d.tileA + (int64_t)ghost * (B + 1), Ncur, B, kTileA);
    plan_walk(d, par ^ 1u, ghost, Ncur);
    if (tid == 0) ctl->table[ghost] = 0u;
    if (tid == 0 && advance) {
        ctl->step = step + (uint32_t)S;
        ctl->chunk += 1u;
    }
}

}  // namespace wbrw
