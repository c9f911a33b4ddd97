// The jumps of the Wigner branching random walk within one time step (Alg. 1,
// Sec. 2): kick sampling, pair decisions, offspring, and the families of
// event parents, jump by jump (take_jump) or, where those do not fit, by a
// general depth-first walk.  The kernels that take ensembles through time
// steps are in wbrw_walk.hpp.
#pragma once
#include <type_traits>

#include "wbrw_dev.hpp"
#include "wbrw_math.hpp"

namespace wbrw {

// ---------------------------------------------------------------------------
// Kernel phase and kick sampling (Sec. 4.2, Remark 3 / Eq. majorant_approach)
// ---------------------------------------------------------------------------
template <int DIM>
__device__ __forceinline__ double phase_offset(const Dev &d, int m, const double *xe, double c)
{
    if (DIM == 1) return xe[0] - c;
    const int a = d.axis[m];
    if (a == 0) return xe[0] - c;
    if (a == 1) return xe[1] - c;
    return (xe[0] - xe[1]) - c;
}

// q from G_m / xi_m: Gaussian (Box-Muller, std 1/(2w)) or inverse CDF of the
// piecewise-constant table with a uniform offset inside the chosen bin.  The
// bin is the last j < n with cum[j] <= u1 cum[n].  A guide table (Chen and
// Asau's method) gives the answer's range: for u1 in bucket i = floor(u1 kg)
// the target u1 cum[n] lies between the rounded bucket ends, so the bin lies
// in the bucket's [lo, hi], nearly always one or two bins wide, which one
// 16-byte entry settles; wider ones are searched.  The bin found is that of
// a search over the whole table (12 dependent loads).
template <bool ONE>
__device__ __forceinline__ double kick_sample(const Dev &d, const InstParam &P, int m, double u1,
                                              double u2)
{
    if (ONE || d.kind[m] == 0) {
        const double R = sqrt(-2.0 * ln_series(1.0 - u1));
        const double z = R * cos_det(kTwoPi * u2);
        return z * P.sq[m];
    }
    const Table &T = d.tab[m];
    const double target = u1 * T.total;
    const GuideEntry g = T.guide[(int)(u1 * (double)T.kg)];
    int lo = g.lo, hi = g.hi;
    if (hi == lo + 1) {
        lo = g.next <= target ? hi : lo;
    } else {
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (T.cum[mid] <= target) lo = mid; else hi = mid - 1;
        }
    }
    return T.q_lo + ((double)lo + u2) * T.dq;
}

// Alg. 4: xi(|r|) by linear interpolation on its grid (constant beyond it)
__device__ __forceinline__ double xi_lerp(const double *tab, double h, double r)
{
    const double a = fabs(r) / h;
    if (!(a < (double)kXiN)) return tab[kXiN];
    const int j = (int)a;
    const double t = a - (double)j;
    return tab[j] + t * (tab[j + 1] - tab[j]);
}

// Alg. 4: kick from V_W^+(x, .)/xi(x) by rejection (proposal from the Gaussian
// majorant, accept iff u < [sgnV sin(2 q r)]^+); false if every proposal failed.
__device__ __forceinline__ bool reject_kick(const Dev &d, const InstParam &P, uint64_t id,
                                            uint32_t step, uint32_t e, int m, double r, double &q_out)
{
    const double sgv = P.H[m] >= 0.0 ? 1.0 : -1.0;
    for (uint32_t i = 0; i < kRejectMax; ++i) {
        const uint32_t ev = e + (i << 12);
        const W4 a = draw(id, step, kTagReject, ev, (uint32_t)m, d.seed, P.key);
        const W4 b = draw(id, step, kTagReject, ev, (uint32_t)(4 + m), d.seed, P.key);
        const double R = sqrt(-2.0 * ln_series(1.0 - unit53(a.a, a.b)));
        const double q = (R * cos_det(kTwoPi * unit53(a.c, a.d))) * P.sq[m];
        const double p = sgv * sin_det((2.0 * q) * r);
        if (unit53(b.a, b.b) < p) { q_out = q; return true; }
    }
    return false;
}

template <int DIM>
__device__ __forceinline__ bool in_kbox(const Dev &d, const double *k)
{
    if (!(k[0] >= d.k_lo && k[0] < d.k_hi)) return false;
    if (DIM == 2 && !(k[1] >= d.k_lo && k[1] < d.k_hi)) return false;
    return true;
}


// ---------------------------------------------------------------------------
// Family trees of event parents
// ---------------------------------------------------------------------------
// Kick and weight of a created pair (see draw_pair).
struct PairDraw {
    double q, arg, sn, sigma, amp;
};

struct Node {
    double x[2], k[2];   // position at t0, wave vector
    double t0;           // start of this particle's walk within the step
    double w;            // sp2 weight
    double D[3];         // tangent
    uint64_t id;
    int32_t sg;          // sp1 sign, 0 for a ghost
    int32_t depth;
    double t;            // time of its latest jump (t0 before the first)
    double te;           // time of the jump being expanded
    double xe[2];        // position at te
    double ua0;          // acceptance uniform of component 0
    uint32_t e;          // jump index
    int32_t m, side, in_ev;
};

// True if the clock draw u certainly gives no jump before the end of the
// step for a clock running from t, i.e. t - ln(1-u)/gamma0 > dt as the exact
// test evaluates it.  -ln(1-u) >= u makes u > gamma0 (dt - t) sufficient in
// exact arithmetic; the relative 2^-30 and absolute dt 2^-40 margins cover
// the rounding of the exact test (the logarithm within a few ulp, the
// division, the sum compared with dt).  Only draws below the bound (a few
// percent) pay for the logarithm.
__device__ __forceinline__ bool surely_no_jump(double u, double t, double dt, double g0)
{
    return u > g0 * ((dt - t) * (1.0 + 0x1p-30) + dt * 0x1p-40);
}

struct Tally {
    int64_t events, pairs, killed, cap;
    int32_t maxdepth;
};

// Pair decision and kick of component m at jump e of particle `id`
// (Alg. 1 rules 3-5 with the majorant sampler of Remark 3, or Alg. 4):
// returns false if no pair is created.

// ONE: a single static Gaussian component with the majorant sampler.
template <int DIM, bool SP2, bool ONE>
__device__ __forceinline__ bool draw_pair(const Dev &d, const InstParam &P, uint64_t id, uint32_t step,
                                          uint32_t e, int m, const double *xe, double te, double ua0,
                                          double w, PairDraw &J)
{
    const uint32_t seed = d.seed, key = P.key;
    double cm = P.c[m], sgv = P.sgnV[m];
    bool alg4 = false;
    if (!ONE && d.sampler[m] == 1) {
        // Alg. 1 sp1 box with Pr = xi(x)/gamma0, kick by Alg. 4
        const double r = phase_offset<DIM>(d, m, xe, P.center[m]);
        double ua = ua0;
        if (m > 0) {
            const W4 ra = draw(id, step, kTagStep, e, (uint32_t)(8 + m), seed, key);
            ua = unit53(ra.a, ra.b);
        }
        const double *tab = d.xi_tab + ((int64_t)(&P - d.ip) * d.M + m) * (kXiN + 1);
        double qk = 0.0;
        if (!(ua < xi_lerp(tab, P.xi_h[m], r) / P.gamma0) || !reject_kick(d, P, id, step, e, m, r, qk))
            return false;
        J.q = qk;
        J.arg = (2.0 * qk) * r;
        J.sn = 1.0;
        sgv = 1.0;
        alg4 = true;
    } else {
        const W4 rq = draw(id, step, kTagStep, e, (uint32_t)(1 + m), seed, key);
        J.q = kick_sample<ONE>(d, P, m, unit53(rq.a, rq.b), unit53(rq.c, rq.d));
        J.arg = (2.0 * J.q) * phase_offset<DIM>(d, m, xe, P.center[m]);
        J.sn = sin_det(J.arg);
    }
    if (!ONE && d.tdep && d.kind[m] == 0 && !alg4) {   // Remark 1: kernel at the absolute jump time
        const double tabs = (double)step * d.dt + te;
        const double f = P.ma[m] + P.mb[m] * cos_det(P.mw[m] * tabs + P.mp[m]);
        const double He = P.H[m] * f;
        cm = ((2.0 * fabs(He)) / d.hbar) / (2.0 * P.gamma0);
        sgv = He >= 0.0 ? 1.0 : -1.0;
    }
    J.sigma = (J.sn > 0.0) ? sgv : -sgv;
    J.amp = 0.0;
    if (!SP2 && !alg4) {
        double ua = ua0;
        if (m > 0) {
            const W4 ra = draw(id, step, kTagStep, e, (uint32_t)(8 + m), seed, key);
            ua = unit53(ra.a, ra.b);
        }
        if (!(ua < cm * fabs(J.sn))) return false;   // no pair: only the survivor continues
    } else if (SP2) {
        J.amp = w * (cm * fabs(J.sn));
    }
    return true;
}

// Offspring `side` (0: "+", 1: "-") of the pair J of component m at jump e;
// rc is the child-id draw of (parent, e, m).  Sets k, sign, weight, id and
// tangent of ch.
template <int DIM>
__device__ __forceinline__ void child_id_k(const Dev &d, const Node &par, uint64_t cls, int m, int side,
                                           const PairDraw &J, const W4 &rc, Node &ch)
{
    ch.id = side == 0 ? ((cls << 62) | ((uint64_t)(rc.b & 0x3FFFFFFFu) << 32) | (uint64_t)rc.a)
                      : ((cls << 62) | ((uint64_t)(rc.d & 0x3FFFFFFFu) << 32) | (uint64_t)rc.c);
    const double kick = J.sigma * J.q;
    ch.k[0] = par.k[0];
    ch.k[1] = par.k[1];
    const int ax = DIM == 1 ? 0 : d.axis[m];
    if (ax == 0) {
        ch.k[0] = side == 0 ? par.k[0] + kick : par.k[0] - kick;
    } else if (ax == 1) {
        ch.k[1] = side == 0 ? par.k[1] + kick : par.k[1] - kick;
    } else {
        ch.k[0] = side == 0 ? par.k[0] + kick : par.k[0] - kick;
        ch.k[1] = side == 0 ? par.k[1] - kick : par.k[1] + kick;
    }
}

template <int DIM, bool SP2, bool TAN>
__device__ __forceinline__ void make_child(const Dev &d, const InstParam &P, const Node &par, int m, int side,
                                           const PairDraw &J, const W4 &rc, Node &ch)
{
    const uint64_t cls = ((par.id >> 62) & 1ull) ? 3ull : 2ull;   // ghost lineages keep bit 62
    child_id_k<DIM>(d, par, cls, m, side, J, rc, ch);
    ch.sg = side == 0 ? par.sg : -par.sg;
    ch.w = side == 0 ? J.amp : -J.amp;
    if constexpr (TAN && SP2) {
        // The wp pair adds w c sgn(V) sin(2qr) [f(k+q) - f(k-q)] with q drawn
        // from G/xi_hat.  Differentiating its expectation: c times the kick
        // density is G/(2 gamma0), whose log-derivative is (1/H, 1/w - 4wq^2, 0);
        // the parent's weight carries D; sin(2q(x - x0)) has x0-derivative
        // -2q cos.  In the children's frame (k +/- sigma q, weights
        // +/- w c|sin|) the "+" child carries
        // X = c|sin| (D + w dlogG) + w c sgn(sin) dsin, the "-" child -X.
        const double wd = P.width[m];
        const double s0 = 1.0 / P.H[m];
        const double s1 = 1.0 / wd - ((4.0 * wd) * J.q) * J.q;
        // tangents require a static kernel, so c is the instance's constant
        const double cm = P.c[m];
        const double a = cm * fabs(J.sn);
        const double g = par.w * (cm * (J.sn > 0.0 ? 1.0 : -1.0));
        const double x0 = a * (par.D[0] + par.w * s0);
        const double x1 = a * (par.D[1] + par.w * s1);
        const double x2 = a * par.D[2] + g * (-(2.0 * J.q) * cos_det(J.arg));
        const double sdir = side == 0 ? 1.0 : -1.0;
        ch.D[0] = sdir * x0;
        ch.D[1] = sdir * x1;
        ch.D[2] = sdir * x2;
    } else if constexpr (TAN) {
        const double wd = P.width[m];
        const double s0 = 1.0 / P.H[m];
        const double s1 = 1.0 / wd - ((4.0 * wd) * J.q) * J.q;
        // tangent mode 2 carries the x0 derivative by derivative pairs instead
        const double s2 = d.tangent == 2 ? 0.0 : -(2.0 * J.q) * (cos_det(J.arg) / J.sn);
        const double sdir = side == 0 ? 1.0 : -1.0;
        const double sgd = (double)ch.sg;
        ch.D[0] = sdir * par.D[0] + sgd * s0;
        ch.D[1] = sdir * par.D[1] + sgd * s1;
        ch.D[2] = sdir * par.D[2] + sgd * s2;
    } else {
        ch.D[0] = ch.D[1] = ch.D[2] = 0.0;
    }
}

// Derivative pair of component m at jump e (tangent mode 2).  The pair
// intensity per unit kick density, c sin(2 q (x - x0)), depends on x0 only
// through the sine, whose x0-derivative gives -2 q c cos(2 q (x - x0)).
// With the jump's own kick q and an independent uniform, a pair of ghosts
// is created with probability c |cos|, directed by sgn(F[V]) sgn(cos); the
// "+" ghost carries the x0-tangent -2 q s and the "-" ghost +2 q s (s the
// parent's sign).  Its expectation is the x0-derivative of the signed pair
// measure with a tangent bounded by 2|q|, where the score -2q cot(2 q r) has
// infinite variance.  Returns false if no pair is created.
__device__ __forceinline__ bool draw_deriv(const Dev &d, const InstParam &P, uint64_t id, uint32_t step,
                                           uint32_t e, int m, const double *xe, PairDraw &J)
{
    const W4 rq = draw(id, step, kTagStep, e, (uint32_t)(1 + m), d.seed, P.key);
    const W4 ru = draw(id, step, kTagDeriv, e, (uint32_t)m, d.seed, P.key);
    J.q = kick_sample<true>(d, P, m, unit53(rq.a, rq.b), unit53(rq.c, rq.d));
    J.arg = (2.0 * J.q) * phase_offset<1>(d, m, xe, P.center[m]);
    const double cs = cos_det(J.arg);
    if (!(unit53(ru.a, ru.b) < P.c[m] * fabs(cs))) return false;
    J.sn = cs;
    J.sigma = (cs > 0.0) ? P.sgnV[m] : -P.sgnV[m];
    J.amp = 0.0;
    return true;
}

// Ghost `side` of the derivative pair J (rc: its id draw); ghost lineage ids.
__device__ __forceinline__ void make_deriv_child(const Dev &d, const Node &par, int m, int side,
                                                 const PairDraw &J, const W4 &rc, Node &ch)
{
    child_id_k<1>(d, par, 3ull, m, side, J, rc, ch);
    ch.sg = 0;
    ch.w = 0.0;
    const double dx0 = (2.0 * J.q) * (double)par.sg;
    ch.D[0] = 0.0;
    ch.D[1] = 0.0;
    ch.D[2] = side == 0 ? -dx0 : dx0;
}

// k-truncation tally of a child that left the k-box (Sec. 2)
template <bool SP2>
__device__ __forceinline__ int64_t killed_amount(const Node &ch)
{
    if (SP2) {
        const int64_t q32 = (int64_t)floor(fabs(ch.w) * 4294967296.0);
        return ch.w < 0.0 ? -q32 : q32;
    }
    return ch.sg;
}

// The block's overflow area of the pool (see kGPool): field f of record g
// is at f * kGPool + g of the doubles.
struct GPoolView {
    double *f;
    uint64_t *id;
    int8_t *sg;
};
__device__ __forceinline__ GPoolView gpool_view(const Dev &d)
{
    char *b = d.gpool + (size_t)blockIdx.x * kGPoolBytes;
    return {(double *)b, (uint64_t *)(b + (size_t)8 * 8 * kGPool), (int8_t *)(b + (size_t)9 * 8 * kGPool)};
}
__device__ __forceinline__ uint32_t gpool_cap(const Dev &d)
{
    return (int)blockIdx.x < d.gpool_blocks ? (uint32_t)kGPool : 0u;
}

// Pair slots of a jump in walk_family: components 0..M-1, then (tangent
// mode 2, signed particles) their derivative pairs as slots M..2M-1.  Without
// tangents these are exactly the pair draw and make_child.
template <bool TAN>
__device__ __forceinline__ int slot_end(const Dev &d, const Node &cur, int M)
{
    if constexpr (TAN) return (d.tangent == 2 && cur.sg != 0) ? 2 * M : M;
    else return M;
}

template <int DIM, bool SP2, bool TAN, bool ONE>
__device__ __forceinline__ bool slot_draw(const Dev &d, const InstParam &P, const Node &cur, uint32_t step,
                                          int slot, int M, PairDraw &J, W4 &rc)
{
    if constexpr (TAN) {
        if (slot >= M) {
            if (!draw_deriv(d, P, cur.id, step, cur.e, slot - M, cur.xe, J)) return false;
            rc = draw(cur.id, step, kTagDeriv, cur.e, (uint32_t)(8 + slot - M), d.seed, P.key);
            return true;
        }
    }
    if (!draw_pair<DIM, SP2, ONE>(d, P, cur.id, step, cur.e, slot, cur.xe, cur.te, cur.ua0, cur.w, J)) return false;
    rc = draw(cur.id, step, kTagChild, cur.e, (uint32_t)slot, d.seed, P.key);
    return true;
}

template <int DIM, bool SP2, bool TAN>
__device__ __forceinline__ void slot_child(const Dev &d, const InstParam &P, const Node &cur, int slot, int M,
                                           int side, const PairDraw &J, const W4 &rc, Node &ch)
{
    if constexpr (TAN) {
        if (slot >= M) {
            make_deriv_child(d, cur, slot - M, side, J, rc, ch);
            return;
        }
    }
    make_child<DIM, SP2, TAN>(d, P, cur, slot, side, J, rc, ch);
}

// General depth-first walk of one family (any number of jumps and levels),
// by one lane: the path of the tiles whose families the pool below cannot
// hold.  Counting (emit false) tallies and counts the records; emitting
// writes every record, the r-th as offspring first_rec + r (< cap) of the
// tile's pages (more: the further ones, see page_slot).  Its stack makes it large, so it is
// a function of its own: the common path keeps its registers.
template <int DIM, bool SP2, bool TAN>
__device__ __noinline__ uint32_t walk_family(const Dev *dp, int b, uint32_t step, const Node *root, bool emit,
                                             Ens out, int64_t base, int64_t first_rec, int64_t cap,
                                             const uint32_t *pages, const uint32_t *more, int sh, int64_t dstride, Tally *tl,
                                             uint32_t *err)
{
    const Dev &d = *dp;
    const InstParam &P = d.ip[b];
    Node stack[kMaxDepth];
    PairDraw stackJ[kMaxDepth];
    W4 stackR[kMaxDepth];
    Node cur = *root;
    int sp = 0;
    uint32_t nrec = 0;
    const uint32_t seed = d.seed, key = P.key;
    const int M = d.M;
    cur.t = cur.t0;
    cur.e = 0;
    cur.in_ev = 0;
    cur.depth = 0;
    for (;;) {
        if (!cur.in_ev) {
            bool done = false;
            if (cur.e >= kEventCap) {
                if (!emit) tl->cap++;
                done = true;
            } else {
                const W4 r = draw(cur.id, step, kTagStep, cur.e, 0u, seed, key);
                const double u = unit53(r.a, r.b);
                const double te = surely_no_jump(u, cur.t, d.dt, P.gamma0)
                                      ? d.dt + 1.0 : cur.t + (-ln_series(1.0 - u) / P.gamma0);
                if (!(te <= d.dt)) {
                    done = true;
                } else {
                    if (!emit) tl->events++;
                    cur.te = te;
                    cur.ua0 = unit53(r.c, r.d);
                    cur.xe[0] = cur.x[0] + (d.vfac * cur.k[0]) * (te - cur.t0);
                    if (DIM == 2) cur.xe[1] = cur.x[1] + (d.vfac * cur.k[1]) * (te - cur.t0);
                    else cur.xe[1] = 0.0;
                    cur.in_ev = 1;
                    cur.m = 0;
                    cur.side = 0;
                }
            }
            if (done) {
                if (sp == 0) break;
                cur = stack[--sp];
                continue;
            }
        }
        if (cur.m >= slot_end<TAN>(d, cur, M)) {
            cur.t = cur.te;
            cur.e += 1u;
            cur.in_ev = 0;
            continue;
        }
        const int m = cur.m;
        PairDraw J;
        W4 rc;
        if (cur.side == 0) {
            if (!slot_draw<DIM, SP2, TAN, false>(d, P, cur, step, m, M, J, rc)) {
                cur.m += 1;
                continue;
            }
            if (!emit && (!TAN || m < M)) tl->pairs++;
        } else {
            J = stackJ[sp];        // saved when this frame descended into its "+" offspring
            rc = stackR[sp];
        }
        bool descend = false;
        Node ch;
        for (int side = cur.side; side < 2 && !descend; ++side) {
            slot_child<DIM, SP2, TAN>(d, P, cur, m, M, side, J, rc, ch);
            if (!in_kbox<DIM>(d, ch.k)) {          // k-truncation (Sec. 2)
                if (!emit) tl->killed += killed_amount<SP2>(ch);
                continue;
            }
            if (emit) {
                const int64_t li = first_rec + nrec;
                if (li < cap) {
                    const int64_t o = base + page_slot(pages, sh, (uint32_t)li, [&] { return more; });
                    out.x0[o] = cur.xe[0] + (d.vfac * ch.k[0]) * (d.dt - cur.te);
                    out.k0[o] = ch.k[0];
                    if (DIM == 2) {
                        out.x1[o] = cur.xe[1] + (d.vfac * ch.k[1]) * (d.dt - cur.te);
                        out.k1[o] = ch.k[1];
                    }
                    if (SP2) out.w[o] = ch.w; else out.sg[o] = (int8_t)ch.sg;
                    out.id[o] = ch.id;
                    if (TAN) {
                        out.D[o] = ch.D[0];
                        out.D[dstride + o] = ch.D[1];
                        out.D[2 * dstride + o] = ch.D[2];
                    }
                } else {
                    *err |= kErrCapacity;
                }
            }
            nrec++;
            ch.depth = cur.depth + 1;
            if (!emit && ch.depth > tl->maxdepth) tl->maxdepth = ch.depth;
            // The child's first clock draw, exactly as its own walk would take
            // it: most children do not jump before the end of the step, and
            // then there is nothing to walk and the parent stays off the stack.
            const W4 r0 = draw(ch.id, step, kTagStep, 0u, 0u, seed, key);
            const double u0 = unit53(r0.a, r0.b);
            if (surely_no_jump(u0, cur.te, d.dt, P.gamma0) ||
                !(cur.te + (-ln_series(1.0 - u0) / P.gamma0) <= d.dt))
                continue;
            if (sp >= kMaxDepth) {
                *err |= kErrDepth;
                continue;
            }
            // descend into the child; the parent resumes with its "-"
            // offspring (pair kept with the frame) or its next component
            if (side == 0) {
                stackJ[sp] = J;
                stackR[sp] = rc;
                cur.side = 1;
            } else {
                cur.side = 0;
                cur.m += 1;
            }
            descend = true;
        }
        if (!descend) {
            cur.side = 0;
            cur.m += 1;
            continue;
        }
        ch.x[0] = cur.xe[0];
        ch.x[1] = cur.xe[1];
        ch.t0 = cur.te;
        ch.t = ch.t0;
        ch.e = 0;
        ch.in_ev = 0;
        ch.m = 0;
        ch.side = 0;
        stack[sp++] = cur;
        cur = ch;
    }
    return nrec;
}

// ---------------------------------------------------------------------------
// The families of a tile, jump by jump.  A unit of work is one jump of one
// particle: its pair decisions, its offspring with their first clock draws,
// and the jumping particle's next clock draw.  Round 0 takes the parents'
// first jumps, one per lane; every further jump found (the particle's next
// one, or an offspring's first) goes to a queue in LDS and is taken in the
// next round, the queue's jumps side by side in the first lanes.  A tile's
// critical path is then its longest chain of jumps (2 to 4 for the barriers)
// at about a thousand instructions each, and a rare second jump costs one
// lane of a full round instead of a walk of its own.
//
// Every kept offspring is a record of the tile's pool.  Its place in the
// canonical depth-first order is its path: one byte per level (jump index
// + 1, pair slot, side), left-aligned in 64 bits, so that an unsigned
// comparison orders a family's records (a node before its offspring).  The
// records of a family are linked, and a record's rank is the number of its
// family's smaller paths.  A particle that jumps again is referred to by its
// record (a parent by a pool entry with path 0, which is no output).
//
// Payloads past kLds go to the block's overflow area in HBM (4D), the paths
// and links stay in LDS.  Parents whose records, queue, levels (8) or jump
// indexes (15) do not fit are taken again: half as many at a time, or, where a
// path does not fit or they are few already, by walk_family.
// Dev::ftile, the parents taken at first, is chosen so that this is rare.
// ---------------------------------------------------------------------------
template <int DIM, bool SP2, bool TAN>
struct Families {
    static constexpr int kLds = DIM == 2 ? (SP2 ? 332 : 384) : 512;           // records whose payload is in LDS
    static constexpr int kRec = kLds + (DIM == 2 ? kGPool : 0); // records in all
    static constexpr int kQueue = DIM == 2 ? 192 : 128;         // further jumps of a round
    static constexpr int kLevels = 8;
    // records
    uint64_t key[kRec], id[kLds];
    double x0[kLds], k0[kLds];
    double x1[DIM == 2 ? kLds : 1], k1[DIM == 2 ? kLds : 1];
    double w[SP2 ? kLds : 1];
    double D[TAN ? 3 : 1][TAN ? kLds : 1];
    uint16_t slot[kRec], next[kRec];
    int8_t sg[kLds];
    // jumps of the next round
    double qx0[kQueue], qx1[DIM == 2 ? kQueue : 1], qt0[kQueue], qte[kQueue], qua[kQueue];
    uint16_t qrec[kQueue], qe[kQueue];
    // per family
    uint32_t cnt[kThreads], first[kThreads];
    uint32_t head[kThreads];
    uint32_t n, nq[2];
    uint32_t overflow;            // bits: 1 records or jumps, 2 paths that do not fit
    uint32_t events, pairs, maxdepth;
    long long killed;
};

constexpr uint32_t kNone = 0xFFFFu;

// Puts node `ch` with path `key` into the pool (end-of-step position from
// the jump at xe, te; a parent's entry has path 0 and is not linked) and
// returns its index, or kNone if the pool is full.
template <int DIM, bool SP2, bool TAN>
__device__ __forceinline__ uint32_t add_record(const Dev &d, Families<DIM, SP2, TAN> &F, uint64_t key, int slot,
                                               const double *xe, double te, const Node &ch)
{
    using FT = Families<DIM, SP2, TAN>;
    const uint32_t r = atomicAdd(&F.n, 1u);
    if (r >= (uint32_t)FT::kRec || (DIM == 2 && r >= (uint32_t)FT::kLds && r - (uint32_t)FT::kLds >= gpool_cap(d))) {
        atomicOr(&F.overflow, 1u);
        return kNone;
    }
    const double x0 = xe[0] + (d.vfac * ch.k[0]) * (d.dt - te);
    const double x1 = DIM == 2 ? xe[1] + (d.vfac * ch.k[1]) * (d.dt - te) : 0.0;
    F.key[r] = key;
    F.slot[r] = (uint16_t)slot;
    if (key) {
        F.next[r] = (uint16_t)atomicExch(&F.head[slot], r);
        atomicAdd(&F.cnt[slot], 1u);
    }
    if (DIM == 1 || r < (uint32_t)FT::kLds) {
        F.x0[r] = x0;
        F.k0[r] = ch.k[0];
        if (DIM == 2) {
            F.x1[r] = x1;
            F.k1[r] = ch.k[1];
        }
        if (SP2) F.w[r] = ch.w; else F.sg[r] = (int8_t)ch.sg;
        F.id[r] = ch.id;
        if (TAN) {
            F.D[0][r] = ch.D[0];
            F.D[1][r] = ch.D[1];
            F.D[2][r] = ch.D[2];
        }
        return r;
    }
    const uint32_t g = r - (uint32_t)FT::kLds;
    const GPoolView v = gpool_view(d);
    v.f[g] = x0;
    v.f[kGPool + g] = ch.k[0];
    if (DIM == 2) {
        v.f[2 * kGPool + g] = x1;
        v.f[3 * kGPool + g] = ch.k[1];
    }
    if (SP2) v.f[4 * kGPool + g] = ch.w; else v.sg[g] = (int8_t)ch.sg;
    if (TAN) {
        v.f[5 * kGPool + g] = ch.D[0];
        v.f[6 * kGPool + g] = ch.D[1];
        v.f[7 * kGPool + g] = ch.D[2];
    }
    v.id[g] = ch.id;
    return r;
}

// Record r's node (its end-of-step position in x): for the particles that
// jump again, and for the output.
template <int DIM, bool SP2, bool TAN>
__device__ __forceinline__ void load_record(const Dev &d, const Families<DIM, SP2, TAN> &F, uint32_t r, Node &n)
{
    using FT = Families<DIM, SP2, TAN>;
    n.x[1] = n.k[1] = n.w = n.D[0] = n.D[1] = n.D[2] = 0.0;
    n.sg = 0;
    if (DIM == 1 || r < (uint32_t)FT::kLds) {
        n.x[0] = F.x0[r];
        n.k[0] = F.k0[r];
        if (DIM == 2) {
            n.x[1] = F.x1[r];
            n.k[1] = F.k1[r];
        }
        if (SP2) n.w = F.w[r]; else n.sg = F.sg[r];
        n.id = F.id[r];
        if (TAN) {
            n.D[0] = F.D[0][r];
            n.D[1] = F.D[1][r];
            n.D[2] = F.D[2][r];
        }
        return;
    }
    const uint32_t g = r - (uint32_t)FT::kLds;
    const GPoolView v = gpool_view(d);
    n.x[0] = v.f[g];
    n.k[0] = v.f[kGPool + g];
    if (DIM == 2) {
        n.x[1] = v.f[2 * kGPool + g];
        n.k[1] = v.f[3 * kGPool + g];
    }
    if (SP2) n.w = v.f[4 * kGPool + g]; else n.sg = v.sg[g];
    if (TAN) {
        n.D[0] = v.f[5 * kGPool + g];
        n.D[1] = v.f[6 * kGPool + g];
        n.D[2] = v.f[7 * kGPool + g];
    }
    n.id = v.id[g];
}

// A further jump, at te, of the particle in record rec born at (x, t0).
template <int DIM, bool SP2, bool TAN>
__device__ __forceinline__ void add_jump(Families<DIM, SP2, TAN> &F, int round, const double *x, double t0, double te,
                                         double ua, uint32_t rec, uint32_t e)
{
    using FT = Families<DIM, SP2, TAN>;
    const uint32_t q = atomicAdd(&F.nq[round & 1], 1u);
    if (q >= (uint32_t)FT::kQueue || rec == kNone) {
        atomicOr(&F.overflow, 1u);
        return;
    }
    F.qx0[q] = x[0];
    if (DIM == 2) F.qx1[q] = x[1];
    F.qt0[q] = t0;
    F.qte[q] = te;
    F.qua[q] = ua;
    F.qrec[q] = (uint16_t)rec;
    F.qe[q] = (uint16_t)e;
}

// One jump: particle cur (x, k at its birth time t0) jumps at te, its e-th
// jump of the step, in family `slot`, with path `key` of `lev` levels.  rec:
// its record, or kNone for a parent's first jump.  The caller takes the pair
// slots m0, m0 + mstep, ... (other wavefronts the others), and with m0 = 0
// what the jump has once.
template <int DIM, bool SP2, bool TAN, bool ONE>
__device__ __forceinline__ void take_jump(const Dev &d, const InstParam &P, uint32_t step, int round, Node &cur,
                                          uint64_t key, int lev, int slot, uint32_t rec, int m0, int mstep,
                                          Families<DIM, SP2, TAN> &F)
{
    using FT = Families<DIM, SP2, TAN>;
    const uint32_t seed = d.seed, pk = P.key;
    const int M = ONE ? 1 : d.M;
    const double te = cur.te, g0 = P.gamma0;
    if (lev >= FT::kLevels || cur.e >= 15u) {
        atomicOr(&F.overflow, 2u);
        return;
    }
    const int sh = 56 - 8 * lev;
    cur.xe[0] = cur.x[0] + (d.vfac * cur.k[0]) * (te - cur.t0);
    cur.xe[1] = DIM == 2 ? cur.x[1] + (d.vfac * cur.k[1]) * (te - cur.t0) : 0.0;
    const int mend = slot_end<TAN>(d, cur, M);
    for (int m = m0; m < mend; m += mstep) {
        PairDraw J;
        W4 rc;
        if (!slot_draw<DIM, SP2, TAN, ONE>(d, P, cur, step, m, M, J, rc)) continue;
        if (!TAN || m < M) atomicAdd(&F.pairs, 1u);
        const uint64_t base = key | ((uint64_t)(((cur.e + 1u) << 4) | ((uint32_t)m << 1)) << sh);
        // both offspring, then the first clock draws of those that may jump
        // again before the end of the step (a few percent): the logarithm
        // is shared by the two
        Node ch;
        uint32_t rr[2], pend = 0u;
        double uu[2], ua[2];
#pragma unroll
        for (int side = 0; side < 2; ++side) {
            slot_child<DIM, SP2, TAN>(d, P, cur, m, M, side, J, rc, ch);
            const W4 l = draw(ch.id, step, kTagStep, 0u, 0u, seed, pk);
            uu[side] = unit53(l.a, l.b);
            ua[side] = unit53(l.c, l.d);
            rr[side] = kNone;
            if (in_kbox<DIM>(d, ch.k)) {
                rr[side] = add_record<DIM, SP2, TAN>(d, F, base | ((uint64_t)side << sh), slot, cur.xe, te, ch);
                if (!surely_no_jump(uu[side], te, d.dt, g0)) pend |= 1u << side;
            } else {                                       // k-truncation (Sec. 2)
                atomicAdd((unsigned long long *)&F.killed, (unsigned long long)killed_amount<SP2>(ch));
            }
        }
        while (pend) {
            const bool s0 = pend & 1u;
            const double tc = te + (-ln_series(1.0 - (s0 ? uu[0] : uu[1])) / g0);
            if (tc <= d.dt)
                add_jump<DIM, SP2, TAN>(F, round, cur.xe, te, tc, s0 ? ua[0] : ua[1], s0 ? rr[0] : rr[1], 0u);
            pend &= s0 ? 2u : 0u;
        }
    }
    if (m0 != 0) return;
    atomicAdd(&F.events, 1u);
    const W4 rn = draw(cur.id, step, kTagStep, cur.e + 1u, 0u, seed, pk);
    const double un = unit53(rn.a, rn.b);
    if (!surely_no_jump(un, te, d.dt, g0)) {
        const double tn = te + (-ln_series(1.0 - un) / g0);
        if (tn <= d.dt) {
            if (rec == kNone) rec = add_record<DIM, SP2, TAN>(d, F, 0ull, slot, cur.xe, te, cur);
            add_jump<DIM, SP2, TAN>(F, round, cur.x, cur.t0, tn, unit53(rn.c, rn.d), rec, cur.e + 1u);
        }
    }
}

}  // namespace wbrw
