// Per-target neighbour search on the uniform grid, G lanes per target.
//
// Selection follows the PCMS paper, Section 3.2.1: the source set of target
// t is { s_j : phi(s_j, t) > 0 }, i.e. the sources strictly inside the
// support radius.  The distance is the metric
//     D = fma(u_{d-1}, u_{d-1}, ... fma(u_1, u_1, u_0 * u_0)),
//     u_k = (t_k - s_k) * g_k,
// evaluated in FP64 in this exact order, so the predicate D < r^2 is bit
// reproducible.  The radius is fixed, grown by doubling r^2 until a minimum
// count is met (Section 3.2.1), or set to the k-th smallest D.  Above k_cap
// sources the k_cap smallest by (D, source index) are kept.
//
// Stencil walk: buckets are row-major with dimension 0 fastest, so for every
// row (c_1..c_{d-1}) the buckets c_0 in [a, b] form one contiguous range of
// sorted sources.  Only rows whose slab is within the radius are visited and
// each row's c_0 range is narrowed to the chord of the ball in that slab.
// The G lanes of a target walk the same rows (uniform control flow) and take
// the candidates of a row in an interleaved order; candidates reach the
// per-step callback in ascending sorted order, which the ordered compaction
// of the lists preserves.
//
// Selection reads the sources' FP32 records and decides by thresholds moved
// apart by a proven bound on the FP32 error; the few candidates between them
// are decided from their FP64 records, so the lists are those of the FP64
// predicate.
#pragma once

#include <type_traits>

#include "bvh.h"
#include "device_common.h"

namespace pcms {

// Candidates per walk step whose loads are issued together: FP64 records
// (two 16-byte loads each in 3-D) and FP32 records (a lane's are adjacent and
// load as whole 16-byte words: three words for four 3-D sources).  The
// FP64 walks are the general path's, which targets in strongly non-uniform
// clouds take.  With two and four records, 300k graded sources, 200k targets:
// kNN 3-D linear 11636 and 9556 us, growing radius 2-D 8986 and 7512, 3-D 12840
// and 10927; on the tree, 600k sources with far outliers, 3-D linear 108159 and
// 104272, quadratic MIXED_REFINE 100651 and 91445.
constexpr int kBatch64 = 4, kBatch32 = 4;

// Bins of the windowed selection.
constexpr int kMaxBins = 64;

template <int D, bool UNIT>
PCMS_HD PCMS_INLINE double metric_d2(const double (&t)[D], const double *__restrict__ s,
                                     const GridParams &p)
{
    double u = UNIT ? (t[0] - s[0]) : (t[0] - s[0]) * p.g[0];
    double acc = u * u;
#pragma unroll
    for (int k = 1; k < D; ++k) {
        u = UNIT ? (t[k] - s[k]) : (t[k] - s[k]) * p.g[k];
        acc = __builtin_fma(u, u, acc);
    }
    return acc;
}

// Fraction of the unit d-ball's volume beyond the hyperplane at distance x
// (0 <= x <= 1) from its centre: the integral of (1 - s^2)^((d-1)/2) over
// [x, 1] over its integral over [-1, 1] (d = 1, 2, 3).
template <int D>
PCMS_HD PCMS_INLINE double ball_beyond(double x)
{
    static_assert(D >= 1 && D <= 3, "closed forms for 1-3 dimensions");
    auto P = [](double s) {
        if constexpr (D == 1) return s;
        else if constexpr (D == 2) return 0.5 * (s * sqrt(fmax(1.0 - s * s, 0.0)) + asin(s));
        else return s - s * s * s / 3.0;
    };
    x = fmin(fmax(x, 0.0), 1.0);
    return (P(1.0) - P(x)) / (P(1.0) - P(-1.0));
}

// Rows of a stencil walk: for radius rho around t, the rows (bucket
// coordinates c_1..c_{d-1}) within reach, each with the range of sorted
// sources in the ball's chord of that row, last row first (DOWN) or first row
// first, kRows rows of consecutive c_1 at a time so that their bucket offsets
// are loaded together.
//
// All distances are in bucket widths (every dimension above 0 with more than
// one bucket has the metric width gp.wm, dimension 0 the width wm / sub) and
// relative to t's own bucket, so for t within the grid FP32 holds its offset
// to 1e-7 of a width however many buckets there are.  The c_1 of a line (fixed
// c_2..c_{d-1}) are those of the chord in that line, so no row out of reach is
// visited.  Every rounding is covered by slack that can only widen a range:
// 2e-5 of a width, 4e-6 relative on rho^2 and 2e-6 on a chord (the bucket
// assignment rounds by far less).  The relative slack also covers t beyond the
// grid, whose offset FP32 holds to 6e-8 of itself, as a ball that reaches the
// grid is no smaller than the offset.  Offsets are clamped at kFar widths: a
// radius up to kFar cannot reach beyond them, and a larger one takes every
// row, as its rho^2 then exceeds the sum of the clamped offsets' squares.
constexpr int kRows = 4;
constexpr double kFar = 1e15;
// Beyond the last bucket from any (a grid has at most 2^30, and the sum of two
// still fits an int).
constexpr float kFarBuckets = 1073741824.0f;

template <int D, bool DOWN>
struct RowLines {
    const GridParams &gp;
    const int *__restrict__ cs;
    float rho2;      // squared radius in bucket widths
    int ct[D];       // t's bucket (clamped to the grid)
    float fr[D];     // t's offset from that bucket's lower edge
    int c[D];        // current buckets of dimensions >= 1, relative to ct ...
    int a[D], b[D];  // ... and their ranges
    float outer;     // squared distance to the slabs of dimensions >= 2
    int row;         // first bucket of the row with c_1 = 0
    bool more;

    PCMS_HD PCMS_INLINE RowLines(const GridParams &gp_, const int *cs_, const double (&t)[D], double r2)
        : gp(gp_), cs(cs_), outer(0.0f), row(0), more(true)
    {
        const double iw = 1.0 / gp.wm;
        const double x2 = r2 * iw * iw * (1.0 + 4e-6);
        rho2 = x2 <= kFar * kFar ? (float)x2 : 1e37f;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const double u = (t[k] - gp.lo[k]) * gp.inv_w[k];
            ct[k] = (int)fmin(fmax(floor(u), 0.0), (double)(gp.n[k] - 1));
            // (a single bucket reaches everywhere; a flat dimension's width is not wm)
            fr[k] = gp.n[k] > 1 ? (float)fmin(fmax(u - (double)ct[k], -kFar), kFar) : 0.5f;
            if (k >= 1) row += ct[k] * gp.stride[k];
        }
        if constexpr (D >= 3) {
#pragma unroll
            for (int k = 2; k < D; ++k) {
                chord(k, rho2);
                c[k] = DOWN ? b[k] : a[k];
                row += c[k] * gp.stride[k];
            }
            outer = outer2();
            if (outer > rho2) next_line();
            else enter();
        } else {
            enter();
        }
    }
    // The buckets of dimension k within sqrt(rem) widths of t, relative to ct.
    PCMS_HD PCMS_INLINE void chord(int k, float rem)
    {
        const float h = __builtin_fmaf(sqrt_approx(rem), 1.0f + 2e-6f, 4e-5f);
        a[k] = max((int)fminf(fmaxf(floorf(fr[k] - h), -kFarBuckets), kFarBuckets), -ct[k]);
        b[k] = min((int)fminf(fmaxf(floorf(fr[k] + h), -kFarBuckets), kFarBuckets), gp.n[k] - 1 - ct[k]);
        // t beyond the grid: the ball may miss it, its nearest bucket is kept
        a[k] = min(a[k], gp.n[k] - 1 - ct[k]);
        b[k] = max(b[k], -ct[k]);
    }
    // Distance to the slab of bucket x of dimension k.
    PCMS_HD PCMS_INLINE float slab(int k, int x) const
    {
        const float y = (float)x - fr[k];
        return fmaxf(fmaxf(y, -1.0f - y) - 2e-5f, 0.0f);
    }
    PCMS_HD PCMS_INLINE float outer2() const
    {
        float s = 0.0f;
#pragma unroll
        for (int k = 2; k < D; ++k) {
            const float d = slab(k, c[k]);
            s = __builtin_fmaf(d, d, s);
        }
        return s;
    }
    PCMS_HD PCMS_INLINE void enter()
    {
        if constexpr (D >= 2) {
            chord(1, rho2 - outer);
            c[1] = DOWN ? b[1] : a[1];
        }
    }
    // The next line within reach (an odometer over c_2..c_{d-1}, unrolled so
    // that c stays in registers).
    PCMS_HD PCMS_INLINE void next_line()
    {
        if constexpr (D >= 3) {
            do {
                bool carry = true;
#pragma unroll
                for (int k = 2; k < D; ++k) {
                    if (carry) {
                        carry = DOWN ? c[k] <= a[k] : c[k] >= b[k];
                        const int step = carry ? (DOWN ? b[k] : a[k]) - c[k] : DOWN ? -1 : 1;
                        row += step * gp.stride[k];
                        c[k] += step;
                    }
                }
                more = !carry;
                outer = outer2();
            } while (more && outer > rho2);
            enter();
        } else {
            more = false;
        }
    }
    // The next rows' source ranges (beg >= end: none in that slot).  False,
    // with every slot empty, when the stencil is exhausted.
    PCMS_HD PCMS_INLINE bool next(int (&beg)[kRows], int (&end)[kRows])
    {
#pragma unroll
        for (int u = 0; u < kRows; ++u) beg[u] = end[u] = 0;
        if (!more) return false;
#pragma unroll
        for (int u = 0; u < (D == 1 ? 1 : kRows); ++u) {
            float rem = rho2;
            int at = row;
            bool ok = true;
            if constexpr (D >= 2) {
                const int x = DOWN ? c[1] - u : c[1] + u;
                const float d = slab(1, x);
                ok = DOWN ? x >= a[1] : x <= b[1];
                rem = fmaxf(rho2 - __builtin_fmaf(d, d, outer), 0.0f);
                at += x * gp.stride[1];
            }
            const float h = __builtin_fmaf(sqrt_approx(rem), (1.0f + 2e-6f) * (float)gp.sub, 4e-5f);
            const int x0 = ct[0] + (int)fminf(fmaxf(floorf(fr[0] - h), -kFarBuckets), kFarBuckets);
            const int x1 = ct[0] + (int)fminf(fmaxf(floorf(fr[0] + h), -kFarBuckets), kFarBuckets);
            if (ok) {
                beg[u] = cs[at + min(max(x0, 0), gp.n[0] - 1)];
                end[u] = cs[at + min(max(x1, 0), gp.n[0] - 1) + 1];
            }
        }
        if constexpr (D >= 2) {
            c[1] += DOWN ? -kRows : kRows;
            if (DOWN ? c[1] < a[1] : c[1] > b[1]) next_line();
        } else {
            more = false;
        }
        return true;
    }
};

// Candidate measures of the walks.  Exact64 loads a source's FP64 record
// and returns the D of the exact predicate.
template <int D, bool UNIT>
struct Exact64 {
    using E = double;
    const GridParams &gp;
    const double *__restrict__ spts;
    const double (&t)[D];
    // candidates p + j * G + q (j < B); those at or past end repeat p
    template <int G, int B>
    PCMS_HD PCMS_INLINE void load(int p, int end, int q, double (&s)[B][D]) const
    {
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int x = p + j * G + q;
            load_src<D>(spts, x < end ? x : p, s[j]);
        }
    }
    PCMS_HD PCMS_INLINE double d2(const double (&s)[D]) const { return metric_d2<D, UNIT>(t, s, gp); }
    // (Image32's bound and thresholds: the measure is exact)
    PCMS_HD PCMS_INLINE double bound(double) const { return 0.0; }
    PCMS_HD PCMS_INLINE double inside(double x) const { return x; }
    PCMS_HD PCMS_INLINE double outside(double x) const { return x; }
};

// Image32 loads a source's FP32 record s32_k = fl32(s_k - lo_k) and returns
// the FP32 image of D: with th_k = fl32(t_k - lo_k),
//     u_k = (th_k - s32_k) * fl32(g_k),   D32 = sum u_k^2
// (the sum as an fma chain).  It differs from the FP64 D by at most
//     m = alpha + beta * D32.
// Derivation: each u_k is within A_k + B |u_k| of its FP64 counterpart, where
// A_k = g_k |th_k| a (a >= 2 * 2^-24: rounding of the source's and of the
// target's image) and B >= 4 * 2^-24 + 2^-24 (the FP32 roundings of u_k and
// of g_k, and the source image through |s32_k| <= |th_k| + |v_k|).  Summing
// |u32_k^2 - u64_k^2| <= (A_k + B |u_k|)(A_k + (2 + B) |u_k|) over k, with
// sum_k A_k |u_k| <= |A| sqrt(D) and sqrt(D) <= (D / c + c) / 2 for any c > 0,
// and adding the d roundings of the FP32 sum, gives alpha and beta (times a
// safety factor of 1.5).  c is chosen near the thresholds of the walk, where
// the bound is tightest.  Differences that can overflow and metric factors
// outside the range of the bound (GridParams::max32) give non-finite thresholds,
// which the callers treat as "unknown".
template <int D, bool UNIT>
struct Image32 {
    using E = float;
    const float *__restrict__ s32;
    float th[D], g[D];
    double alpha, beta;

    PCMS_HD PCMS_INLINE Image32(const GridParams &gp, const float *s32_, const double (&t)[D],
                                double c)
        : s32(s32_)
    {
        constexpr double kA = 1.2e-7, kB = 3.1e-7, kR = 6.0e-8, kSafe = 1.5;
        double a2 = 0.0;
        bool known = true;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            th[k] = (float)(t[k] - gp.lo[k]);
            g[k] = UNIT ? 1.0f : (float)gp.g[k];
            known &= fabsf(th[k]) < gp.max32;
            const double ak = (UNIT ? 1.0 : gp.g[k]) * fabs((double)th[k]) * kA;
            a2 += ak * ak;
        }
        const double A = sqrt(a2);
        c = fmin(fmax(c, 1e-150), 1e150);
        alpha = known ? kSafe * (A * A + (1.0 + kB) * A * c) + 1e-36 : INFINITY;
        beta = kSafe * ((1.0 + kB) * A / c + 2.0 * kB + kB * kB + D * kR) * (1.0 + 1e-6);
    }
    // Candidates p + j * G + q (j < B); the values of those at or past end
    // are unspecified.  One lane's (G = 1) are B D adjacent floats, read as
    // 16-byte words: the records' storage has room for B - 1 records past the
    // last (the fixed-point records and kPad32 floats follow it).
    template <int G, int B>
    PCMS_HD PCMS_INLINE void load(int p, int end, int q, float (&s)[B][D]) const
    {
        if constexpr (G == 1) {
            static_assert(B * D % 4 == 0 && (B - 1) * D <= kPad32, "whole 16-byte words");
            const float4u *b = reinterpret_cast<const float4u *>(s32 + (size_t)p * D);
            float x[B * D];
#pragma unroll
            for (int i = 0; i < B * D / 4; ++i) {
                const float4u v = b[i];
#pragma unroll
                for (int h = 0; h < 4; ++h) x[4 * i + h] = v[h];
            }
#pragma unroll
            for (int j = 0; j < B; ++j)
#pragma unroll
                for (int k = 0; k < D; ++k) s[j][k] = x[j * D + k];
        } else {
#pragma unroll
            for (int j = 0; j < B; ++j) {
                const int x = p + j * G + q;
                load_src32<D>(s32, x < end ? x : p, s[j]);
            }
        }
    }
    PCMS_HD PCMS_INLINE float d2(const float (&s)[D]) const
    {
        float u = UNIT ? th[0] - s[0] : (th[0] - s[0]) * g[0];
        float acc = u * u;
#pragma unroll
        for (int k = 1; k < D; ++k) {
            u = UNIT ? th[k] - s[k] : (th[k] - s[k]) * g[k];
            acc = __builtin_fmaf(u, u, acc);
        }
        return acc;
    }
    // the bound on |D - D32| for D32 up to d
    PCMS_HD PCMS_INLINE double bound(double d) const { return alpha + beta * d; }
    // Thresholds for the exact predicate D < x: D32 < inside(x) implies
    // D < x, and D32 >= outside(x) implies D >= x.
    PCMS_HD PCMS_INLINE float inside(double x) const
    {
        return (float)((x - alpha) / (1.0 + beta) * (1.0 - 1.3e-7) - 1e-36);
    }
    PCMS_HD PCMS_INLINE float outside(double x) const
    {
        return beta < 0.5 ? (float)((x + alpha) / (1.0 - beta) * (1.0 + 1.3e-7) + 1e-36) : INFINITY;
    }
};

// Calls f(p, x, valid) for the sorted sources p of [beg, end), x being the
// measure's value (D, or its FP32 image), kBatch * G candidates per step (the
// loads of a step are issued together); every lane of the group calls f the
// same number of times, with valid = false on the padding slots past the end.
template <int D, int G, int kBatch, class Meas, class F>
PCMS_HD PCMS_INLINE void walk_step(const Meas &meas, int p, int end, int q, F &&f)
{
    typename Meas::E sb[kBatch][D];
    meas.template load<G, kBatch>(p, end, q, sb);
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
        const int x = p + j * G + q;
        f(x, meas.d2(sb[j]), x < end);
    }
}

// The ranges of sorted sources that can hold a source with D < rho2 (a
// superset of the ball); rho2 may be +inf.  next() yields up to kSlots of them
// (beg >= end: none in that slot), false at the end.  kDown: later ranges
// come first (if asked, on the grid); else in ascending order.
template <int D, bool UNIT, bool BVH, bool DOWN>
struct Ranges {
    static constexpr int kSlots = kRows;
    static constexpr bool kDown = DOWN;
    RowLines<D, DOWN> it;
    PCMS_HD PCMS_INLINE Ranges(const GridParams &gp, const int *cs, const BvhView &,
                               const double (&t)[D], double rho2)
        : it(gp, cs, t, rho2)
    {
    }
    PCMS_HD PCMS_INLINE bool next(int (&beg)[kSlots], int (&end)[kSlots]) { return it.next(beg, end); }
};

template <int D, bool UNIT, bool DOWN>
struct Ranges<D, UNIT, true, DOWN> {
    static constexpr int kSlots = 1;
    static constexpr bool kDown = false;
    BvhIter<D, UNIT> it;
    PCMS_HD PCMS_INLINE Ranges(const GridParams &gp, const int *, const BvhView &bv,
                               const double (&t)[D], double rho2)
        : it(gp, bv, t, rho2)
    {
    }
    PCMS_HD PCMS_INLINE bool next(int (&beg)[1], int (&end)[1]) { return it.next(beg[0], end[0]); }
};

// Search state of one target, shared by its G lanes.  The target's `words`
// LDS words L[0..words) hold the kept list (k_cap entries) and, during the
// radius search, the bins of the windowed selection or a buffer of words / 2
// doubles (double j in words 2j, 2j+1).
template <int D, bool UNIT, int G, bool BVH = false>
struct Search {
    const GridParams &gp;
    const int *__restrict__ cs;
    const double *__restrict__ spts;
    const float *__restrict__ spts32;   // FP32 records
    const int *__restrict__ perm;
    double t[D];
    int *L;     // this target's LDS words
    int k_cap;
    int words;  // >= max(k_cap, 2)
    Grp<G> g;
    BvhView bv; // the tree (BVH only)
    int lim = 0;   // words below it are the caller's during scan32

    PCMS_HD PCMS_INLINE int &at(int e)
    {
#ifdef PCMS_HOST_EMULATION
        if (e < 0 || e >= words) pcms_emu_lds_fault(e, words);
#endif
        return L[e];
    }
    PCMS_HD PCMS_INLINE void dstore(int j, double v)
    {
        unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
        at(2 * j) = (int)(unsigned)(bits & 0xffffffffull);
        at(2 * j + 1) = (int)(unsigned)(bits >> 32);
    }
    PCMS_HD PCMS_INLINE double dload(int j)
    {
        unsigned long long lo = (unsigned)at(2 * j);
        unsigned long long hi = (unsigned)at(2 * j + 1);
        return __builtin_bit_cast(double, (hi << 32) | lo);
    }
    // Calls f(p, x, valid) for the candidates of the ball D < rho2, range by
    // range, x the measure's value (the general paths), in ascending order.
    template <int kBatch, class Meas, class F>
    PCMS_HD PCMS_INLINE void each_of(const Meas &meas, double rho2, F &&f)
    {
        using R = Ranges<D, UNIT, BVH, false>;
        count_walk();
        R rng(gp, cs, bv, t, rho2);
        auto range = [&](int p, int e) {
            count_range(p, e);
            for (; p < e; p += kBatch * G) walk_step<D, G, kBatch>(meas, p, e, g.q, f);
        };
        if constexpr (BVH) {
            rng.it.each(range);
        } else {
            int beg[R::kSlots], end[R::kSlots];
            while (rng.next(beg, end)) {
#pragma unroll 1
                for (int u = 0; u < R::kSlots; ++u) {
                    int p = beg[0], e = end[0];
#pragma unroll
                    for (int x = 1; x < R::kSlots; ++x)
                        if (u == x) {
                            p = beg[x];
                            e = end[x];
                        }
                    range(p, e);
                }
            }
        }
    }
    template <class F>
    PCMS_HD PCMS_INLINE void each(double rho2, F &&f)
    {
        each_of<kBatch64>(Exact64<D, UNIT>{gp, spts, t}, rho2, f);
    }

    // Calls f(p, x, valid) for the candidates of the ball D < rho2, x the
    // measure's value (the FP32 image, in general).  The ranges are first listed in a table at the end of the target's words (the
    // first used() words are the caller's), one word each: length (12 bits)
    // and start relative to the table's first range (20 bits).  Then one loop
    // steps through the candidates of all of them: a lane that has finished a
    // range takes its next one while other lanes are inside theirs.  With a
    // loop per row, a wave's every row took its longest lane's steps (349
    // candidate slots per walk against 200, in a host model of the 4M-source
    // kNN search), and fetching the rows inside the steps' loop made every
    // step pay for some lane's row.  A step's records are loaded before the
    // previous step's are used.  The earliest range stands first and is taken
    // first, so the words next to the caller's are free again first: f may use
    // words below `lim` as it goes, up to the next range's word, which has been
    // read.  That depends on the range alone and not on the step, so a list
    // meets the table at the same candidate with any number of lanes.  A table's
    // candidates come in ascending order; a table that does not hold all ranges
    // is filled again.
    // False if it can hold none (no room, or a range too long).
    template <class Meas, class U, class F>
    PCMS_HD PCMS_INLINE bool scan32(const Meas &im, double rho2, U &&used, F &&f)
    {
        using R = Ranges<D, UNIT, BVH, true>;
        constexpr int S = R::kSlots;
        count_walk();
        R rng(gp, cs, bv, t, rho2);
        int beg[S], end[S];
        bool more = rng.next(beg, end), fits = true;
        while (more) {
            // (in 4-D and 5-D half of the words, as the list grows faster than
            // the many rows of a full table are taken)
            const int room = D >= 4 ? (words - used()) / 2 : words - used();
            int n = 0, base = 0;
            // slots that do not fit stay for the next table
            bool left = false;
            do {
#pragma unroll
                for (int u = 0; u < S; ++u) {
                    if (beg[u] < end[u]) {
                        if (n == 0) base = beg[u];
                        const unsigned rel = (unsigned)(R::kDown ? base - beg[u] : beg[u] - base);
                        const unsigned len = (unsigned)(end[u] - beg[u]);
                        if (n < room && (rel >> 20) == 0 && !left) {
                            count_range(beg[u], end[u]);
                            fits &= len < 4096u;
                            if (g.q == 0) at(words - 1 - n) = (int)((rel << 12) | (len & 4095u));
                            ++n;
                            end[u] = beg[u];
                        } else {
                            left = true;
                        }
                    }
                }
                if (!left) more = rng.next(beg, end);
            } while (more && !left);
            if (left && n == 0) fits = false;
            if (!g.all(fits)) return false;
            g.sync();
            int tab = words - n;
            if (!R::kDown) {   // the earliest range first
                for (int i = g.q; 2 * i < n - 1; i += G) {
                    const int x = at(tab + i), y = at(words - 1 - i);
                    at(tab + i) = y;
                    at(words - 1 - i) = x;
                }
                g.sync();
            }
            int p = 0, e = 0;
            unsigned w = n > 0 ? (unsigned)at(tab) : 0u;
            auto take = [&]() {   // the next range, from w
                p = R::kDown ? base - (int)(w >> 12) : base + (int)(w >> 12);
                e = p + (int)(w & 4095u);
                ++tab;
                w = tab < words ? (unsigned)at(tab) : 0u;
            };
            if (n > 0) {
                take();
                int next_lim = min(tab + 1, words);
                typename Meas::E s[kBatch32][D];
                im.template load<G, kBatch32>(p, e, g.q, s);
                for (;;) {
                    const int p0 = p, e0 = e;
                    lim = next_lim;
                    p += kBatch32 * G;
                    const bool on = p < e || tab < words;
                    if (p >= e && on) {
                        take();
                        next_lim = min(tab + 1, words);
                    }
                    typename Meas::E nx[kBatch32][D];
                    if (on) im.template load<G, kBatch32>(p, e, g.q, nx);
#pragma unroll
                    for (int j = 0; j < kBatch32; ++j) {
                        const int x = p0 + j * G + g.q;
                        f(x, im.d2(s[j]), x < e0);
                    }
                    if (!on) break;
#pragma unroll
                    for (int j = 0; j < kBatch32; ++j)
#pragma unroll
                        for (int k = 0; k < D; ++k) s[j][k] = nx[j][k];
                }
            }
            g.sync();
        }
        return true;
    }

    PCMS_HD PCMS_INLINE void count_walk() const
    {
#ifdef PCMS_HOST_EMULATION
        if (g.q == 0) ++pcms_emu_walks;
#endif
    }
    PCMS_HD PCMS_INLINE void count_range(int beg, int end) const
    {
#ifdef PCMS_HOST_EMULATION
        if (g.q == 0) {
            ++pcms_emu_rows;
            pcms_emu_cands += end - beg;
        }
#else
        (void)beg;
        (void)end;
#endif
    }

    // Squared metric distance from t to the farthest corner of the bucket
    // box; every source lies closer, so a larger radius covers all sources.
    PCMS_HD PCMS_INLINE double far2() const
    {
        double acc = 0.0;
#pragma unroll
        for (int k = 0; k < D; ++k) {
            double lo = gp.lo[k], hi = gp.lo[k] + gp.n[k] * gp.w[k];
            double dd = fmax(fabs(t[k] - lo), fabs(hi - t[k])) * gp.g[k];
            acc += dd * dd;
        }
        return acc * (1.0 + 1e-6) + 1e-300;
    }

    // Collects every source with D < r2 into the list (up to k_cap, in walk
    // order); returns the count (the same on every lane of the group), and
    // leaves the list unfinished where it is above k_cap, as the k_cap nearest
    // are then selected afresh.  The walk reads FP32 records; a candidate
    // between the two thresholds is decided from its FP64 record.
    PCMS_HD PCMS_INLINE int collect(double r2)
    {
        const Image32<D, UNIT> im(gp, spts32, t, sqrt(r2));
        const float in = im.inside(r2), out = im.outside(r2);
        int n = 0;
        // In 1-D and 2-D, with few and long rows and FP64 records of one word,
        // the plain walk is as fast (2-D lattice, 1M targets: 345 us against
        // 355 with the FP32 records and 375 with the table).
        bool done = false;
        if ((D >= 3 || BVH) && out < INFINITY) {
            bool kept = true;
            auto add = [&](int p, float d, bool ok) {
                bool acc = ok & (d < out);
                if (acc && !(d < in)) {
#ifdef PCMS_HOST_EMULATION
                    ++pcms_emu_exact;
#endif
                    acc = d2_of(p) < r2;
                }
                const unsigned m = g.ballot(acc);
                if (acc) {
                    const int pos = n + g.below(m);
                    if (pos < lim) at(pos) = p;
                    else kept &= pos >= k_cap;
                }
                n += __builtin_popcount(m);
            };
            done = scan32(im, r2, [&]() { return min(n, k_cap); }, add);
            if (done && n <= k_cap) done = g.all(kept);
        }
        if (!done) {   // (no FP32 threshold, no room for the table, or none for the list)
            n = 0;
            each_of<kBatch64>(Exact64<D, UNIT>{gp, spts, t}, r2, [&](int p, double d2, bool ok) {
                const bool acc = ok & (d2 < r2);
                const unsigned m = g.ballot(acc);
                if (acc) {
                    const int pos = n + g.below(m);
                    if (pos < k_cap) at(pos) = p;
                }
                n += __builtin_popcount(m);
            });
        }
        g.sync();
        return n;
    }

    // Radius of a ball expected to hold k sources, from the bucket counts
    // around t (no point loads): the 3^d block of bucket widths around t's
    // bucket, which in dimension 0 spans sub + sub/2 slices to each side.
    PCMS_HD PCMS_INLINE double knn_radius_guess(int k) const
    {
        if constexpr (BVH) return box_corrected(bvh_radius_guess<D, UNIT>(gp, bv, t, k));
        int a[D], b[D], c[D];
        double vol = 1.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
            const int h = j == 0 ? gp.sub + gp.sub / 2 : 1;
            int cj = bucket_of(gp, j, t[j]);
            a[j] = max(cj - h, 0);
            b[j] = min(cj + h, gp.n[j] - 1);
            c[j] = a[j];
            vol *= (double)(b[j] - a[j] + 1) * gp.w[j] * gp.g[j];
        }
        long long count = 0;
        for (;;) {
            int row = 0;
#pragma unroll
            for (int j = 1; j < D; ++j) row += c[j] * gp.stride[j];
            count += cs[row + b[0] + 1] - cs[row + a[0]];
            bool carry = true;
#pragma unroll
            for (int j = 1; j < D; ++j) {
                if (carry) {
                    if (c[j] < b[j]) {
                        c[j]++;
                        carry = false;
                    } else {
                        c[j] = a[j];
                    }
                }
            }
            if (carry) break;
        }
        // unit-ball volume pi^(D/2) / Gamma(D/2 + 1)
        const double vball = D == 1 ? 2.0 : D == 2 ? M_PI : D == 3 ? 4.18879020478639098
                           : D == 4 ? 4.93480220054467931 : 5.26378901489003940;
        if (count <= 0) {
            double half = 0.0;
#pragma unroll
            for (int j = 0; j < D; ++j) half = fmax(half, 1.5 * gp.w[j] * gp.g[j]);
            return 2.0 * half;
        }
        return box_corrected(pow((double)k * vol / ((double)count * vball), 1.0 / D));
    }

    // Every source lies in the bounding box, so the part of a ball beyond a
    // face holds none: the radius g0 expected to hold k sources at the local
    // density is grown until the part inside the box is expected to hold k
    // (faces taken one at a time, two fixed-point steps; a face behind the
    // target cuts nothing here).  Each dimension keeps at least half of the
    // ball, as at a face: a box thinner than the ball (flat or coincident
    // sources) holds a lower-dimensional cloud, which this model does not
    // describe, so the radius grows at most 2x.  In 1-3 dimensions (where
    // knn_select narrows the grid's window to match).
    PCMS_HD PCMS_INLINE double box_corrected(double g0) const
    {
        if constexpr (D > 3) {
            return g0;
        } else {
            double gr = g0;
            bool cut = false;
#pragma unroll
            for (int j = 0; j < D; ++j)
                cut |= fmin(t[j] - gp.lo[j], gp.hi[j] - t[j]) * (UNIT ? 1.0 : gp.g[j]) < g0;
            if (!cut) return g0;   // no face within the ball
            for (int it = 0; it < 2; ++it) {
                double f = 1.0;
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    const double s = (UNIT ? 1.0 : gp.g[j]) / gr;
                    f *= fmax(1.0 - ball_beyond<D>((t[j] - gp.lo[j]) * s) -
                                  ball_beyond<D>((gp.hi[j] - t[j]) * s),
                              0.5);
                }
                gr = g0 * pow(f, -1.0 / D);
            }
            return gr < INFINITY ? gr : g0;
        }
    }

    // Appends the values D in [lo, hi) to the buffer (ordered compaction,
    // at most cb kept); returns (group-uniform) the counts below lo and in
    // [lo, hi).
    PCMS_HD PCMS_INLINE void buffer_bracket(double lo, double hi, int cb, int &c_lo, int &n_in)
    {
        int below = 0, n = 0;
        each(hi, [&](int, double d2, bool ok) {
            below += ok & (d2 < lo);
            const bool in = ok & (d2 >= lo) & (d2 < hi);
            const unsigned m = g.ballot(in);
            if (in) {
                const int pos = n + g.below(m);
                if (pos < cb) dstore(pos, d2);
            }
            n += __builtin_popcount(m);
        });
        g.sync();
        c_lo = g.sum(below);
        n_in = n;
    }

    // r-th smallest (1-based) of the n doubles in the buffer; the lanes rank
    // interleaved entries and the group takes the minimum found.
    PCMS_HD PCMS_INLINE double buffer_rank(int n, int r)
    {
        double ans = INFINITY;
        for (int a0 = 0; a0 < n; a0 += G) {
            const int a = a0 + g.q;
            if (a < n) {
                const double v = dload(a);
                int less = 0, le = 0;
                for (int b = 0; b < n; ++b) {
                    const double x = dload(b);
                    less += x < v;
                    le += x <= v;
                }
                if (less < r && r <= le) ans = v;
            }
        }
        return g.min(ans);
    }

    // D of sorted source p
    PCMS_HD PCMS_INLINE double d2_of(int p) const
    {
        double sb[D];
        load_src<D>(spts, p, sb);
        return metric_d2<D, UNIT>(t, sb, gp);
    }

    // kNN selection in two walks, for k <= k_cap + 1: select_window over the
    // window [(a g)^2, (b g)^2), g the estimate of the radius.  With the
    // grid's estimate corrected for the bounding box (1-3 dimensions) the
    // window is [0.8 g, 1.18 g); else, and for the LBVH's noisier estimate,
    // [0.78 g, 1.3 g).  On success r2 is the k-th smallest D, the list holds
    // every source with D < r2 and n_found their count (< k).  When the k-th
    // lies outside the window, one more window beside it is tried,
    // [b g, 1.5 b g) or [0.6 a g, a g): two walks instead of the general
    // path's bracketing.  False leaves the general path to the caller.
    PCMS_HD PCMS_INLINE bool knn_select(int k, double &r2, int &n_found)
    {
        constexpr bool kTight = !BVH && D <= 3;
        constexpr double a = kTight ? 0.8 : 0.78, b = kTight ? 1.18 : 1.3;
        const double gr = knn_radius_guess(k);
        double lo = (a * gr) * (a * gr), hi = (b * gr) * (b * gr);
        // one call site, so that the selection is inlined once
        for (int attempt = 0; attempt < 2; ++attempt) {
            int side = 0;
            if (select_window<false>(k, lo, hi, r2, n_found, &side)) return true;
            if (side > 0) {
                lo = hi;
                hi = (1.5 * b * gr) * (1.5 * b * gr);
            } else if (side < 0) {
                hi = lo;
                lo = (0.6 * a * gr) * (0.6 * a * gr);
            } else {
                return false;
            }
        }
        return false;
    }

    // The k-th smallest D in two walks, given a window [lo, hi) expected to
    // hold it.  The first walk, over the ball D < hi, histograms the FP32
    // images into nb bins of equal width (16-bit counts in the target's first
    // words), number 1 the window's first and number 0 everything below lo.  (A
    // k-th in the window's first bin must not be taken for one below: a target
    // then goes to the general path, and its wave waits for five walks or more.
    // With the two in one bin a third of a kNN search's waves held such a target:
    // 3-D linear FP64 on the tree, 70k and 300k targets, 1136 and 1466 us against
    // 744 and 1105 now.)  The k-th smallest image
    // lies in some bin b, and since every D is within the image's bound m of
    // its image, the k-th smallest D lies within m of that bin: in [e0, e1],
    // the bin widened by m and the rounding of the binning.  The second walk
    // lists the sources below e0 for sure, and sets aside those that are not
    // but may be below e1.  Every other source has D >= e1, so the k-th
    // smallest D is ranked among those set aside (their D recomputed in FP64:
    // one or two with untied distances, up to kReg in registers, more in a
    // further walk), and those below it complete the list.  On success v is
    // the k-th smallest D and the list holds every source with D < v, n their
    // count (< k); with TIES the list is then completed to k entries with
    // sources at D = v, smallest source index first, and n = k (the words then
    // begin at the list: L moves).  Returns false when the k-th image lies
    // outside [lo, hi) or the list does not fit the words; then *side (if
    // given) is -1 if the k-th lies below lo, +1 if at or above hi, 0
    // otherwise.
    template <bool TIES>
    PCMS_HD PCMS_INLINE bool select_window(int k, double lo, double hi, double &v, int &n_out,
                               int *side = nullptr)
    {
        constexpr int kReg = 7;
        // In 1-D the records are as large in FP64 as they are loaded, and a
        // cloud of many sources has radii near the images' rounding, so that
        // most of a window would be set aside (kNN 10, 1M targets among 4M and
        // 20M uniform sources: 788 and 2567 us with the images).
        using Meas = typename std::conditional<D == 1, Exact64<D, UNIT>, Image32<D, UNIT>>::type;
        using E = typename Meas::E;
        const Meas im = [&]() {
            if constexpr (D == 1) return Meas{gp, spts, t};
            else return Meas(gp, spts32, t, sqrt(hi));
        }();
        const int nb = min(words, kMaxBins), nbw = (nb + 3) / 2;
        const double bw = (hi - lo) / nb;
        const E hi32 = (E)hi, ibw = (E)(1.0 / bw), off = (E)(1.0 - lo / bw);
        for (int j = g.q; j < nbw; j += G) at(j) = 0;
        g.sync();
        const bool full = scan32(im, hi, [&]() { return nbw; }, [&](int, E d, bool ok) {
            if (ok & (d < hi32)) {
                const float y = fminf(fmaxf((float)fma_t(d, ibw, off), 0.0f), (float)(nb + 1));
                const int j = (int)y;
                lds_add(&at(j >> 1), j & 1 ? 1 << 16 : 1);
            }
        });
        g.sync();
        // (a count beyond 16 bits misleads, and is caught below)
        int b = -1, cum = 0, c_in = 0;   // c_in: images up to the end of bin b
        for (int j = 0; j < nbw; ++j) {
            const unsigned x = (unsigned)at(j);
            const int c0 = cum + (int)(x & 0xffffu), c1 = c0 + (int)(x >> 16);
            if (b < 0 && c1 >= k) {
                b = c0 >= k ? 2 * j : 2 * j + 1;
                c_in = c0 >= k ? c0 : c1;
            }
            cum = c1;
        }
        g.sync();   // every lane has read the bins before the list overwrites them
        if (side) *side = 0;
        if (!full) return false;
        if (b < 0 || (b == 0 && lo > 0.0)) {
            if (side) *side = b < 0 ? 1 : -1;
            return false;
        }
        // All of these would be listed or set aside, so a window whose k-th
        // bin is too full is given up after one walk (a radius that grew far
        // beyond the cap).
        if (c_in > words) return false;
        const double m = im.bound(hi) + 1e-6 * hi;
        const double e0 = lo + (double)(b - 1) * bw - m, e1 = lo + (double)b * bw + m;
        const E in = im.inside(e0), out = im.outside(e1);
        if (!(out < INFINITY)) return false;
        // the first kReg words hold those set aside, the list follows
        int n = 0, nm = 0;
        bool room = words >= kReg + k;
        if (room) {
            const bool whole = scan32(im, e1, [&]() { return kReg + min(n, k); }, [&](int p, E d, bool ok) {
                const bool acc = ok & (d < out), sure = acc & (d < in);
                const unsigned ma = g.ballot(acc), ms = g.ballot(sure);
                if (acc) {
                    const int pos = sure ? kReg + n + g.below(ms) : nm + g.below(ma & ~ms);
                    if (pos < (sure ? lim : kReg)) at(pos) = p;
                    else room &= !sure;
                }
                n += __builtin_popcount(ms);
                nm += __builtin_popcount(ma & ~ms);
            });
            g.sync();
            if (whole && n + nm > words) return false;
            room = g.all(room && whole);
            // (fewer than k, or k below e0: only where the images mislead)
            if (room && (n >= k || n + nm < k)) return false;
        }
        if (room && nm <= kReg) {
            double dm[kReg];
            int pm[kReg], id[kReg];
#pragma unroll
            for (int j = 0; j < kReg; ++j) {
                dm[j] = INFINITY;
                pm[j] = id[j] = 0;
                if (j < nm) {
                    pm[j] = at(j);
                    dm[j] = d2_of(pm[j]);
                }
            }
            g.sync();
            v = INFINITY;
#pragma unroll
            for (int j = 0; j < kReg; ++j) {
                int less = 0, le = 0;
#pragma unroll
                for (int i = 0; i < kReg; ++i) {
                    less += dm[i] < dm[j];
                    le += dm[i] <= dm[j];
                }
                if (less < k - n && k - n <= le) v = dm[j];
            }
            if (!(v >= e0 && v <= e1)) return false;   // cannot happen
            int need = k - n;   // sources at v to keep (TIES)
            if (TIES) {
#pragma unroll
                for (int j = 0; j < kReg; ++j) {
                    need -= dm[j] < v;
                    if (dm[j] == v) id[j] = perm[pm[j]];
                }
            }
#pragma unroll
            for (int j = 0; j < kReg; ++j) {
                bool take = dm[j] < v;
                if (TIES && dm[j] == v) {
                    int rank = 0;
#pragma unroll
                    for (int i = 0; i < kReg; ++i) rank += dm[i] == v && id[i] < id[j];
                    take = rank < need;
                }
                if (take) {
                    if (g.q == 0) at(kReg + n) = pm[j];
                    ++n;
                }
            }
            L += kReg;
            words -= kReg;
            g.sync();
            n_out = n;
            return true;
        }
        // many set aside, or no words for the table: they are listed at the
        // end of the words, the last one first, and ranked there
        int c_b = 0, n_b = 0;
        each_of<kBatch32>(im, e1, [&](int p, E d, bool ok) {
            const bool acc = ok & (d < out), sure = acc & (d < in);
            const unsigned ma = g.ballot(acc), ms = g.ballot(sure);
            if (acc) {
                const int pos = sure ? c_b + g.below(ms) : words - 1 - n_b - g.below(ma & ~ms);
                if ((unsigned)pos < (unsigned)words) at(pos) = p;
            }
            c_b += __builtin_popcount(ms);
            n_b += __builtin_popcount(ma & ~ms);
        });
        g.sync();
        if (c_b + n_b > words || c_b >= k || c_b + n_b < k) return false;
        const int base = words - n_b, r = k - c_b;
        double ans = INFINITY;
        for (int a0 = 0; a0 < n_b; a0 += G) {
            const int a = a0 + g.q;
            if (a < n_b) {
                const double x0 = d2_of(at(base + a));
                int less = 0, le = 0;
                for (int j = 0; j < n_b; ++j) {
                    const double x = d2_of(at(base + j));
                    less += x < x0;
                    le += x <= x0;
                }
                if (less < r && r <= le) ans = x0;
            }
        }
        v = g.min(ans);
        if (!(v >= e0 && v <= e1)) return false;
        if (TIES) {
            // the k - (c_b + #(those below v)) sources at D = v of smallest
            // source index join the list: each round marks the next one (its
            // word holds ~p until it is appended)
            int below_v = 0;
            for (int j0 = 0; j0 < n_b; j0 += G) {
                const int j = j0 + g.q;
                below_v += j < n_b && d2_of(at(base + j)) < v;
            }
            int prev = -1;
            for (int need = k - c_b - g.sum(below_v); need > 0; --need) {
                int best = 0x7fffffff, bj = -1;
                for (int j0 = 0; j0 < n_b; j0 += G) {
                    const int j = j0 + g.q;
                    if (j < n_b) {
                        const int x = at(base + j);
                        if (x >= 0) {
                            const int idx = perm[x];
                            if (idx > prev && idx < best && d2_of(x) == v) {
                                best = idx;
                                bj = j;
                            }
                        }
                    }
                }
                const int gb = g.min(best);
                g.sync();
                if (best == gb && bj >= 0) at(base + bj) = ~at(base + bj);
                g.sync();
                prev = gb;
            }
        }
        // append those below v and the chosen ties; entry j is read before
        // position c_b + j (<= base + j) can be written
        int cnt = c_b;
        for (int j0 = 0; j0 < n_b; j0 += G) {
            const int j = j0 + g.q;
            const int x = j < n_b ? at(base + j) : 0;
            const int p = x < 0 ? ~x : x;
            const bool take = j < n_b && (x < 0 || d2_of(p) < v);
            const unsigned mt = g.ballot(take);
            g.sync();
            if (take) at(cnt + g.below(mt)) = p;
            cnt += __builtin_popcount(mt);
        }
        g.sync();
        n_out = cnt;
        return true;
    }

    // Squared distance of the k-th nearest source.  One walk counts the
    // sources below lo = ((1 - h) g)^2 and buffers those in
    // [lo, hi = ((1 + h) g)^2), g the bucket-count estimate of the radius;
    // when the k-th falls in the buffered interval it is ranked there,
    // otherwise the general bracketing search continues from what the walk
    // established.
    PCMS_HD PCMS_INLINE double knn_r2(int k)
    {
        const double gr = knn_radius_guess(k);
        const int cb = words / 2;
        // expected count in the window k ((1 + h)^D - (1 - h)^D) ~ 2 D h k,
        // sized to about 3/4 of the buffer
        const double h = fmin(0.15, fmax(0.02, 0.75 * (double)cb / (2.0 * D * (double)k)));
        const double lo = (1.0 - h) * (1.0 - h) * gr * gr, hi = (1.0 + h) * (1.0 + h) * gr * gr;
        int c_lo, n_in;
        buffer_bracket(lo, hi, cb, c_lo, n_in);
        if (c_lo < k && k <= c_lo + n_in && n_in <= cb) return buffer_rank(n_in, k - c_lo);
        // (one call site, so that the search is inlined once)
        double from = lo, to = hi;
        int c = c_lo;
        if (c_lo >= k) {
            from = 0.0;
            to = lo;
            c = 0;
        } else if (c_lo + n_in < k) {
            from = hi;
            to = 4.0 * hi;
            c = c_lo + n_in;
        }
        return kth(k, from, c, to, cb);
    }

    // Exact k-th smallest D (1-based) over all sources, given a bracket:
    // #(D < lo) = c_lo < k, and hi a first guess for an upper bound (grown
    // when #(D < hi) < k).  Each round counts the sources of [lo, hi) into 8
    // sub-intervals with one walk; once the interval holding the k-th has at
    // most `sb` (<= words / 2) sources they are copied into the buffer and
    // ranked.
    PCMS_HD PCMS_INLINE double kth(int k, double lo, int c_lo, double hi, int sb)
    {
        constexpr int NB = 8;
        const double farr = far2();
        for (int it = 0; it < 400; ++it) {
            double sp[NB];
            const bool from_zero = (lo == 0.0);
#pragma unroll
            for (int j = 0; j < NB - 1; ++j) {
                // from zero: equal expected counts, ((j + 1) / NB)^(2 / D) of
                // the interval; otherwise linear in D
                const double x = (double)(j + 1) / NB;
                const double f0 = D == 1 ? x * x : D == 2 ? x : D == 3 ? cbrt(x * x)
                                : D == 4 ? sqrt(x) : pow(x, 0.4);
                const double f = from_zero ? f0 : x;
                sp[j] = fmin(fmax(lo + (hi - lo) * f, lo), hi);
            }
            sp[NB - 1] = hi;
            int cnt[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) cnt[j] = 0;
            const double l0 = lo, h0 = hi;
            double vmin = h0;   // smallest D in [lo, hi) and its multiplicity
            int neq = 0;
            each(h0, [&](int, double d2, bool ok) {
                if (ok & (d2 >= l0) & (d2 < h0)) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) cnt[j] += d2 < sp[j];
                    if (d2 < vmin) {
                        vmin = d2;
                        neq = 0;
                    }
                    neq += d2 == vmin;
                }
            });
#pragma unroll
            for (int j = 0; j < NB; ++j) cnt[j] = g.sum(cnt[j]);
            {
                const double gmin = g.min(vmin);
                neq = g.sum(vmin == gmin ? neq : 0);
                vmin = gmin;
            }
            if (c_lo + cnt[NB - 1] < k) {     // the k-th lies at or above hi
                // every source has D < farr, so the count reaches k there
                // (k <= n_src); nothing above it is left to search
                if (!(hi < farr)) return hi;
                c_lo += cnt[NB - 1];
                lo = hi;
                hi = fmin(fmax(hi * 16.0, farr * 1e-12), farr);
                continue;
            }
            // #(D < vmin) = c_lo: the k-th is vmin when its copies reach rank k
            if (c_lo + neq >= k) return vmin;
            int bsel = NB - 1;
#pragma unroll
            for (int j = NB - 1; j >= 0; --j)
                if (c_lo + cnt[j] >= k) bsel = j;
            int below = 0;
            double nlo = lo, nhi = hi;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (j + 1 == bsel) {
                    below = cnt[j];
                    nlo = sp[j];
                }
                if (j == bsel) nhi = sp[j];
            }
            int nin = cnt[bsel] - below;
            lo = nlo;
            hi = nhi;
            c_lo += below;
            if (nin == cnt[NB - 1] && vmin >= lo) {
                // no split separated the values (many equal ones): step past
                // the smallest, whose copies all rank below k
                lo = nextafter(vmin, INFINITY);
                c_lo += neq;
                nin -= neq;
            }
            if (nin <= sb) {
                int cl, n;
                buffer_bracket(lo, hi, sb, cl, n);
                const double ans = buffer_rank(min(n, sb), k - c_lo);
                return ans < INFINITY ? ans : hi;
            }
            // a single representable value left in [lo, hi): it is the answer
            if (!(nextafter(lo, INFINITY) < hi)) return lo;
        }
        return hi;
    }

    // Keeps the k_cap smallest (D, source index) among D < r2 in the list
    // (called when more than k_cap sources are inside); returns the number of
    // list entries written.
    PCMS_HD PCMS_INLINE int cap_collect(double r2, int n_found)
    {
        // usually two walks: the k_cap-th lies in the window [0, r2).  In 4-D
        // and 5-D, where most of the ball is near its surface and its bins
        // would hold many sources, in the part of it expected to hold the
        // sources of rank k_cap - 5 sqrt(k_cap) to k_cap + 5 sqrt(k_cap).
        double vw, lo = 0.0, hi = r2;
        int nw;
        if constexpr (D >= 4) {
            const float s = 5.0f * sqrt_approx((float)k_cap), f = 1.0f / (float)n_found;
            lo = r2 * (double)powf(fmaxf((float)k_cap - s, 0.0f) * f, 2.0f / D);
            hi = r2 * (double)powf(fminf(((float)k_cap + s) * f, 1.0f), 2.0f / D);
        }
        // (one call site, so that the selection is inlined once)
        for (int attempt = 0; attempt < (D >= 4 ? 2 : 1); ++attempt) {
            int side = 0;
            if (select_window<true>(k_cap, lo, hi, vw, nw, &side)) return nw;
            if (side == 0) break;   // in the window, but too many: wider bins hold more
            lo = 0.0;
            hi = r2;
        }
        const double v = kth(k_cap, 0.0, 0, r2, words / 2);
        const double vnext = nextafter(v, INFINITY);
        int n = 0, c_eq = 0;
        each(vnext, [&](int p, double d2, bool ok) {
            const bool acc = ok & (d2 < v);
            const unsigned m = g.ballot(acc);
            if (acc) {
                const int pos = n + g.below(m);
                if (pos < k_cap) at(pos) = p;
            }
            n += __builtin_popcount(m);
            c_eq += ok & (d2 == v);
        });
        g.sync();
        c_eq = g.sum(c_eq);
        const int need = k_cap - n;
        if (need <= 0) return k_cap;
        int jthr = 0x7fffffff;
        if (need < c_eq) {        // ties at v: the smallest source indices win
            int prev = -1;
            for (int r = 0; r < need; ++r) {
                int best = 0x7fffffff;
                each(vnext, [&](int p, double d2, bool ok) {
                    if (ok & (d2 == v)) {
                        const int j = perm[p];
                        if (j > prev && j < best) best = j;
                    }
                });
                prev = g.min(best);
            }
            jthr = prev;
        }
        each(vnext, [&](int p, double d2, bool ok) {
            const bool acc = ok & (d2 == v) && perm[p] <= jthr;
            const unsigned m = g.ballot(acc);
            if (acc) {
                const int pos = n + g.below(m);
                if (pos < k_cap) at(pos) = p;
            }
            n += __builtin_popcount(m);
        });
        g.sync();
        return min(n, k_cap);
    }
};

}  // namespace pcms
