// Declarations shared by the kernels and their host emulation build.
//
// Everything here is plain arithmetic on plain pointers, marked host+device,
// so the same code runs inside the HIP kernels and in the CPU emulation that
// the test-suite builds with address sanitising to check indexing.
#pragma once

#include <stdint.h>

#ifdef PCMS_HOST_EMULATION
#include <algorithm>
#include <cmath>
#define PCMS_HD
#define PCMS_INLINE inline
using std::exp;
using std::fabs;
using std::floor;
using std::fmax;
using std::fmin;
using std::isinf;
using std::isnan;
using std::max;
using std::min;
using std::nextafter;
using std::pow;
using std::rint;
using std::log2;
using std::ldexp;
using std::ceil;
using std::sqrt;
// Called by the emulation build when a lane addresses LDS words outside its own.
[[noreturn]] void pcms_emu_lds_fault(int e, int words);
// The HIP vector type the walks load records with.
struct alignas(16) float4 {
    float x, y, z, w;
};
// Work counters of the emulation build (rows walked, candidates tested, walks,
// candidates of FP32 walks that needed their FP64 record, LBVH records read).
extern thread_local long long pcms_emu_rows, pcms_emu_cands, pcms_emu_walks, pcms_emu_exact,
    pcms_emu_nodes;
// Collective operations of a lane group, provided by the emulation driver:
// the G lanes of a group run as G threads meeting at a barrier per operation.
struct EmuGroup;
unsigned pcms_emu_ballot(EmuGroup *g, int q, bool p);
double pcms_emu_sum(EmuGroup *g, int q, double x);
float pcms_emu_sum(EmuGroup *g, int q, float x);
int pcms_emu_sum(EmuGroup *g, int q, int x);
double pcms_emu_min(EmuGroup *g, int q, double x);
int pcms_emu_min(EmuGroup *g, int q, int x);
void pcms_emu_sync(EmuGroup *g, int q);
#else
#include <hip/hip_runtime.h>
#define PCMS_HD __host__ __device__
#define PCMS_INLINE __forceinline__
#endif

#include "pcms_mls.h"

namespace pcms {

constexpr int kMaxDim = PCMS_MAX_DIM;
// Slices of dimension 0 per bucket width in the grids the library builds.
constexpr int kRowSlices = 4;
constexpr int kMaxKcap = PCMS_MAX_KCAP;

// Device-resident description of a uniform grid.  Bucket coordinates of a
// point x are c_k = clamp(floor((x_k - lo_k) * inv_w_k), 0, n_k - 1); the
// linear bucket id is row-major with dimension 0 fastest, so the buckets of
// one "row" (fixed c_1..c_{d-1}) are contiguous in sorted order.  Dimension
// 0 is cut `sub` times finer than the others (w_0 = w / sub in metric
// units): a search pays per row it visits, not per bucket, so the finer
// slices narrow each row's range to the ball's chord at no cost in rows.
struct GridParams {
    int dim;
    int sub;    // slices of dimension 0 per bucket width (1: cubic buckets)
    int n_cells;
    int n[kMaxDim];
    int stride[kMaxDim];
    double lo[kMaxDim];
    double hi[kMaxDim];     // upper corner of the sources' bounding box
    double w[kMaxDim];      // bucket width, raw coordinates
    double inv_w[kMaxDim];  // 1 / w
    double g[kMaxDim];      // metric factors
    double qs[kMaxDim];     // quantum of the 32-bit source records (a power of two)
    double iqs[kMaxDim];    // 1 / qs
    double wm;              // metric bucket width (of dimension 0: wm / sub)
    double density;         // sources per unit metric volume of the bounding box
    float max32;            // |t_k - lo_k| below which FP32 distances are bounded (0: never)
};

PCMS_HD PCMS_INLINE int bucket_of(const GridParams &p, int k, double x)
{
    double f = floor((x - p.lo[k]) * p.inv_w[k]);
    f = fmax(f, 0.0);                     // also maps NaN to 0
    f = fmin(f, (double)(p.n[k] - 1));
    return (int)f;
}

// Bucket sizing from the bounding box [lo, hi]: width cell_width (metric
// units) if > 0, else sized for about pts_per_cell sources per cubic bucket
// of that width; dimension 0 is then cut into `sub` slices per width (a
// power of two; 1 in one dimension).  Until the bucket count fits `cap`,
// sub halves first, then the width grows.
PCMS_HD inline void grid_params_compute(const double *lo, const double *hi, int dim, int64_t n,
                                        const double *g, double cell_width, double pts_per_cell,
                                        int cap, int sub, GridParams *out)
{
    GridParams p;
    p.dim = dim;
    p.sub = dim > 1 && sub > 1 ? sub : 1;
    double ext[kMaxDim];
    double vol = 1.0;
    int d_eff = 0;
    for (int k = 0; k < kMaxDim; ++k) {
        p.lo[k] = 0.0;
        p.hi[k] = 0.0;
        p.g[k] = 1.0;
        p.n[k] = 1;
        p.w[k] = 1.0;
        p.inv_w[k] = 1.0;
        p.stride[k] = 0;
        p.qs[k] = 1.0;
        p.iqs[k] = 1.0;
        ext[k] = 0.0;
    }
    for (int k = 0; k < dim; ++k) {
        p.g[k] = g[k];
        double l = lo[k], h = hi[k];
        if (!(l <= h)) {
            l = 0.0;
            h = 0.0;
        }
        p.lo[k] = l;
        p.hi[k] = h;
        // quantum 2^(E - 32) with 2^E just above the extent: every source of
        // the box maps to an integer in [0, 2^32)
        if (h > l) {
            const int e = (int)ceil(log2((h - l) * (1.0 + 1.0 / 1048576.0)));
            p.qs[k] = ldexp(1.0, e - 32);
            p.iqs[k] = ldexp(1.0, 32 - e);
        }
        ext[k] = (h - l) * p.g[k];
        if (ext[k] > 0.0) {
            vol *= ext[k];
            d_eff++;
        }
    }
    double wm;
    if (cell_width > 0.0) {
        wm = cell_width;
    } else {
        double ppc = pts_per_cell > 0.0 ? pts_per_cell : (double)(1 << dim);
        wm = d_eff > 0 ? pow(ppc * vol / (double)(n > 0 ? n : 1), 1.0 / d_eff) : 1.0;
        if (!(wm > 0.0) || !(wm < INFINITY)) wm = 1.0;
    }
    double total = 1.0;
    for (int it = 0; it < 4000; ++it) {
        total = 1.0;
        for (int k = 0; k < dim; ++k) {
            const double wk = k == 0 ? wm / p.sub : wm;
            if (ext[k] > 0.0) {
                double nk = floor(ext[k] / wk) + 1.0;
                nk = fmin(nk, 1073741825.0);   // beyond any cap
                p.n[k] = (int)nk;
                p.w[k] = wk / p.g[k];
            } else {
                p.n[k] = 1;
                p.w[k] = 1.0 / p.g[k];
            }
            p.inv_w[k] = 1.0 / p.w[k];
            total *= (double)p.n[k];
        }
        if (total <= (double)cap) break;
        if (p.sub > 1)
            p.sub /= 2;
        else
            wm *= 1.25;
    }
    if (total > (double)cap) {      // never exceed the allocated bucket count
        p.sub = 1;
        for (int k = 0; k < dim; ++k) {
            p.n[k] = 1;
            p.w[k] = (ext[k] > 0.0 ? 2.0 * ext[k] : 1.0) / p.g[k];
            p.inv_w[k] = 1.0 / p.w[k];
        }
    }
    int s = 1;
    for (int k = 0; k < dim; ++k) {
        p.stride[k] = s;
        s *= p.n[k];
    }
    p.n_cells = s;
    p.wm = wm;
    p.density = d_eff > 0 ? (double)n / vol : 0.0;
    // FP32 differences of coordinates must not overflow, and a metric factor must
    // be a normal FP32 number, below 1e20: the error of a subnormal coordinate,
    // 2^-149, then stays below the absolute slack of the bounds (1e-36 of Image32
    // in search.h, 1e-43 of BoxTest32 in bvh.h)
    p.max32 = 1e38f;
    for (int k = 0; k < dim; ++k)
        if (!(p.hi[k] - p.lo[k] < 1e38 && p.g[k] > 1.2e-38 && p.g[k] < 1e20)) p.max32 = 0.0f;
    *out = p;
}

// The buckets whose first sorted position is i (0 <= i <= n), from the n
// sorted bucket keys (each < n_cells): [lo, hi], none when hi < lo.
// Position 0 starts [0, key[0]], position i (0 < i < n) starts
// (key[i-1], key[i]] and the end n starts (key[n-1], n_cells].
PCMS_HD PCMS_INLINE void cell_run(const unsigned *keys, int n, int n_cells, int i, int &lo, int &hi)
{
    lo = i == 0 ? 0 : (int)keys[i - 1] + 1;
    hi = i == n ? n_cells : (int)keys[i];
}

PCMS_HD PCMS_INLINE unsigned bucket_key(const GridParams &p, const double *x)
{
    int id = 0;
    for (int k = 0; k < p.dim; ++k) id += bucket_of(p, k, x[k]) * p.stride[k];
    return (unsigned)id;
}

// Processing order of the targets: tiles of 8 cubic buckets per side (the
// slices of dimension 0 merged; tiled in every dimension with at least 16
// such buckets) in row-major order, and Morton order of the buckets inside
// a tile, so that a wave's consecutive targets cover a compact block of
// buckets.  Keys are below tile_key_bound(n_cells, dim).
PCMS_HD PCMS_INLINE unsigned target_key(const GridParams &p, const double *x)
{
    unsigned tile = 0, tstride = 1, local = 0;
    int nt = 0;   // tiled dimensions so far
    int tiled[kMaxDim], c[kMaxDim];
    int nk[kMaxDim];
    for (int k = 0; k < p.dim; ++k) {
        // the slices of dimension 0 are merged back into cubic buckets
        const int s = k == 0 ? p.sub : 1;
        c[k] = bucket_of(p, k, x[k]) / s;
        nk[k] = (p.n[k] + s - 1) / s;
        tiled[k] = nk[k] >= 16;
        nt += tiled[k];
    }
    int r = 0;
    for (int k = 0; k < p.dim; ++k) {
        const int sh = tiled[k] ? 3 : 0;
        tile += (unsigned)(c[k] >> sh) * tstride;
        tstride *= (unsigned)((nk[k] + (1 << sh) - 1) >> sh);
        if (tiled[k]) {
            for (int b = 0; b < 3; ++b) local |= (unsigned)((c[k] >> b) & 1) << (b * nt + r);
            ++r;
        }
    }
    return (tile << (3 * nt)) | local;
}

// Upper bound of the target keys: each tiled dimension rounds its bucket
// count up to a multiple of 8 (at most 23/16 of it, as it has >= 16).
inline double tile_key_bound(double n_cells, int dim)
{
    double f = 1.0;
    for (int k = 0; k < dim; ++k) f *= 23.0 / 16.0;
    return n_cells * f + 1.0;
}

// Sorted source coordinates are stored with an even stride (3-D points take
// four doubles), so that every point starts on a 16-byte boundary and loads
// as whole 16-byte words.
PCMS_HD PCMS_INLINE constexpr int padded_dim(int d) { return (d + 1) & ~1; }

template <int D>
PCMS_HD PCMS_INLINE void load_src(const double *__restrict__ spts, int p, double (&s)[D])
{
    constexpr int DP = padded_dim(D);
    const double *b = spts + (size_t)p * DP;
#ifdef PCMS_HOST_EMULATION
    for (int k = 0; k < D; ++k) s[k] = b[k];
#else
#pragma unroll
    for (int j = 0; j < DP / 2; ++j) {
        const double2 v = reinterpret_cast<const double2 *>(b)[j];
        s[2 * j] = v.x;
        if (2 * j + 1 < D) s[2 * j + 1] = v.y;
    }
#endif
}

// Sorted sources also keep an FP32 image of their coordinates relative to
// the grid origin, fl32(s_k - lo_k), packed with no padding (a 3-D point is
// 12 bytes and loads as one 12-byte word: ten records share a 128-byte line
// instead of eight); the searches classify candidates from it.

// Floats of storage after the FP32 and fixed-point records, which a walk's
// whole-word loads may read past the last record.
constexpr int kPad32 = 16;
#ifndef PCMS_HOST_EMULATION
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
#else
typedef float float4u __attribute__((vector_size(16), aligned(4), may_alias));
#endif

// Square root to within 2^-22 (one instruction on the GPU).
PCMS_HD PCMS_INLINE float sqrt_approx(float x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_sqrtf(x);
#else
    return sqrt(x);
#endif
}

template <int D>
PCMS_HD PCMS_INLINE void load_src32(const float *__restrict__ s32, int p, float (&s)[D])
{
    // adjacent scalar loads, which the compiler merges into one wide load
    const float *b = s32 + (size_t)p * D;
#pragma unroll
    for (int k = 0; k < D; ++k) s[k] = b[k];
}

// Sorted sources also keep a 32-bit fixed-point image of their coordinates,
// q_k = round((s_k - lo_k) / qs_k) with the power-of-two quantum qs_k of
// their box, packed with no padding (a 3-D point is 12 bytes, one load).  The
// mixed-precision fit passes read it instead of the FP64 record: it places
// the source within qs_k / 2 (about 1.2e-10 of the box) of its position, and
// (q_k - (t_k - lo_k) / qs_k) * qs_k is formed in FP64 without cancellation.
PCMS_HD PCMS_INLINE uint32_t quantize(double x, double lo, double iqs)
{
    const double v = rint((x - lo) * iqs);
    return (uint32_t)fmin(fmax(v, 0.0), 4294967295.0);
}

template <int D>
PCMS_HD PCMS_INLINE void load_srcq(const uint32_t *__restrict__ sq, int p, uint32_t (&q)[D])
{
    // adjacent scalar loads, which the compiler merges into one wide load
    const uint32_t *b = sq + (size_t)p * D;
#pragma unroll
    for (int k = 0; k < D; ++k) q[k] = b[k];
}

// Fused multiply-add in the arithmetic of its operands (__builtin_fma on
// floats would promote them and compute in FP64).
PCMS_HD PCMS_INLINE float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
PCMS_HD PCMS_INLINE double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Square root of finite x >= 0 in FP64: the reciprocal root's approximation, one
// Goldschmidt step and two Newton corrections (Markstein, "Software division and
// square root using Goldschmidt's algorithms", RNC 6, 2004), as accurate as sqrt
// (the same bits) for x from 1e-200 on; smaller ones, zero among them, give
// 1e-100.  It leaves out the range scaling of sqrt, half of its instructions.
PCMS_HD PCMS_INLINE double sqrt_unit(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    x = fmax(x, 1e-200);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return __builtin_fma(__builtin_fma(-g, g, x), h, g);
#else
    return sqrt(x < 1e-200 ? 1e-200 : x);
#endif
}

// Two consecutive doubles from a 16-byte aligned address, in one load.
PCMS_HD PCMS_INLINE void load_pair(const double *__restrict__ p, double &x, double &y)
{
#ifdef PCMS_HOST_EMULATION
    x = p[0];
    y = p[1];
#else
    const double2 v = *reinterpret_cast<const double2 *>(p);
    x = v.x;
    y = v.y;
#endif
}

// Two consecutive doubles to a 16-byte aligned address, in one store.
PCMS_HD PCMS_INLINE void store_pair(double *__restrict__ p, double x, double y)
{
#ifdef PCMS_HOST_EMULATION
    p[0] = x;
    p[1] = y;
#else
    *reinterpret_cast<double2 *>(p) = make_double2(x, y);
#endif
}

// Atomic add to a word of the block's LDS.
PCMS_HD PCMS_INLINE void lds_add(int *w, int v)
{
#ifdef PCMS_HOST_EMULATION
    __atomic_fetch_add(w, v, __ATOMIC_RELAXED);
#else
    atomicAdd(w, v);
#endif
}

// --- lane groups -----------------------------------------------------------
// G consecutive lanes of a wave (G a power of two, <= 16) cooperate on one
// target.  Group operations must be reached by all G lanes together (the
// control flow around them is uniform within the group).
template <int G>
struct Grp {
    int q;   // lane index inside the group
#ifdef PCMS_HOST_EMULATION
    EmuGroup *emu;
    unsigned ballot(bool p) const { return pcms_emu_ballot(emu, q, p); }
    template <class T>
    T sum(T x) const { return pcms_emu_sum(emu, q, x); }
    template <class T>
    T min(T x) const { return pcms_emu_min(emu, q, x); }
    bool all(bool p) const { return pcms_emu_min(emu, q, (int)p) != 0; }
    void sync() const { pcms_emu_sync(emu, q); }
    // lane j's x, on every lane
    template <class T>
    T from(T x, int j) const { return (T)pcms_emu_sum(emu, q, q == j ? (double)x : 0.0); }
#else
    __device__ PCMS_INLINE unsigned ballot(bool p) const
    {
        const unsigned long long m = __ballot(p);
        const int base = (int)(__lane_id() & ~(unsigned)(G - 1));
        return (unsigned)(m >> base) & ((1u << G) - 1u);
    }
    // butterfly: every lane ends with the same value, summed in the same order
    template <class T>
    __device__ PCMS_INLINE T sum(T x) const
    {
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            T y = __shfl_xor(x, off, 64);
            x = (q & off) ? y + x : x + y;
        }
        return x;
    }
    template <class T>
    __device__ PCMS_INLINE T min(T x) const
    {
#pragma unroll
        for (int off = G / 2; off > 0; off >>= 1) {
            T y = __shfl_xor(x, off, 64);
            x = y < x ? y : x;
        }
        return x;
    }
    __device__ PCMS_INLINE bool all(bool p) const { return min((int)p) != 0; }
    // lane j's x, on every lane (j a constant once unrolled)
    __device__ PCMS_INLINE uint32_t from(uint32_t x, int j) const
    {
        static_assert(G == 4, "quads");
        const int v = (int)x;
        return (uint32_t)(j == 0   ? __builtin_amdgcn_mov_dpp(v, 0x00, 0xf, 0xf, true)
                          : j == 1 ? __builtin_amdgcn_mov_dpp(v, 0x55, 0xf, 0xf, true)
                          : j == 2 ? __builtin_amdgcn_mov_dpp(v, 0xaa, 0xf, 0xf, true)
                                   : __builtin_amdgcn_mov_dpp(v, 0xff, 0xf, 0xf, true));
    }
    __device__ PCMS_INLINE double from(double x, int j) const
    {
        const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
        const unsigned long long lo = from((uint32_t)b, j), hi = from((uint32_t)(b >> 32), j);
        return __builtin_bit_cast(double, (hi << 32) | lo);
    }
    // orders this lane's LDS accesses against the group's (one wavefront)
    __device__ PCMS_INLINE void sync() const
    {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
#endif
    // lanes of mask m below this one
    PCMS_HD PCMS_INLINE int below(unsigned m) const
    {
        return __builtin_popcount(m & ((1u << q) - 1u));
    }
};

#ifndef PCMS_HOST_EMULATION
// One lane per target: the collectives are the lane's own values (the general
// form's wave ballots and shifts cost six instructions per candidate).
template <>
struct Grp<1> {
    int q;
    PCMS_HD PCMS_INLINE unsigned ballot(bool p) const { return p ? 1u : 0u; }
    template <class T>
    PCMS_HD PCMS_INLINE T sum(T x) const { return x; }
    template <class T>
    PCMS_HD PCMS_INLINE T min(T x) const { return x; }
    PCMS_HD PCMS_INLINE bool all(bool p) const { return p; }
    template <class T>
    PCMS_HD PCMS_INLINE T from(T x, int) const { return x; }
    PCMS_HD PCMS_INLINE void sync() const {}
    PCMS_HD PCMS_INLINE int below(unsigned) const { return 0; }
};
#endif

// --- pieces of the stable radix sort (one 8-bit digit per pass) ---------------
constexpr int kSortThreads = 256;          // 4 waves of 64
constexpr int kSortRounds = 16;            // keys per thread of a block
constexpr int kSortItems = kSortThreads * kSortRounds;
// Blocks up to which a scatter sums the other blocks' counts itself: one launch
// less per pass, for 256 nb more reads per block.
constexpr int kDirectBlocks = 32;

// Slot in its block of thread t's key of round r: each wave has a quarter of the
// block's keys, 64 a round.
PCMS_HD PCMS_INLINE int sort_slot(int t, int r)
{
    return (t >> 6) * (kSortItems / 4) + r * 64 + (t & 63);
}

// Lanes of one wave holding the same digit: AND of the per-bit ballots.
PCMS_HD PCMS_INLINE unsigned long long digit_match(unsigned long long valid,
                                                   const unsigned long long (&bits)[8], int digit)
{
    unsigned long long mask = valid;
    for (int b = 0; b < 8; ++b) mask &= ((digit >> b) & 1) ? bits[b] : ~bits[b];
    return mask;
}

PCMS_HD PCMS_INLINE unsigned long long lanes_below(int lane)
{
    return lane == 0 ? 0ull : ((~0ull) >> (64 - lane));
}

// The waves' counts of a digit become their offsets in the digit's run; returns
// the run's length.
PCMS_HD PCMS_INLINE int wave_offsets(int (&cnt)[4][256], int digit)
{
    int run = 0;
    for (int v = 0; v < 4; ++v) {
        const int c = cnt[v][digit];
        cnt[v][digit] = run;
        run += c;
    }
    return run;
}

// A digit's keys in all nb blocks and in those before block b, from its row of
// the blocks' counts (DIRECT) or of their inclusive sums.
template <bool DIRECT>
PCMS_HD PCMS_INLINE void digit_counts(const int *row, int nb, int b, int &total, int &before)
{
    before = 0;
    if (DIRECT) {
        total = 0;
        for (int x = 0; x < nb; ++x) {
            const int c = row[x];
            before += x < b ? c : 0;
            total += c;
        }
    } else {
        total = row[nb - 1];
        if (b > 0) before = row[b - 1];
    }
}

}  // namespace pcms
