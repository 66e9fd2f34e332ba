// Launchers of the one-problem neighbour-list and field-transfer kernels
// (kernels.h): LDS sizing, block choice, XCD-aware grid, variant dispatch.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "internal.h"
#include "kernels.h"

namespace pcms {

namespace {

__global__ void k_zero_ints(int32_t *p, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

KernelFn xfer_for(int d, int p, int precision, bool unit, bool bvh, bool quad)
{
    if (bvh) {
        switch (d) {
        case 1: return transfer_kernel_bvh<1>(p, precision, unit);
        case 2: return transfer_kernel_bvh<2>(p, precision, unit);
        case 3: return transfer_kernel_bvh<3>(p, precision, unit);
        case 4: return transfer_kernel_bvh<4>(p, precision, unit);
        case 5: return transfer_kernel_bvh<5>(p, precision, unit);
        }
        return nullptr;
    }
    switch (d) {
    case 1: return quad ? transfer_kernel<1, kQuad>(p, precision, unit) : transfer_kernel<1, 1>(p, precision, unit);
    case 2: return quad ? transfer_kernel<2, kQuad>(p, precision, unit) : transfer_kernel<2, 1>(p, precision, unit);
    case 3: return quad ? transfer_kernel<3, kQuad>(p, precision, unit) : transfer_kernel<3, 1>(p, precision, unit);
    case 4: return quad ? transfer_kernel<4, kQuad>(p, precision, unit) : transfer_kernel<4, 1>(p, precision, unit);
    case 5: return quad ? transfer_kernel<5, kQuad>(p, precision, unit) : transfer_kernel<5, 1>(p, precision, unit);
    }
    return nullptr;
}

KernelFn op_for(int d, int p, int precision, bool unit, bool bvh, bool quad)
{
    if (bvh) {
        switch (d) {
        case 1: return operator_kernel_bvh<1>(p, precision, unit);
        case 2: return operator_kernel_bvh<2>(p, precision, unit);
        case 3: return operator_kernel_bvh<3>(p, precision, unit);
        case 4: return operator_kernel_bvh<4>(p, precision, unit);
        case 5: return operator_kernel_bvh<5>(p, precision, unit);
        }
        return nullptr;
    }
    switch (d) {
    case 1: return quad ? operator_kernel<1, kQuad>(p, precision, unit) : operator_kernel<1, 1>(p, precision, unit);
    case 2: return quad ? operator_kernel<2, kQuad>(p, precision, unit) : operator_kernel<2, 1>(p, precision, unit);
    case 3: return quad ? operator_kernel<3, kQuad>(p, precision, unit) : operator_kernel<3, 1>(p, precision, unit);
    case 4: return quad ? operator_kernel<4, kQuad>(p, precision, unit) : operator_kernel<4, 1>(p, precision, unit);
    case 5: return quad ? operator_kernel<5, kQuad>(p, precision, unit) : operator_kernel<5, 1>(p, precision, unit);
    }
    return nullptr;
}

KernelFn nbr_for(int d, bool unit, bool bvh, bool quad)
{
    if (bvh) {
        switch (d) {
        case 1: return nbr_kernel_bvh<1>(unit);
        case 2: return nbr_kernel_bvh<2>(unit);
        case 3: return nbr_kernel_bvh<3>(unit);
        case 4: return nbr_kernel_bvh<4>(unit);
        case 5: return nbr_kernel_bvh<5>(unit);
        }
        return nullptr;
    }
    switch (d) {
    case 1: return quad ? nbr_kernel<1, kQuad>(unit) : nbr_kernel<1, 1>(unit);
    case 2: return quad ? nbr_kernel<2, kQuad>(unit) : nbr_kernel<2, 1>(unit);
    case 3: return quad ? nbr_kernel<3, kQuad>(unit) : nbr_kernel<3, 1>(unit);
    case 4: return quad ? nbr_kernel<4, kQuad>(unit) : nbr_kernel<4, 1>(unit);
    case 5: return quad ? nbr_kernel<5, kQuad>(unit) : nbr_kernel<5, 1>(unit);
    }
    return nullptr;
}

bool unit_metric(const Grid *g)
{
    for (int k = 0; k < g->dim; ++k)
        if (g->g[k] != 1.0) return false;
    return true;
}

// LDS words of a target (target_words); the per-target stride is odd so
// neighbouring targets start in different banks.
int lane_words(const LaunchSpec &ls)
{
    return target_words(ls.radius.mode, ls.radius.k, ls.k_cap, ls.grid->dim);
}
int target_stride(const LaunchSpec &ls) { return lane_words(ls) | 1; }

// Lanes per target.  A lane alone takes its target's some hundred dependent
// loads one after another, which only pays when enough waves are resident to
// hide them; four lanes share a target's candidates and the loads of its fit,
// and its LDS is a quarter per wave, but they repeat the fit's arithmetic.
// Four pay where
// * there are few targets: kernel times with one lane and with four: 2-D linear,
//   1.5k targets, 76 and 37 us; 3-D linear, 15k targets, 118 and 62 us; 3-D
//   linear, 30k targets among 3M sources, 376 and 215 us; 3-D quadratic, 500k
//   targets, 733 and 967 us.  The line is one wave of quads for each of the
//   SIMD slots that the kernel's registers leave: 3 x 1024, and 2 x 1024 for the
//   quadratic bases in 4-D and 5-D.  Calls in us with one lane and with four,
//   kNN on a kept grid of 200k sources: linear, 49k targets, 3-D 296 and 265,
//   5-D 1785 and 1390, MIXED_REFINE 4-D 568 and 605 (growing radius 536 and
//   423), 5-D 1811 and 1592; 3-D quadratic, 16k targets 293 and 256, 49k 305 and 293,
//   MIXED_REFINE 322 and 320; 4-D quadratic MIXED_REFINE, 32k targets 708 and
//   562, 49k 691 and 746; 5-D 2016 and 1840, 2196 and 2550; MIXED, 4-D 685 and
//   551, 674 and 719; 5-D 2038 and 2084, 2238 and 3041.  The FP64 kernels of
//   those bases spill 2 KB per lane, which four lanes do four times, so
//   their line is one wave of quads per CU: 4-D, 4k targets 681 and 581, 8k 713
//   and 698, 16k 714 and 802, 32k 814 and 1335; 5-D, 2766 and 2193, 2841 and
//   3136, 2949 and 3563, 3926 and 6401.
// * or long lists leave few one-lane waves per CU, the fit is small, and the
//   radius is not a k-th distance (whose window walks share badly).  Calls in
//   us with one lane and with four, growing radius: 5-D linear FP64, 1M
//   targets, k_cap 96 (5 waves): 16121 and 9600, MIXED_REFINE 16279 and 12763;
//   5-D k_cap 80 (6 waves) 1023 and 884, MIXED_REFINE 1029 and 1083; k_cap 128
//   (4 waves): 4-D 1377 and 1063, 3-D 1188 and 1065, 2-D 738 and 762; k_cap 96
//   in 3-D (5 waves) 906 and 958; quadratic bases lose everywhere (4-D, k_cap
//   96: 4605 and 11204).
// * The lists alone have no fit, and the ranking by source index is shared:
//   growing radius, k_cap 64 (7-8 waves): 2-D 497 and 397, 3-D 601 and 500,
//   4-D 613 and 563, 5-D 938 and 817; k_cap 32 420 and 426 (3-D).  k-th
//   distances: k 85 (6 waves) 1016 and 743 (2-D), 1347 and 1039 (3-D), 4151
//   and 3664 (5-D); k 64 (8 waves) 1681 and 1673 (4-D), 2496 and 2564 (5-D).
constexpr int kCus = 256, kQuadsPerWave = 64 / kQuad;
constexpr int kListsAlone = -1;   // for a degree
int64_t quad_targets(int dim, int degree, int precision)
{
    if (dim < 4 || degree < 2) return 3 * 4 * kCus * kQuadsPerWave;
    return (precision == PCMS_FP64 ? 1 : 2 * 4) * kCus * kQuadsPerWave;
}
int target_lanes(const LaunchSpec &ls, int degree, int precision)
{
    if (ls.grid->lbvh) return 1;
    // (a launch has fewer than 2^32 threads)
    if (ls.n_tgt > ((int64_t)1 << 29)) return 1;
    if (ls.n_tgt <= quad_targets(ls.grid->dim, degree, precision)) return kQuad;
    const int waves = (160 << 10) / (64 * target_stride(ls) * (int)sizeof(int));
    const bool knn = ls.radius.mode == PCMS_RADIUS_KNN;
    if (degree == kListsAlone) return waves <= (knn ? 6 : 9) ? kQuad : 1;
    const int dim = ls.grid->dim;
    return degree <= 1 && !knn && dim >= 3 && waves <= (dim == 5 ? 5 : 4) ? kQuad : 1;
}

// Threads per block: the targets' LDS fits 64 KiB, or the block is one wave,
// whose 64 targets of kMaxWords take 67,840 bytes at most (a workgroup may have
// 160 KiB).  Single
// waves fill what the LDS of a CU leaves (5-D linear, k_cap 96, 2M targets, one
// lane per target: blocks of 128, the most that fit, keep 4 waves and take 44.8
// ms, single waves 5 and 31.2), and no wave waits for its block's others: 1M
// neighbour lists 1243 -> 1154 us, the LBVH 4281 -> 4195; the 3-D quadratic
// kernel measures the same (4.26 and 4.28 ms).
int pick_block(int requested, const LaunchSpec &ls, int lanes)
{
    int b = requested > 0 ? requested : 64;
    while (b > 64 && (size_t)(b / lanes) * target_stride(ls) * sizeof(int) > 65536) b >>= 1;
    return b;
}

size_t block_lds(int block, const LaunchSpec &ls, int lanes)
{
    return (size_t)(block / lanes) * target_stride(ls) * sizeof(int);
}

KArgs base_args(const LaunchSpec &ls, int block, int lanes)
{
    KArgs a{};
    a.gp = ls.grid->params;
    a.cs = ls.grid->cell_start;
    a.spts = ls.grid->spts;
    a.spts32 = ls.grid->spts32;
    a.sq = ls.grid->sq;
    a.bvh_nodes = ls.grid->bvh_nodes;
    a.perm = ls.grid->perm;
    a.tgt = ls.tgt;
    a.tperm = ls.tperm;
    a.n_tgt = (int)ls.n_tgt;
    a.mode = ls.radius.mode;
    a.k = ls.radius.k;
    a.n_min = ls.radius.n_min;
    a.max_iter = ls.radius.max_iter;
    a.r = ls.radius.r;
    a.k_cap = ls.k_cap;
    const int tpb = block / lanes;
    a.n_blocks = (int)((ls.n_tgt + tpb - 1) / tpb);
    a.words = lane_words(ls);
    a.stride = target_stride(ls);
    a.summary = ls.summary;
    return a;
}

}  // namespace

pcms_status zero_ints(int32_t *p, int n, hipStream_t s)
{
    k_zero_ints<<<(n + 255) / 256, 256, 0, s>>>(p, n);
    PCMS_HIP(hipGetLastError());
    return PCMS_OK;
}

pcms_status launch_neighbors(const LaunchSpec &ls, int32_t *nbr, int32_t *n_kept,
                             int32_t *n_found, double *r2, uint8_t *status, hipStream_t s)
{
    if (ls.n_tgt == 0) return PCMS_OK;
    const int lanes = target_lanes(ls, kListsAlone, PCMS_FP64);
    const int block = pick_block(ls.block, ls, lanes);
    KArgs a = base_args(ls, block, lanes);
    a.nbr = nbr;
    a.n_kept = n_kept;
    a.n_found = n_found;
    a.r2 = r2;
    a.status = status;
    KernelFn fn = nbr_for(ls.grid->dim, unit_metric(ls.grid), ls.grid->lbvh != 0, lanes > 1);
    const int launch = launch_blocks(a.n_blocks);
    const size_t shm = block_lds(block, ls, lanes);
    hipLaunchKernelGGL(fn, dim3(launch), dim3(block), shm, s, a);
    PCMS_HIP(hipGetLastError());
    return PCMS_OK;
}

pcms_status launch_transfer(const LaunchSpec &ls, const double *svals, int n_fields, int degree,
                            int weight, int precision, double lambda, double *out,
                            double *stage, uint8_t *status, hipStream_t s)
{
    if (ls.n_tgt == 0) return PCMS_OK;
    const int lanes = target_lanes(ls, degree, precision);
    const int block = pick_block(ls.block, ls, lanes);
    KArgs a = base_args(ls, block, lanes);
    a.svals = svals;
    a.nf = n_fields;
    a.nfs = padded_dim(n_fields);
    a.weight = weight;
    a.lambda = lambda;
    a.out = out;
    a.stage = stage;
    a.status = status;
    KernelFn fn = xfer_for(ls.grid->dim, degree, precision, unit_metric(ls.grid),
                           ls.grid->lbvh != 0, lanes > 1);
    const int launch = launch_blocks(a.n_blocks);
    const size_t shm = block_lds(block, ls, lanes);
    hipLaunchKernelGGL(fn, dim3(launch), dim3(block), shm, s, a);
    PCMS_HIP(hipGetLastError());
    return PCMS_OK;
}

pcms_status launch_operator(const LaunchSpec &ls, int degree, int weight, int precision,
                            double lambda, double *op_w, int32_t *op_c, int32_t *op_n,
                            uint8_t *status, hipStream_t s)
{
    if (ls.n_tgt == 0) return PCMS_OK;
    const int lanes = target_lanes(ls, degree, precision);
    const int block = pick_block(ls.block, ls, lanes);
    KArgs a = base_args(ls, block, lanes);
    a.weight = weight;
    a.lambda = lambda;
    a.op_w = op_w;
    a.op_c = op_c;
    a.op_n = op_n;
    a.status = status;
    KernelFn fn = op_for(ls.grid->dim, degree, precision, unit_metric(ls.grid),
                         ls.grid->lbvh != 0, lanes > 1);
    const int launch = launch_blocks(a.n_blocks);
    const size_t shm = block_lds(block, ls, lanes);
    hipLaunchKernelGGL(fn, dim3(launch), dim3(block), shm, s, a);
    PCMS_HIP(hipGetLastError());
    return PCMS_OK;
}

// Slots per target of an operator: the most entries of a kept list.
int operator_width(const LaunchSpec &ls)
{
    return target_kept(ls.radius.mode, ls.radius.k, ls.k_cap);
}

}  // namespace pcms
