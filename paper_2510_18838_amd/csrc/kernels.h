// The one-problem neighbour-list and field-transfer kernels (one or four lanes
// per target, targets in tiled Morton order so that the lanes of a wave search
// overlapping stencils), instantiated per dimension in mls_d1.hip .. mls_d5.hip
// and mls4_d1.hip .. mls4_d5.hip so that the variants compile in parallel.  The per-target work
// (search, moment assembly, Cholesky, evaluation) is in fit.h / search.h.
#pragma once

#include <hip/hip_runtime.h>

#include "fit.h"
#include "launch_common.h"

namespace pcms {

// Lanes per target (G consecutive lanes of a wave): one, or four for few
// targets and for long lists (target_lanes in mls.hip).  The block's targets are consecutive
// in processing order and each owns `stride` LDS words.
constexpr int kQuad = 4;

using KernelFn = void (*)(KArgs);

// Kernel of dimension D and G lanes per target for (degree, precision, unit
// metric); defined in mls_d<D>.hip and, for quads, mls4_d<D>.hip; the same on
// an LBVH in bvh_d<D>.hip.
template <int D, int G>
KernelFn transfer_kernel(int degree, int precision, bool unit);
template <int D, int G>
KernelFn nbr_kernel(bool unit);
template <int D>
KernelFn transfer_kernel_bvh(int degree, int precision, bool unit);
template <int D>
KernelFn nbr_kernel_bvh(bool unit);
// The operator-emission variant of transfer_kernel; defined in op_d<D>.hip
// and op4_d<D>.hip, and on an LBVH in bvh_op_d<D>.hip.
template <int D, int G>
KernelFn operator_kernel(int degree, int precision, bool unit);
template <int D>
KernelFn operator_kernel_bvh(int degree, int precision, bool unit);

namespace {

template <int D, bool UNIT, int G, bool BVH = false>
__global__ void __launch_bounds__(256) k_neighbors(KArgs a)
{
    extern __shared__ int lds[];
    const int lb = logical_block(a.n_blocks);
    if (lb >= a.n_blocks) return;
    const int slot = (int)threadIdx.x / G;
    const int i = lb * ((int)blockDim.x / G) + slot;
    const bool active = i < a.n_tgt;   // uniform within a group
    const Grp<G> g{(int)(threadIdx.x & (G - 1))};
    int st = 0;
    if (active) {
        const GridParams gp = *a.gp;
        st = nbr_target<D, UNIT, G, BVH>(a, gp, i, lds + slot * a.stride, g);
    }
    add_summary(a.summary, st, active && g.q == 0);
}

// Waves per SIMD the register allocator targets (168 VGPRs for 3, 256 for
// 2): three, except for MIXED_REFINE in 4-D and 5-D (240-1100 bytes of
// spill per lane under 168 VGPRs) and the 4-D and 5-D quadratic bases in
// any precision (1-2 KB), which get two.  Measured with the row walks that
// the row tables replaced: the 5-D linear MIXED_REFINE kernel went from 3-6 %
// slower than FP64 to level with it (74.3 against 76.1 ms).  (With the tables
// and four lanes, which need fewer registers, that kernel measures 26.0 ms with
// two and 23.5 with three on 2M targets.)  The low-dimensional kernels need the
// third wave for latency even where they spill a little: at two, the 3-D
// quadratic MIXED_REFINE kernel slowed from 7.0 to 9.2 ms and the 2-D quadratic
// one from 0.43 to 0.48 ms.
template <int PREC, int D, int P>
constexpr int waves_for()
{
    return D >= 4 && (PREC == PCMS_MIXED_REFINE || P == 2) ? 2 : 3;
}

template <int D, int P, int PREC, bool UNIT, int G, bool BVH = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_for<PREC, D, P>())))
k_transfer(KArgs a)
{
    extern __shared__ int lds[];
    const int lb = logical_block(a.n_blocks);
    if (lb >= a.n_blocks) return;
    const int slot = (int)threadIdx.x / G;
    const int i = lb * ((int)blockDim.x / G) + slot;
    const bool active = i < a.n_tgt;   // uniform within a group
    const Grp<G> g{(int)(threadIdx.x & (G - 1))};
    int st = 0;
    if (active) {
        const GridParams gp = *a.gp;
        st = xfer_target<D, P, PREC, UNIT, G, false, BVH>(a, gp, i, lds + slot * a.stride, g);
    }
    add_summary(a.summary, st, active && g.q == 0);
}

// The same kernel writing the transfer operator instead of field values.
template <int D, int P, int PREC, bool UNIT, int G, bool BVH = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_for<PREC, D, P>())))
k_operator(KArgs a)
{
    extern __shared__ int lds[];
    const int lb = logical_block(a.n_blocks);
    if (lb >= a.n_blocks) return;
    const int slot = (int)threadIdx.x / G;
    const int i = lb * ((int)blockDim.x / G) + slot;
    const bool active = i < a.n_tgt;   // uniform within a group
    const Grp<G> g{(int)(threadIdx.x & (G - 1))};
    int st = 0;
    if (active) {
        const GridParams gp = *a.gp;
        st = xfer_target<D, P, PREC, UNIT, G, true, BVH>(a, gp, i, lds + slot * a.stride, g);
    }
    add_summary(a.summary, st, active && g.q == 0);
}

template <int D, int P, bool UNIT, int G, bool BVH = false>
KernelFn pick_prec(int precision)
{
    return precision == PCMS_FP64  ? (KernelFn)k_transfer<D, P, PCMS_FP64, UNIT, G, BVH>
         : precision == PCMS_MIXED ? (KernelFn)k_transfer<D, P, PCMS_MIXED, UNIT, G, BVH>
                                   : (KernelFn)k_transfer<D, P, PCMS_MIXED_REFINE, UNIT, G, BVH>;
}

template <int D, int P, bool UNIT, int G, bool BVH = false>
KernelFn pick_prec_op(int precision)
{
    return precision == PCMS_FP64  ? (KernelFn)k_operator<D, P, PCMS_FP64, UNIT, G, BVH>
         : precision == PCMS_MIXED ? (KernelFn)k_operator<D, P, PCMS_MIXED, UNIT, G, BVH>
                                   : (KernelFn)k_operator<D, P, PCMS_MIXED_REFINE, UNIT, G, BVH>;
}

}  // namespace

// Body of the per-dimension definitions.
#define PCMS_DEFINE_DIM_KERNELS(DD, GG)                                                \
    template <>                                                                        \
    KernelFn transfer_kernel<DD, GG>(int degree, int precision, bool unit)             \
    {                                                                                  \
        if (unit)                                                                      \
            return degree == 0 ? pick_prec<DD, 0, true, GG>(precision)                 \
                 : degree == 1 ? pick_prec<DD, 1, true, GG>(precision)                 \
                               : pick_prec<DD, 2, true, GG>(precision);                \
        return degree == 0 ? pick_prec<DD, 0, false, GG>(precision)                    \
             : degree == 1 ? pick_prec<DD, 1, false, GG>(precision)                    \
                           : pick_prec<DD, 2, false, GG>(precision);                   \
    }                                                                                  \
    template <>                                                                        \
    KernelFn nbr_kernel<DD, GG>(bool unit)                                             \
    {                                                                                  \
        return unit ? (KernelFn)k_neighbors<DD, true, GG>                              \
                    : (KernelFn)k_neighbors<DD, false, GG>;                            \
    }

#define PCMS_DEFINE_DIM_BVH(DD)                                                        \
    template <>                                                                        \
    KernelFn transfer_kernel_bvh<DD>(int degree, int precision, bool unit)             \
    {                                                                                  \
        if (unit)                                                                      \
            return degree == 0 ? pick_prec<DD, 0, true, 1, true>(precision)            \
                 : degree == 1 ? pick_prec<DD, 1, true, 1, true>(precision)            \
                               : pick_prec<DD, 2, true, 1, true>(precision);           \
        return degree == 0 ? pick_prec<DD, 0, false, 1, true>(precision)               \
             : degree == 1 ? pick_prec<DD, 1, false, 1, true>(precision)               \
                           : pick_prec<DD, 2, false, 1, true>(precision);              \
    }                                                                                  \
    template <>                                                                        \
    KernelFn nbr_kernel_bvh<DD>(bool unit)                                             \
    {                                                                                  \
        return unit ? (KernelFn)k_neighbors<DD, true, 1, true>                         \
                    : (KernelFn)k_neighbors<DD, false, 1, true>;                       \
    }

#define PCMS_DEFINE_DIM_OPERATOR_BVH(DD)                                               \
    template <>                                                                        \
    KernelFn operator_kernel_bvh<DD>(int degree, int precision, bool unit)             \
    {                                                                                  \
        if (unit)                                                                      \
            return degree == 0 ? pick_prec_op<DD, 0, true, 1, true>(precision)         \
                 : degree == 1 ? pick_prec_op<DD, 1, true, 1, true>(precision)         \
                               : pick_prec_op<DD, 2, true, 1, true>(precision);        \
        return degree == 0 ? pick_prec_op<DD, 0, false, 1, true>(precision)            \
             : degree == 1 ? pick_prec_op<DD, 1, false, 1, true>(precision)            \
                           : pick_prec_op<DD, 2, false, 1, true>(precision);           \
    }

#define PCMS_DEFINE_DIM_OPERATOR(DD, GG)                                               \
    template <>                                                                        \
    KernelFn operator_kernel<DD, GG>(int degree, int precision, bool unit)             \
    {                                                                                  \
        if (unit)                                                                      \
            return degree == 0 ? pick_prec_op<DD, 0, true, GG>(precision)              \
                 : degree == 1 ? pick_prec_op<DD, 1, true, GG>(precision)              \
                               : pick_prec_op<DD, 2, true, GG>(precision);             \
        return degree == 0 ? pick_prec_op<DD, 0, false, GG>(precision)                 \
             : degree == 1 ? pick_prec_op<DD, 1, false, GG>(precision)                 \
                           : pick_prec_op<DD, 2, false, GG>(precision);                \
    }

}  // namespace pcms
