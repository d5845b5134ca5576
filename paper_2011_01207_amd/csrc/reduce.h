// Deterministic FP64 reductions without device-wide fences or atomics (paper, "Precision study
// and Validation": tree reductions keep the rounding error logarithmic).  A kernel reduces its
// values per 256-thread workgroup in a fixed tree order and writes one partial per workgroup;
// the next kernel of the stream sums the partials in index order (redundantly in every
// workgroup that needs the total), so the result does not depend on scheduling and no
// workgroup waits on another.
#pragma once
#include "common.h"

namespace amoeba {

// Sum of NV values over the 256 threads of a workgroup, in a fixed order; every thread gets
// the totals.  Each wave folds its 64 values with shuffles (lane 0's association order is the
// one kept), then the four wave sums are added in wave order.  Must be reached by all threads
// of the workgroup.
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV])
{
    __shared__ double sh[NV][4];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < NV; ++k)
            v[k] += __shfl_xor(v[k], off);
    __syncthreads();   // an earlier call's readers are done with sh
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < NV; ++k)
            sh[k][w] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k)
        v[k] = (sh[k][0] + sh[k][1]) + (sh[k][2] + sh[k][3]);
}

// Total of n partials of NV values each (layout [n][NV]), in a fixed order; every thread of
// the workgroup gets the totals.
template <int NV>
__device__ __forceinline__ void sum_partials(const double* __restrict__ part, int n, double (&tot)[NV])
{
    for (int k = 0; k < NV; ++k)
        tot[k] = 0.0;
    for (int b = threadIdx.x; b < n; b += 256)
        for (int k = 0; k < NV; ++k)
            tot[k] += part[(size_t)b * NV + k];
    block_sum<NV>(tot);
}

// v of the lane whose index differs by the mask of a quad permutation
template <int CTRL> __device__ __forceinline__ double quad_swap(double v)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false));
}

// E_real of slot s = eipart[s] + sum of the jbuf slots of s in the reverse index (JSum), by four
// consecutive lanes (thread = 4 s + lane of the quad; all four call it): each takes every fourth
// entry, two loads in flight, and writes one component.  Bound by the latency of its dependent loads
// (about nine entries a slot) and their bytes: 41 us at 864,000 atoms in mixed precision, 61 in FP64; one
// lane per slot, four loads in flight, took 48 and 70 us.
template <typename R>
__device__ __forceinline__ void real_reduce(int thread, const double* __restrict__ eipart, const R* __restrict__ jbuf,
                                            const int* __restrict__ rev_ptr, const int* __restrict__ rev_idx,
                                            double* __restrict__ ereal)
{
    using R4 = typename V4<R>::T;
    using J = JSum<R>;
    const int s = thread >> 2, q = thread & 3;
    const R4* jb = reinterpret_cast<const R4*>(jbuf);
    const int k0 = rev_ptr[s], k1 = rev_ptr[s + 1];
    const double ei = q < 3 ? eipart[3 * (size_t)s + q] : 0.0;
    double e0 = 0.0, e1 = 0.0, e2 = 0.0;
    for (int k = k0 + q; k < k1; k += 8) {
        const bool two = k + 4 < k1;
        const int i0 = rev_idx[k], i1 = two ? rev_idx[k + 4] : i0;
        const R4 a = jb[i0], b = jb[i1];
        e0 += J::term(a.x);
        e1 += J::term(a.y);
        e2 += J::term(a.z);
        if (two) {
            e0 += J::term(b.x);
            e1 += J::term(b.y);
            e2 += J::term(b.z);
        }
    }
    e0 += quad_swap<0xb1>(e0);  // lane ^ 1
    e1 += quad_swap<0xb1>(e1);
    e2 += quad_swap<0xb1>(e2);
    e0 += quad_swap<0x4e>(e0);  // lane ^ 2
    e1 += quad_swap<0x4e>(e1);
    e2 += quad_swap<0x4e>(e2);
    if (q < 3)
        ereal[3 * (size_t)s + q] = J::finish(J::start(ei) + (q == 0 ? e0 : q == 1 ? e1 : e2));
}

}  // namespace amoeba
