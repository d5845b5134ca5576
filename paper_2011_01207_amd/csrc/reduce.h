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

// E_real of slot s = eipart[s] + sum of the jbuf slots of s in the reverse index (JSum; four loads
// in flight).
template <typename R>
__device__ __forceinline__ void real_reduce(int s, const double* __restrict__ eipart, const R* __restrict__ jbuf,
                                            const int* __restrict__ rev_ptr, const int* __restrict__ rev_idx,
                                            double* __restrict__ ereal)
{
    using R4 = typename V4<R>::T;
    using J = JSum<R>;
    double e0 = J::start(eipart[3 * (size_t)s]), e1 = J::start(eipart[3 * (size_t)s + 1]),
           e2 = J::start(eipart[3 * (size_t)s + 2]);
    const R4* jb = reinterpret_cast<const R4*>(jbuf);
    const int k1 = rev_ptr[s + 1];
    int k = rev_ptr[s];
    for (; k + 4 <= k1; k += 4) {
        R4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = jb[rev_idx[k + u]];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            e0 += J::term(v[u].x);
            e1 += J::term(v[u].y);
            e2 += J::term(v[u].z);
        }
    }
    for (; k < k1; ++k) {
        const R4 v = jb[rev_idx[k]];
        e0 += J::term(v.x);
        e1 += J::term(v.y);
        e2 += J::term(v.z);
    }
    ereal[3 * (size_t)s] = J::finish(e0);
    ereal[3 * (size_t)s + 1] = J::finish(e1);
    ereal[3 * (size_t)s + 2] = J::finish(e2);
}

}  // namespace amoeba
