// Device code of the plane path's spread (plane.hip), shared with the launch of a small system's
// tiles and spread together (realspace.hip).  What the passes are: plane.hip.
#pragma once
#include <type_traits>

#include "common.h"
#include "plane_fft.h"
#include "spline.h"

namespace amoeba {

template <typename R> struct PlT;
template <> struct PlT<float> { using C = float2; using R4 = float4; };
template <> struct PlT<double> { using C = double2; using R4 = double4; };

constexpr int kPlThreads = 512;         // threads per workgroup of the row-chunk passes (spread, gather)
constexpr int kPlThreadsLarge = 256;    // the same on large grids, in smaller row chunks
constexpr int kPlLargeWG = 1024;        // row-chunk workgroups of 512 threads above which a grid is large
constexpr int kPlTargetWGLarge = 3456;  // row-chunk workgroups the chunking aims at on a large grid
constexpr int kPlColThreads = 512;      // threads per workgroup of the column passes at most
constexpr int kPlYxyThreads = 1024;     // threads per workgroup of the one-launch y-x-y pass at most
constexpr size_t kPlLdsMax = 64 * 1024; // LDS of one workgroup
constexpr int kPlTargetWG = 432;        // workgroups per row-chunk pass the chunking aims at
// Wave priority of the transform and interpolation passes: they run beside the real-space tiles
// (second stream) and are latency bound, so their waves issue first where both share a SIMD;
// the tiles fill the remaining issue slots (solve 1.44 -> 1.40 ms on water_96000).
constexpr int kPlPassPrio = 3;

// Geometry and chunking shared by the passes.  Rows y = 2p and 2p + 1 form row pair p; the
// spread and the interpolation work on chunks of Pc consecutive pairs, the y and x transforms
// on chunks of kc consecutive kz columns.
struct PlaneGeom {
    int nt;       // threads per workgroup of the row-chunk passes
    int nty, ntx; // threads per workgroup of the y and the x pass
    int npad;     // slots (the plane shares are [5][npad])
    int K0, K1, K2;
    int kh;       // K2 / 2 + 1
    int ks;       // row stride of G (complex values): kh rounded up to whole 128-byte lines
    int S;        // line stride of a pair (complex values): 2 kh
    int P;        // row pairs: ceil(K1 / 2)
    int Pc, nyc;  // pairs per row chunk, row chunks
    int Pf, nyf;  // the same of the gradient's interpolation (one line per row)
    int kc, kcs, nkc;  // columns per column chunk (a power of two), its exponent, column chunks
    int kl;       // LDS line stride of a column chunk (kc made odd: whole-line strides put every
                  // point of a transform stage in one LDS bank)
    double klx, kly, klz;
};

// a[t] by selects; the empty asm keeps the compiler from turning the chain back into an
// indexed (scratch-memory) array access
template <typename R> __device__ __forceinline__ R pick5(const R (&a)[5], int t)
{
    R v = a[0];
#pragma unroll
    for (int q = 1; q < 5; ++q) {
        v = t == q ? a[q] : v;
        asm("" : "+v"(v));
    }
    return v;
}

// NR ranges of the (x, y)-binned atom entries; entry i of their concatenation and the x-weight
// index t of its range (selects, so that the arrays stay in registers).
template <int NR> struct BinRanges {
    int lo[NR], pre[NR + 1], tq[NR];
    __device__ __forceinline__ int total() const { return pre[NR]; }
    __device__ __forceinline__ int entry(int i, int& t) const
    {
        t = tq[0];
        int e = lo[0] + i;
#pragma unroll
        for (int q = 1; q < NR; ++q) {
            const bool in = i >= pre[q];
            t = in ? tq[q] : t;
            e = in ? lo[q] + i - pre[q] : e;
        }
        return e;
    }
};

// Row chunk c of the grid: pairs [p0, p0 + np), rows [ya, yb).
struct RowChunk {
    int np, ya, yb;
    __device__ __forceinline__ RowChunk(const PlaneGeom& g, int c, int pairs)
    {
        const int p0 = c * pairs;
        np = min(pairs, g.P - p0);
        ya = 2 * p0;
        yb = min(g.K1, 2 * (p0 + np));
    }
};

// the spline weights of an atom entry (arguments w; second derivatives x2, y2, z2 when SECOND)
// and its z grid lines, doubled for the pair layout
template <typename R, bool SECOND = false>
__device__ __forceinline__ void entry_splines(const typename PlT<R>::R4& w, int fz, int K2, R (&x0)[5], R (&x1)[5],
                                              R (&y0)[5], R (&y1)[5], R (&z0)[5], R (&z1)[5], int (&zi)[5],
                                              R* x2 = nullptr, R* y2 = nullptr, R* z2 = nullptr)
{
    R dum[3][5];
    spline5<R, SECOND>(w.x, x0, x1, SECOND ? x2 : dum[0]);
    spline5<R, SECOND>(w.y, y0, y1, SECOND ? y2 : dum[1]);
    spline5<R, SECOND>(w.z, z0, z1, SECOND ? z2 : dum[2]);
#pragma unroll
    for (int tz = 0; tz < 5; ++tz) {
        int zz = fz - tz;
        zz += zz < 0 ? K2 : 0;
        zi[tz] = 2 * zz;
    }
}

// Last stage of the z transform of nl complex lines in LDS, in place (a butterfly's outputs take
// the places of its points).
template <int SIGN, typename C>
__device__ __forceinline__ void last_stage_rows(C* pl, int nl, int rad, const PlaneGeom& g, const C* tw)
{
    with_radix(rad, [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K2 / RAD;
        const SmallDiv dnb(nb);
        for (int i0 = threadIdx.x; i0 < nl * nb; i0 += blockDim.x) {
            const int i = opaque(i0), lq = dnb.quot(i), j = i - lq * nb;
            C* line = pl + lq * g.S + j;
            C v[RAD];
            rooted_points<RAD, SIGN>(v, tw, j, [&](int r) { return line[r * nb]; });
            dft<RAD, SIGN>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                line[q * nb] = v[q];
        }
    });
}

// Pass 1 (spread, z transform): workgroup (row chunk c, plane x).  The atoms whose support
// meets the chunk's rows of plane x have fx in x..x+4 and fy in [ya, yb + 4) (mod K); they add
// p_x M' M M + p_y M M' M + p_z M M M' (derivatives scaled by K/L) at their in-chunk points,
// or with PERM their permanent multipoles, q M M M + d . grad(M M M) + Theta : grad grad (M M M) / 3
// (src then holds three R4 per atom: (q, d), (Txx, Txy, Txz, Tyy), (Tyz, Tzz, 0, 0)); sstride R4
// from one atom's record to the next.
// Then every row pair is transformed along z, separated into the two rows' half spectra, and
// the rows are written to G[x][y][0, kh).
template <typename R, bool FIX, bool PERM, int NT>
__device__ __forceinline__ void spread_z(double* pl_smem, int item, const PlaneGeom& g, const PlaneDim& dz,
                                         const int* __restrict__ xy_start, const int4* __restrict__ xb_rec,
                                         const typename PlT<R>::R4* __restrict__ xb_w,
                                         const typename PlT<R>::R4* __restrict__ src, int sstride,
                                         const typename PlT<R>::C* __restrict__ roots_z,
                                         typename PlT<R>::C* __restrict__ gout)
{
    using C = typename PlT<R>::C;
    using R4 = typename PlT<R>::R4;
    const int tid = threadIdx.x;
    const int c = item / g.K0, x = item - c * g.K0;
    const RowChunk rc(g, c, g.Pc);
    const int n2 = 2 * rc.np * g.S;                    // doubles of the chunk's accumulation
    double* acc = pl_smem;
    C* tw_z = reinterpret_cast<C*>(pl_smem + 2 * g.Pc * g.S);
    for (int i = tid; i < n2; i += NT)
        acc[i] = 0.0;
    for (int i = tid; i < g.K2; i += NT)
        tw_z[i] = roots_z[i];
    BinRanges<10> br;
    {
        const int L = min(g.K1, rc.yb - rc.ya + 4), f1 = rc.ya + L;
        br.pre[0] = 0;
#pragma unroll
        for (int t = 0; t < 5; ++t) {
            int bx = x + t;
            bx -= bx >= g.K0 ? g.K0 : 0;
            const int* st = xy_start + (size_t)bx * g.K1;
            const int a0 = st[rc.ya], a1 = st[min(f1, g.K1)];
            br.lo[2 * t] = a0;
            br.tq[2 * t] = t;
            br.pre[2 * t + 1] = br.pre[2 * t] + a1 - a0;
            const int b1 = f1 > g.K1 ? st[f1 - g.K1] : st[0];
            br.lo[2 * t + 1] = st[0];
            br.tq[2 * t + 1] = t;
            br.pre[2 * t + 2] = br.pre[2 * t + 1] + b1 - st[0];
        }
    }
    __syncthreads();
    const R klx = (R)g.klx, kly = (R)g.kly, klz = (R)g.klz;
    const int nyr = rc.yb - rc.ya;
    // two atoms per thread and round, their loads issued together
    for (int i0 = tid; i0 < br.total(); i0 += 2 * NT) {
        int tq[2];
        int4 rec[2];
        R4 w[2], m[2][PERM ? 3 : 1];
        bool ok[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int i = i0 + u * NT;
            ok[u] = i < br.total();
            const int e = br.entry(ok[u] ? i : i0, tq[u]);
            rec[u] = xb_rec[e];
            w[u] = xb_w[e];
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int k = 0; k < (PERM ? 3 : 1); ++k)
                m[u][k] = src[sstride * (size_t)rec[u].x + k];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (!ok[u])
                continue;
            const int t = tq[u];
            R x0[5], x1[5], y0[5], y1[5], z0[5], z1[5], x2[5], y2[5], z2[5];
            int zi[5];
            entry_splines<R, PERM>(w[u], rec[u].w, g.K2, x0, x1, y0, y1, z0, z1, zi, x2, y2, z2);
            const R X0 = pick5(x0, t), X1 = pick5(x1, t) * klx;
#pragma unroll
            for (int tz = 0; tz < 5; ++tz) {
                z1[tz] *= klz;
                if (PERM)
                    z2[tz] *= klz * klz;
            }
            // per y weight: c0 (times M_z), c1 (times M'_z), c2 (times M''_z)
            R a0 = 0, a1 = 0, a2 = 0, b0 = 0, b1 = 0, b2 = 0, e0 = 0;
            if (PERM) {
                const R X2 = pick5(x2, t) * klx * klx, third = (R)1 / (R)3;
                const R4 m0 = m[u][0], m1 = m[u][1], m2 = m[u][PERM ? 2 : 0];
                // c0 = a0 y0 + a1 y1 + a2 y2, c1 = b0 y0 + b1 y1, c2 = e0 y0
                a0 = m0.x * X0 + m0.y * X1 + third * m1.x * X2;
                a1 = m0.z * X0 + (R)2 * third * m1.y * X1;
                a2 = third * m1.w * X0;
                b0 = m0.w * X0 + (R)2 * third * m1.z * X1;
                b1 = (R)2 * third * m2.x * X0;
                e0 = third * m2.y * X0;
            } else {
                a0 = m[u][0].x * X1;
                a1 = m[u][0].y * X0;
                b0 = m[u][0].z * X0;
            }
            if (FIX) {
                // every point's value is linear in these: scaled by 2^38 (exactly), the values
                // arrive in the units of the fixed-point sums
                a0 *= (R)kFixQScaleF;
                a1 *= (R)kFixQScaleF;
                a2 *= (R)kFixQScaleF;
                b0 *= (R)kFixQScaleF;
                b1 *= (R)kFixQScaleF;
                e0 *= (R)kFixQScaleF;
            }
#pragma unroll
            for (int ty = 0; ty < 5; ++ty) {
                int yy = rec[u].z - ty;
                yy += yy < 0 ? g.K1 : 0;
                const int yl = yy - rc.ya;
                if (yl < 0 || yl >= nyr)
                    continue;
                const R yw1 = y1[ty] * kly;
                R c0, c1, c2 = 0;
                if (PERM) {
                    const R yw2 = y2[ty] * kly * kly;
                    c0 = a0 * y0[ty] + a1 * yw1 + a2 * yw2;
                    c1 = b0 * y0[ty] + b1 * yw1;
                    c2 = e0 * y0[ty];
                } else {
                    c0 = a0 * y0[ty] + a1 * yw1;
                    c1 = b0 * y0[ty];
                }
                double* row = acc + 2 * (yl >> 1) * g.S + (yl & 1);
#pragma unroll
                for (int tz = 0; tz < 5; ++tz) {
                    R v = c0 * z0[tz] + c1 * z1[tz];
                    if (PERM)
                        v += c2 * z2[tz];
                    if (FIX)
                        atomicAdd(reinterpret_cast<unsigned long long*>(row + zi[tz]), fixq_scaled((float)v));
                    else
                        atomicAdd(row + zi[tz], (double)v);
                }
            }
        }
    }
    __syncthreads();
    // z transform of the row pairs: the first stage reads the sums (fixed point or FP64), the
    // complex lines replace them
    C* pl = reinterpret_cast<C*>(pl_smem);
    with_radix(dz.rad[0], [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K2 / RAD;
        const SmallDiv dnb(nb);
        const int it = opaque(tid), lq = dnb.quot(it), j = it - lq * nb;
        const bool act = it < rc.np * nb;   // the workgroup holds every butterfly of the stage
        C v[RAD];
        if (act) {
            const double2* a = reinterpret_cast<const double2*>(acc) + lq * g.S + j;
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const double2 u = a[r * nb];
                if constexpr (FIX)
                    v[r] = C{(float)fixq_value((unsigned long long)__double_as_longlong(u.x)),
                             (float)fixq_value((unsigned long long)__double_as_longlong(u.y))};
                else
                    v[r] = C{(R)u.x, (R)u.y};
            }
            dft<RAD, -1>(v);
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                pl[lq * g.S + j * RAD + q] = v[q];
        }
    });
    __syncthreads();
    mid_stages<-1>(pl, rc.np, dz, 1, tw_z, LineMap{g.S, 1});
    last_stage_rows<-1>(pl, rc.np, dz.rad[dz.nr - 1], g, tw_z);
    __syncthreads();
    // the two rows of every pair separated into their half spectra: (z + conj zr) / 2 and
    // (z - conj zr) / 2i with zr at K2 - k
    C* out = gout + ((size_t)x * g.K1 + rc.ya) * g.ks;
    const SmallDiv dkh(g.kh);
    for (int i = tid; i < rc.np * g.kh; i += NT) {
        const int p = dkh.quot(i), k = i - p * g.kh;
        const C z = pl[p * g.S + k], zr = pl[p * g.S + (k == 0 ? 0 : g.K2 - k)];
        out[(size_t)(2 * p) * g.ks + k] = C{(R)0.5 * (z.x + zr.x), (R)0.5 * (z.y - zr.y)};
        if (2 * p + 1 < nyr)
            out[(size_t)(2 * p + 1) * g.ks + k] = C{(R)0.5 * (z.y + zr.y), (R)0.5 * (zr.x - z.x)};
    }
}

// What the spread half of a small system's first launch needs (PlanePlan, PlanePasses): its LDS
// bytes, and whether a finished solve ends it.
template <typename R> struct HeadSpread {
    using C = typename PlT<R>::C;
    PlaneGeom g;
    PlaneDim dz;
    const C* roots_z;
    C* gout;
    size_t lds;
    int use_done;
};
template <typename R> void launch_product_head(amoeba_ctx* c, const HeadSpread<R>& s);  // realspace.hip

}  // namespace amoeba
