// Reciprocal dipole field of the smooth PME in five passes over the grid (paper, "Reciprocal
// space scheme": spread of the dipoles with B-spline derivatives, forward FFT, scalar product
// with the influence function, backward FFT, interpolation of the field; Essmann et al. 1995).
//
// The grid is [K0][K1][K2] with z fastest; G is the half-complex grid [K0][K1][K2/2 + 1].
//
//   1 (row chunk, plane x): the atoms whose support meets the chunk's rows of plane x spread
//     into them in LDS; each row is transformed along z (real to half-complex) into G[x][y].
//   2 (plane x, kz chunk):  FFT of the y-lines of G.
//   3 (ky, kz chunk):       FFT of the x-lines, product with the influence function, inverse.
//   4 (plane x, kz chunk):  inverse FFT of the y-lines.
//   5 (row chunk, plane x): the chunk's rows and the four below it are transformed back along
//     z into the potential in LDS; every atom whose top y line lies in the chunk interpolates
//     its share of the field from plane x and writes it to its slot for that plane offset.
//
// A per-atom combine sums the five plane shares in a fixed order (plus, in the PCG product,
// the real-space pieces and the operator assembly).  Every pass has a few hundred small
// workgroups, so all CUs share the work.  There are no grid-size global atomics and no grid
// clearing pass; in mixed precision the spread sums are 64-bit fixed point (exact, so the
// result does not depend on the order of the additions) and every later step is a fixed
// sequence of operations, which makes the reciprocal field bitwise reproducible.
//
// Rows y = 2p and 2p+1 share one complex line (real and imaginary part) of stride
// S = 2 (K2/2 + 1).  A complex FFT of the line along z gives the spectra of both rows,
// separated by X_2p[k] = (Z[k] + conj Z[K2-k]) / 2 and X_2p+1[k] = (Z[k] - conj Z[K2-k]) / 2i;
// the inverse runs the same steps backwards.  The one-dimensional transforms (plane_fft.h) take
// their first points straight from global memory (or from the spread's sums) and cross LDS once
// where the length is a product of two supported radices; the roots of unity are in LDS (computed
// in FP64).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "plane_fft.h"
#include "plane_spread.h"
#include "reduce.h"
#include "spline.h"

namespace amoeba {

template <typename R, bool FIX, bool PERM, int NT>
__global__ __launch_bounds__(NT) void k_pme_spread_z(PlaneGeom g, PlaneDim dz, const int* __restrict__ xy_start,
                                                     const int4* __restrict__ xb_rec,
                                                     const typename PlT<R>::R4* __restrict__ xb_w,
                                                     const typename PlT<R>::R4* __restrict__ src, int sstride,
                                                     const typename PlT<R>::C* __restrict__ roots_z,
                                                     typename PlT<R>::C* __restrict__ gout,
                                                     const PcgScalars* __restrict__ sc, int use_done)
{
    extern __shared__ __align__(16) double pl_smem[];
    if (use_done && sc->done)
        return;
    spread_z<R, FIX, PERM, NT>(pl_smem, xcd_remap(blockIdx.x, gridDim.x), g, dz, xy_start, xb_rec, xb_w, src, sstride,
                               roots_z, gout);
}

// First and last stage of a column pass: thread (column col, butterfly j), the workgroup holding
// every butterfly.  The first reads the butterfly's points from src (point stride ss) and leaves
// its outputs in LDS; the last takes them from LDS to dst.  Offsets from the two bases stay below
// 2^32 bytes (a column pass spans one grid), which leaves one address register per access.
template <typename C> __device__ __forceinline__ C load_at(const C* base, unsigned byte_off)
{
    return *reinterpret_cast<const C*>(reinterpret_cast<const char*>(base) + byte_off);
}
template <typename C> __device__ __forceinline__ void store_at(C* base, unsigned byte_off, C v)
{
    *reinterpret_cast<C*>(reinterpret_cast<char*>(base) + byte_off) = v;
}

template <int SIGN, typename C>
__device__ __forceinline__ void first_stage_cols(const C* __restrict__ src, unsigned ss, C* buf, int rad,
                                                 const PlaneGeom& g, int N)
{
    with_radix(rad, [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = N / RAD, tid = opaque(threadIdx.x), col = tid & (g.kc - 1);
        const int j = tid >> g.kcs;
        if (j < nb) {
            const unsigned off = (j * ss + col) * sizeof(C), step = nb * ss * sizeof(C);
            C v[RAD];
#pragma unroll
            for (int r = 0; r < RAD; ++r)
                v[r] = load_at(src, off + r * step);
            dft<RAD, SIGN>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                buf[(j * RAD + q) * g.kl + col] = v[q];
        }
    });
}

template <int SIGN, typename C>
__device__ __forceinline__ void last_stage_cols(const C* buf, C* __restrict__ dst, unsigned ds, int rad,
                                                const PlaneGeom& g, int N, const C* tw)
{
    with_radix(rad, [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = N / RAD, tid = opaque(threadIdx.x), col = tid & (g.kc - 1);
        const int j = tid >> g.kcs;
        if (j < nb) {
            C v[RAD];
            const C* pt = buf + j * g.kl + col;
            rooted_points<RAD, SIGN>(v, tw, j, [&](int r) { return pt[r * nb * g.kl]; });
            dft<RAD, SIGN>(v);
            const unsigned off = (j * ds + col) * sizeof(C), step = nb * ds * sizeof(C);
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                store_at(dst, off + q * step, v[q]);
        }
    });
}

// The real-space reduction of a product, taken by the workgroups of a transform launch beyond its
// own (small systems).
template <typename R> struct RealReduceArgs {
    int npad;  // 0: none
    const double* eipart;
    const R* jbuf;
    const int *rev_ptr, *rev_idx;
    double* ereal;
    __device__ __forceinline__ void run(int wg) const
    {
        const int t = wg * blockDim.x + threadIdx.x;
        if (t < 4 * npad)
            real_reduce<R>(t, eipart, jbuf, rev_ptr, rev_idx, ereal);
    }
};

// Passes 2 and 4 (y transform, SIGN -1 forward, +1 inverse): workgroup (plane x, column chunk):
// the y-lines G[x][.][kz] for kz in the chunk, in place.  A chunk is one 128-byte line of columns
// (the padding columns of a row are transformed along; nothing reads them).  The y index of the
// launch selects the grid (the gradient transforms two at once).
// Bound by the grid's bytes through the caches: 42 MB in and out at 216^3 in FP32.  The stages that
// all went through LDS (a fill, three stages and a store) took y + x + y 128 us there, 255 us in
// FP64, and 69 / 91 us at 144^3; with the first and last stage in registers they take 71 and 122 us,
// and 43 / 51 us.
template <typename R, int SIGN>
__global__ __launch_bounds__(kPlColThreads) void k_pme_ylines(PlaneGeom g, PlaneDim dy,
                                                           typename PlT<R>::C* __restrict__ gc,
                                                           typename PlT<R>::C* __restrict__ gc1,
                                                           const typename PlT<R>::C* __restrict__ roots_y,
                                                           RealReduceArgs<R> rr,
                                                           const PcgScalars* __restrict__ sc, int use_done)
{
    __builtin_amdgcn_s_setprio(kPlPassPrio);
    using C = typename PlT<R>::C;
    extern __shared__ __align__(16) double pl_smem[];
    if (use_done && sc->done)
        return;
    const int item = blockIdx.x;
    if (item >= g.K0 * g.nkc) {
        rr.run(item - g.K0 * g.nkc);
        return;
    }
    const int x = item / g.nkc, kz0 = (item - x * g.nkc) * g.kc;
    C* buf = reinterpret_cast<C*>(pl_smem);
    C* tw = buf + g.K1 * g.kl;
    C* base = (blockIdx.y ? gc1 : gc) + (size_t)x * g.K1 * g.ks + kz0;
    first_stage_cols<SIGN>(base, (unsigned)g.ks, buf, dy.rad[0], g, g.K1);
    for (int i = threadIdx.x; i < g.K1; i += blockDim.x)
        tw[i] = roots_y[i];
    __syncthreads();
    mid_stages<SIGN>(buf, g.kc, dy, 1, tw, LineMap{1, g.kl});
    last_stage_cols<SIGN>(buf, base, (unsigned)g.ks, dy.rad[dy.nr - 1], g, g.K1, tw);
}

// Pass 3: workgroup (ky, column chunk): the x-lines of G for kz in the chunk: FFT, product with
// the influence function theta (column-chunk layout), inverse FFT, in place.  The last stage of
// the forward transform leaves X[j + q nb] in the thread of butterfly j, which is what the first
// stage of the inverse with the same radix takes there, so the product is made in registers.
template <typename R>
__global__ __launch_bounds__(kPlColThreads) void k_pme_xconv(PlaneGeom g, PlaneDim dx,
                                                          typename PlT<R>::C* __restrict__ gc,
                                                          typename PlT<R>::C* __restrict__ gc1,
                                                          const R* __restrict__ theta,
                                                          const typename PlT<R>::C* __restrict__ roots_x,
                                                          const PcgScalars* __restrict__ sc, int use_done)
{
    __builtin_amdgcn_s_setprio(kPlPassPrio);
    using C = typename PlT<R>::C;
    extern __shared__ __align__(16) double pl_smem[];
    if (use_done && sc->done)
        return;
    const int item = blockIdx.x;
    const int ky = item / g.nkc, kz0 = (item - ky * g.nkc) * g.kc;
    C* buf = reinterpret_cast<C*>(pl_smem);
    C* tw = buf + g.K0 * g.kl;
    const unsigned xs = (unsigned)(g.K1 * g.ks);   // stride of x in G
    C* base = (blockIdx.y ? gc1 : gc) + (size_t)ky * g.ks + kz0;
    first_stage_cols<-1>(base, xs, buf, dx.rad[0], g, g.K0);
    for (int i = threadIdx.x; i < g.K0; i += blockDim.x)
        tw[i] = roots_x[i];
    __syncthreads();
    const LineMap am{1, g.kl};
    mid_stages<-1>(buf, g.kc, dx, 1, tw, am);
    const R* th = theta + (size_t)item * g.K0 * g.kc;
    with_radix(dx.rad[dx.nr - 1], [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K0 / RAD, tid = opaque(threadIdx.x), col = tid & (g.kc - 1), j = tid >> g.kcs;
        C v[RAD];
        if (j < nb) {   // the workgroup holds every butterfly of the stage
            R f[RAD];
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                f[q] = th[(j + q * nb) * g.kc + col];
            const C* pt = buf + j * g.kl + col;
            rooted_points<RAD, -1>(v, tw, j, [&](int r) { return pt[r * nb * g.kl]; });
            dft<RAD, -1>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q) {
                v[q].x *= f[q];
                v[q].y *= f[q];
            }
            dft<RAD, +1>(v);
        }
        __syncthreads();
        if (j < nb) {
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                buf[(j * RAD + q) * g.kl + col] = v[q];
        }
    });
    __syncthreads();
    mid_stages<+1>(buf, g.kc, dx, -1, tw, am);
    last_stage_cols<+1>(buf, base, xs, dx.rad[0], g, g.K0, tw);
}

// Passes 2 to 4 in one launch for a small grid: workgroup kz (and grid, the y index of the launch)
// holds that column's K0 x K1 points in LDS, one butterfly per thread in every stage.  A stage whose
// outputs take other places than its points has a barrier between its reads and its writes; the
// last stage of a transform replaces its own points.
template <int SIGN, bool LAST, int W, typename C, typename IN, typename OUT>
__device__ __forceinline__ void yxy_stage(int rad, int N, int nl, const C* tw, IN in, OUT out)
{
    // LAST: roots on the way in, outputs to j + q N/RAD; else outputs to j RAD + q.  Thread index:
    // W = 0 butterflies fastest (lines are rows of the plane), 1 lines fastest (columns).
    with_radix(rad, [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = N / RAD, it = opaque(threadIdx.x);
        const SmallDiv dv(W == 0 ? nb : nl);
        const int hi = dv.quot(it), lo = it - hi * (W == 0 ? nb : nl);
        const int l = W == 0 ? hi : lo, j = W == 0 ? lo : hi;
        const bool act = it < nl * nb;
        C v[RAD];
        if (act) {
            if constexpr (LAST) {
                rooted_points<RAD, SIGN>(v, tw, j, [&](int r) { return in(l, j + r * nb); });
            } else {
#pragma unroll
                for (int r = 0; r < RAD; ++r)
                    v[r] = in(l, j + r * nb);
            }
            dft<RAD, SIGN>(v);
        }
        if constexpr (!LAST)
            __syncthreads();
        if (act) {
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                out(l, LAST ? j + q * nb : j * RAD + q, v[q]);
        }
    });
    __syncthreads();
}

template <typename R>
__global__ __launch_bounds__(kPlYxyThreads) void k_pme_yxy(PlaneGeom g, PlaneDim dy, PlaneDim dx,
                                                  typename PlT<R>::C* __restrict__ gc,
                                                  typename PlT<R>::C* __restrict__ gc1,
                                                  const R* __restrict__ theta,
                                                  const typename PlT<R>::C* __restrict__ roots_y,
                                                  const typename PlT<R>::C* __restrict__ roots_x,
                                                  RealReduceArgs<R> rr,
                                                  const PcgScalars* __restrict__ sc, int use_done)
{
    using C = typename PlT<R>::C;
    extern __shared__ __align__(16) double pl_smem[];
    if (use_done && sc->done)
        return;
    const int kz = blockIdx.x, tid = threadIdx.x;
    if (kz >= g.kh) {
        rr.run(kz - g.kh);
        return;
    }
    C* base = (blockIdx.y ? gc1 : gc) + kz;
    C* buf = reinterpret_cast<C*>(pl_smem);
    const int lp = g.K1 | 1;
    C* tw_y = buf + g.K0 * lp;
    C* tw_x = tw_y + g.K1;
    auto mem = [&](int x, int y) -> C& { return buf[x * lp + y]; };
    auto at = [&](int x, int y) { return mem(x, y); };
    auto to = [&](int x, int y, C v) { mem(x, y) = v; };
    auto at_t = [&](int y, int x) { return mem(x, y); };
    auto to_t = [&](int y, int x, C v) { mem(x, y) = v; };
    auto global = [&](int x, int y) { return (unsigned)((x * g.K1 + y) * g.ks) * (unsigned)sizeof(C); };
    for (int i = tid; i < g.K1 + g.K0; i += blockDim.x)
        tw_y[i] = i < g.K1 ? roots_y[i] : roots_x[i - g.K1];
    // y forward, from the grid
    yxy_stage<-1, false, 0>(dy.rad[0], g.K1, g.K0, tw_y, [&](int x, int y) { return load_at(base, global(x, y)); }, to);
    yxy_stage<-1, true, 0>(dy.rad[1], g.K1, g.K0, tw_y, at, to);
    // x forward, the influence function and the first stage back in registers (as in k_pme_xconv)
    yxy_stage<-1, false, 1>(dx.rad[0], g.K0, g.K1, tw_x, at_t, to_t);
    const R* th = theta + (size_t)(kz >> g.kcs) * g.K0 * g.kc + (kz & (g.kc - 1));
    const unsigned ths = (unsigned)(g.nkc * g.K0 * g.kc);
    with_radix(dx.rad[1], [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K0 / RAD, it = opaque(tid);
        const SmallDiv dv(g.K1);
        const int j = dv.quot(it), y = it - j * g.K1;
        const bool act = it < g.K1 * nb;
        C v[RAD];
        if (act) {
            R f[RAD];
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                f[q] = th[y * ths + (j + q * nb) * g.kc];
            rooted_points<RAD, -1>(v, tw_x, j, [&](int r) { return mem(j + r * nb, y); });
            dft<RAD, -1>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q) {
                v[q].x *= f[q];
                v[q].y *= f[q];
            }
            dft<RAD, +1>(v);
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                mem(j * RAD + q, y) = v[q];
        }
    });
    __syncthreads();
    yxy_stage<+1, true, 1>(dx.rad[0], g.K0, g.K1, tw_x, at_t, to_t);
    // y back, to the grid
    yxy_stage<+1, false, 0>(dy.rad[1], g.K1, g.K0, tw_y, at, to);
    yxy_stage<+1, true, 0>(dy.rad[0], g.K1, g.K0, tw_y, at,
                           [&](int x, int y, C v) { store_at(base, global(x, y), v); });
}

// Pass 5 (z transform back, interpolation): workgroup (row chunk c, plane x).  The potential
// rows [ya - 4, yb) (mod K1) are rebuilt from their half spectra (two rows per complex line:
// Z[k] = A[k] + i B[k] with the Hermitian extension A[k] = conj A[K2 - k] for k >= kh, the
// imaginary parts of the real terms k = 0 and K2/2 dropped as a real inverse transform does)
// and transformed back along z; then every atom with fx in x..x+4 and fy in [ya, yb) adds up its
// share of the field from plane x: part[t npad + s] = (M'_x M_y M_z psi, M_x M'_y M_z psi,
// M_x M_y M'_z psi) over its 25 (y, z) points, t its weight index for the plane (the K/L
// factors and the sign are applied by the combine).
template <typename R, int NT>
__global__ __launch_bounds__(NT, sizeof(R) == 8 ? 4 : 1) void k_pme_z_gather(PlaneGeom g, PlaneDim dz,
                                                             const typename PlT<R>::C* __restrict__ gc,
                                                             const int* __restrict__ xy_start,
                                                             const int4* __restrict__ xb_rec,
                                                             const typename PlT<R>::R4* __restrict__ xb_w,
                                                             const typename PlT<R>::C* __restrict__ roots_z,
                                                             typename PlT<R>::R4* __restrict__ part,
                                                             const PcgScalars* __restrict__ sc, int use_done)
{
    __builtin_amdgcn_s_setprio(kPlPassPrio);
    using C = typename PlT<R>::C;
    using R4 = typename PlT<R>::R4;
    extern __shared__ __align__(16) double pl_smem[];
    if (use_done && sc->done)
        return;
    const int tid = threadIdx.x;
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const int c = item / g.K0, x = item - c * g.K0;
    const RowChunk rc(g, c, g.Pc);
    const int nrows = rc.yb - rc.ya + 4, npl = (nrows + 1) / 2;
    C* pl = reinterpret_cast<C*>(pl_smem);
    C* tw_z = pl + (g.Pc + 2) * g.S;
    for (int i = tid; i < g.K2; i += NT)
        tw_z[i] = roots_z[i];
    // the first stage of the inverse along z reads the half spectra and forms the complex lines
    with_radix(dz.rad[dz.nr - 1], [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K2 / RAD;
        const SmallDiv dnb(nb);
        for (int i0 = tid; i0 < npl * nb; i0 += NT) {
            const int i = opaque(i0), lq = dnb.quot(i), j = i - lq * nb;
            int gy0 = rc.ya - 4 + 2 * lq, gy1 = gy0 + 1;
            gy0 += gy0 < 0 ? g.K1 : 0;
            gy1 += gy1 < 0 ? g.K1 : 0;
            const bool two = 2 * lq + 1 < nrows;  // the last line may hold one row only
            const C* ra = gc + ((size_t)x * g.K1 + gy0) * g.ks;
            const C* rb = gc + ((size_t)x * g.K1 + (two ? gy1 : gy0)) * g.ks;
            C v[RAD];
#pragma unroll
            for (int r = 0; r < RAD; ++r) {
                const int k = j + r * nb;
                const bool up = k >= g.kh;
                const int kk = up ? g.K2 - k : k;
                C a = ra[kk], b = rb[kk];
                if (!two)
                    b.x = b.y = (R)0;
                if (kk == 0 || 2 * kk == g.K2)
                    a.y = b.y = (R)0;
                if (up) {
                    a.y = -a.y;
                    b.y = -b.y;
                }
                v[r] = C{a.x - b.y, a.y + b.x};
                if (sizeof(R) == 8 && r % kRootGroup == kRootGroup - 1)
                    __builtin_amdgcn_sched_barrier(0);  // as in rooted_points: bounds the registers
            }
            dft<RAD, +1>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                pl[lq * g.S + j * RAD + q] = v[q];
        }
    });
    __syncthreads();
    mid_stages<+1>(pl, npl, dz, -1, tw_z, LineMap{g.S, 1});
    last_stage_rows<+1>(pl, npl, dz.rad[0], g, tw_z);
    __syncthreads();
    // potential of local row r (global row ya - 4 + r), point z: component r mod 2 of
    // pl[(r div 2) S + z]
    const R* psi = reinterpret_cast<const R*>(pl_smem);
    BinRanges<5> br;
    br.pre[0] = 0;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        int bx = x + t;
        bx -= bx >= g.K0 ? g.K0 : 0;
        const int* st = xy_start + (size_t)bx * g.K1;
        br.lo[t] = st[rc.ya];
        br.tq[t] = t;
        br.pre[t + 1] = br.pre[t] + st[rc.yb] - br.lo[t];
    }
    const int yorg = rc.ya - 4;
    // two atoms per thread and round, their loads issued together
    for (int i0 = tid; i0 < br.total(); i0 += 2 * NT) {
        int tq[2];
        int4 rec[2];
        R4 w[2];
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
        for (int u = 0; u < 2; ++u) {
            if (!ok[u])
                continue;
            R x0[5], x1[5], y0[5], y1[5], z0[5], z1[5];
            int zi[5];
            entry_splines<R>(w[u], rec[u].w, g.K2, x0, x1, y0, y1, z0, z1, zi);
            R ax = 0, ay = 0, az = 0;
#pragma unroll
            for (int ty = 0; ty < 5; ++ty) {
                const int r = rec[u].z - ty - yorg;   // in [0, nrows): fy lies in [ya, yb)
                const R* row = psi + 2 * (r >> 1) * g.S + (r & 1);
                R s0 = 0, s1 = 0;
#pragma unroll
                for (int tz = 0; tz < 5; ++tz) {
                    const R v = row[zi[tz]];
                    s0 += z0[tz] * v;
                    s1 += z1[tz] * v;
                }
                ax += y0[ty] * s0;
                ay += y1[ty] * s0;
                az += y0[ty] * s1;
            }
            const R tx0 = pick5(x0, tq[u]), tx1 = pick5(x1, tq[u]);
            part[(size_t)tq[u] * g.npad + rec[u].x] = R4{tx1 * ax, tx0 * ay, tx0 * az, (R)0};
        }
    }
}

// Weights of the gradient's interpolation: B-spline values and derivatives up to the third, the
// k-th times scale^k (polynomial pieces as in spline5; the third derivatives are linear).
__device__ __forceinline__ void spline5_third(double w, double scale, double (&m0)[5], double (&m1)[5],
                                              double (&m2)[5], double (&m3)[5])
{
    spline5<double, true>(w, m0, m1, m2);
    const double v = 1.0 - w;
    m3[0] = w;
    m3[1] = 1.0 - 4.0 * w;
    m3[2] = 6.0 * w - 3.0;
    m3[3] = 4.0 * v - 1.0;
    m3[4] = -v;
    const double s2 = scale * scale;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        m1[t] *= scale;
        m2[t] *= s2;
        m3[t] *= s2 * scale;
    }
}

// Pass 5 of the polarization gradient: workgroup (row chunk c, plane x) of two transformed grids,
// the potentials psi_p of the multipoles (gp) and psi_m of the dipoles (gm).  Each row is one
// complex line, psi_p in the real and psi_m in the imaginary part, so that a point's two
// potentials are one LDS read.  Then every atom with fx in x..x+4 and fy in [ya, yb) adds up its
// share from plane x of
//   sum_k psi_a(k) (H mu) + psi_m(k) (q grad W + H d + 1/3 sum_bc Theta_bc d_a d_b d_c W),
//   H_ab = d_a d_b W, psi_a = psi_m + psi_p,
// in FP64 (weights, sums and the contraction with the multipoles), into part[t npad + s].
// Bound by FP64 issue (about 550 instructions per atom and plane) beside the two grids' bytes: 79 us
// at 288,000 atoms beside the pair tiles, 16 us at 23,559 atoms in FP64.
template <typename R, int NT>
__global__ __launch_bounds__(NT) void k_pme_z_force(PlaneGeom g, PlaneDim dz,
                                                    const typename PlT<R>::C* __restrict__ gp,
                                                    const typename PlT<R>::C* __restrict__ gm,
                                                    const int* __restrict__ xy_start,
                                                    const int4* __restrict__ xb_rec,
                                                    const double4* __restrict__ pos_s,
                                                    const typename PlT<R>::C* __restrict__ roots_z,
                                                    const double4* __restrict__ mp, const double* __restrict__ mu,
                                                    double4* __restrict__ part)
{
    using C = typename PlT<R>::C;
    extern __shared__ __align__(16) double pl_smem[];
    const int tid = threadIdx.x;
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    const int c = item / g.K0, x = item - c * g.K0;
    const RowChunk rc(g, c, g.Pf);
    const int nrows = rc.yb - rc.ya + 4;
    C* pl = reinterpret_cast<C*>(pl_smem);
    C* tw_z = pl + (2 * g.Pf + 4) * g.S;
    for (int i = tid; i < g.K2; i += NT)
        tw_z[i] = roots_z[i];
    with_radix(dz.rad[dz.nr - 1], [&](auto rc_) {
        constexpr int RAD = decltype(rc_)::value;
        const int nb = g.K2 / RAD;
        const SmallDiv dnb(nb);
        for (int i0 = tid; i0 < nrows * nb; i0 += NT) {
            const int i = opaque(i0), r = dnb.quot(i), j = i - r * nb;
            int gy = rc.ya - 4 + r;
            gy += gy < 0 ? g.K1 : 0;
            const size_t row = ((size_t)x * g.K1 + gy) * g.ks;
            C v[RAD];
#pragma unroll
            for (int q = 0; q < RAD; ++q) {
                const int k = j + q * nb;
                const bool up = k >= g.kh;
                const int kk = up ? g.K2 - k : k;
                C a = gp[row + kk], b = gm[row + kk];
                if (kk == 0 || 2 * kk == g.K2)
                    a.y = b.y = (R)0;
                if (up) {
                    a.y = -a.y;
                    b.y = -b.y;
                }
                v[q] = C{a.x - b.y, a.y + b.x};
                if (q % kRootGroup == kRootGroup - 1)
                    __builtin_amdgcn_sched_barrier(0);  // as in rooted_points: bounds the registers
            }
            dft<RAD, +1>(v);
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                pl[r * g.S + j * RAD + q] = v[q];
        }
    });
    __syncthreads();
    mid_stages<+1>(pl, nrows, dz, -1, tw_z, LineMap{g.S, 1});
    last_stage_rows<+1>(pl, nrows, dz.rad[0], g, tw_z);
    __syncthreads();
    BinRanges<5> br;
    br.pre[0] = 0;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        int bx = x + t;
        bx -= bx >= g.K0 ? g.K0 : 0;
        const int* st = xy_start + (size_t)bx * g.K1;
        br.lo[t] = st[rc.ya];
        br.tq[t] = t;
        br.pre[t + 1] = br.pre[t] + st[rc.yb] - br.lo[t];
    }
    const int yorg = rc.ya - 4;
    for (int i = tid; i < br.total(); i += NT) {
        int t;
        const int e = br.entry(i, t);
        const int4 rec = xb_rec[e];
        const int s = rec.x;
        const double4 p = pos_s[s];
        double y0[5], y1[5], y2[5], y3[5], z0[5], z1[5], z2[5], z3[5];
        int f;
        double w;
        grid_coord(p.z, g.klz, g.K2, f, w);
        spline5_third(w, g.klz, z0, z1, z2, z3);
        grid_coord(p.y, g.kly, g.K1, f, w);
        spline5_third(w, g.kly, y0, y1, y2, y3);
        int zi[5];
#pragma unroll
        for (int tz = 0; tz < 5; ++tz) {
            zi[tz] = rec.w - tz;
            zi[tz] += zi[tz] < 0 ? g.K2 : 0;
        }
        // plane sums: a_bc (psi_a, b + c <= 2), m_bc (psi_m, b + c <= 3) with b y- and c z-derivatives
        double a00 = 0, a01 = 0, a02 = 0, a10 = 0, a11 = 0, a20 = 0;
        double m00 = 0, m01 = 0, m02 = 0, m03 = 0, m10 = 0, m11 = 0, m12 = 0, m20 = 0, m21 = 0, m30 = 0;
#pragma unroll
        for (int ty = 0; ty < 5; ++ty) {
            const C* row = pl + (rec.z - ty - yorg) * g.S;   // rows in [0, nrows): fy lies in [ya, yb)
            double sa0 = 0, sa1 = 0, sa2 = 0, sm0 = 0, sm1 = 0, sm2 = 0, sm3 = 0;
#pragma unroll
            for (int tz = 0; tz < 5; ++tz) {
                const C u = row[zi[tz]];
                const double pm = (double)u.y, pa = (double)u.x + pm;
                sa0 = fma(z0[tz], pa, sa0);
                sa1 = fma(z1[tz], pa, sa1);
                sa2 = fma(z2[tz], pa, sa2);
                sm0 = fma(z0[tz], pm, sm0);
                sm1 = fma(z1[tz], pm, sm1);
                sm2 = fma(z2[tz], pm, sm2);
                sm3 = fma(z3[tz], pm, sm3);
            }
            a00 = fma(y0[ty], sa0, a00);
            a01 = fma(y0[ty], sa1, a01);
            a02 = fma(y0[ty], sa2, a02);
            a10 = fma(y1[ty], sa0, a10);
            a11 = fma(y1[ty], sa1, a11);
            a20 = fma(y2[ty], sa0, a20);
            m00 = fma(y0[ty], sm0, m00);
            m01 = fma(y0[ty], sm1, m01);
            m02 = fma(y0[ty], sm2, m02);
            m03 = fma(y0[ty], sm3, m03);
            m10 = fma(y1[ty], sm0, m10);
            m11 = fma(y1[ty], sm1, m11);
            m12 = fma(y1[ty], sm2, m12);
            m20 = fma(y2[ty], sm0, m20);
            m21 = fma(y2[ty], sm1, m21);
            m30 = fma(y3[ty], sm0, m30);
        }
        double X0, X1, X2, X3;
        {
            double x0[5], x1[5], x2[5], x3[5];
            grid_coord(p.x, g.klx, g.K0, f, w);
            spline5_third(w, g.klx, x0, x1, x2, x3);
            X0 = pick5(x0, t);
            X1 = pick5(x1, t);
            X2 = pick5(x2, t);
            X3 = pick5(x3, t);
        }
        const double ux = mu[3 * (size_t)s], uy = mu[3 * (size_t)s + 1], uz = mu[3 * (size_t)s + 2];
        const double4 q0 = mp[3 * (size_t)s], q1 = mp[3 * (size_t)s + 1], q2 = mp[3 * (size_t)s + 2];
        const double q = q0.x, dx = q0.y, dy = q0.z, dz_ = q0.w;
        const double third = 1.0 / 3.0;
        const double txx = third * q1.x, txy = 2.0 * third * q1.y, txz = 2.0 * third * q1.z, tyy = third * q1.w,
                     tyz = 2.0 * third * q2.x, tzz = third * q2.y;
        // second derivatives of psi_a and of psi_m on this plane
        const double hxx = X2 * a00, hxy = X1 * a10, hxz = X1 * a01, hyy = X0 * a20, hyz = X0 * a11, hzz = X0 * a02;
        const double kxx = X2 * m00, kxy = X1 * m10, kxz = X1 * m01, kyy = X0 * m20, kyz = X0 * m11, kzz = X0 * m02;
        double4 o;
        o.x = hxx * ux + hxy * uy + hxz * uz + q * X1 * m00 + kxx * dx + kxy * dy + kxz * dz_ + txx * X3 * m00 +
              X2 * (txy * m10 + txz * m01) + X1 * (tyy * m20 + tyz * m11 + tzz * m02);
        o.y = hxy * ux + hyy * uy + hyz * uz + q * X0 * m10 + kxy * dx + kyy * dy + kyz * dz_ + txx * X2 * m10 +
              X1 * (txy * m20 + txz * m11) + X0 * (tyy * m30 + tyz * m21 + tzz * m12);
        o.z = hxz * ux + hyz * uy + hzz * uz + q * X0 * m01 + kxz * dx + kyz * dy + kzz * dz_ + txx * X2 * m01 +
              X1 * (txy * m11 + txz * m02) + X0 * (tyy * m21 + tyz * m12 + tzz * m03);
        o.w = 0.0;
        part[(size_t)t * g.npad + s] = o;
    }
}

// Per-atom combine of the plane shares: E_rec = -(K/L) sum_t part[t npad + s] (fixed order).
// MODE 0 writes E_rec (slot order, FP64).  MODE 1 assembles the PCG operator product
// q = p / alpha - (E_real + E_rec + self p): the real-space field is the atom's block i-field
// plus the tile j-fields listed in the reverse index, in index order (or, MODE 2, the same sum
// already in ereal); optionally the workgroup's p.q partial.
template <typename R, int MODE>
__global__ __launch_bounds__(256) void k_plane_combine(int npad, double3 kl, const int* __restrict__ perm,
                                                       const typename PlT<R>::R4* __restrict__ part,
                                                       const double* __restrict__ alpha_inv,
                                                       const double* __restrict__ p, double self,
                                                       const double* __restrict__ eipart,
                                                       const typename PlT<R>::R4* __restrict__ jbuf,
                                                       const int* __restrict__ rev_ptr,
                                                       const int* __restrict__ rev_idx,
                                                       const double* __restrict__ ereal, double* __restrict__ out,
                                                       const PcgScalars* __restrict__ sc,
                                                       double* __restrict__ pq_part, int use_done, int dot)
{
    using R4 = typename PlT<R>::R4;
    if (use_done && sc->done)
        return;
    const int s = blockIdx.x * 256 + threadIdx.x;
    double pq[1] = {0.0};
    if (s < npad) {
        double e[3] = {0.0, 0.0, 0.0};
        if (perm[s] >= 0) {
            double sx = 0.0, sy = 0.0, sz = 0.0;
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                const R4 v = part[(size_t)t * npad + s];
                sx += (double)v.x;
                sy += (double)v.y;
                sz += (double)v.z;
            }
            e[0] = -sx * kl.x;
            e[1] = -sy * kl.y;
            e[2] = -sz * kl.z;
        }
        if (MODE == 0) {
            for (int a = 0; a < 3; ++a)
                out[3 * (size_t)s + a] = e[a];
        } else if (perm[s] >= 0 && MODE == 2) {
            const double ainv = alpha_inv[s];
            for (int a = 0; a < 3; ++a) {
                const size_t i = 3 * (size_t)s + a;
                const double pa = p[i];
                const double qa = pa * ainv - (ereal[i] + e[a] + self * pa);
                out[i] = qa;
                pq[0] += pa * qa;
            }
        } else if (perm[s] >= 0) {
            using J = JSum<R>;
            double er[3] = {J::start(eipart[3 * (size_t)s]), J::start(eipart[3 * (size_t)s + 1]),
                            J::start(eipart[3 * (size_t)s + 2])};
            const int k1 = rev_ptr[s + 1];
            int k = rev_ptr[s];
            // four independent loads in flight
            for (; k + 4 <= k1; k += 4) {
                R4 j[4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    j[u] = jbuf[rev_idx[k + u]];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    er[0] += J::term(j[u].x);
                    er[1] += J::term(j[u].y);
                    er[2] += J::term(j[u].z);
                }
            }
            for (; k < k1; ++k) {
                const R4 j = jbuf[rev_idx[k]];
                er[0] += J::term(j.x);
                er[1] += J::term(j.y);
                er[2] += J::term(j.z);
            }
            for (int a = 0; a < 3; ++a)
                er[a] = J::finish(er[a]);
            const double ainv = alpha_inv[s];
            for (int a = 0; a < 3; ++a) {
                const size_t i = 3 * (size_t)s + a;
                const double pa = p[i];
                const double qa = pa * ainv - (er[a] + e[a] + self * pa);
                out[i] = qa;
                pq[0] += pa * qa;
            }
        } else {
            for (int a = 0; a < 3; ++a)
                out[3 * (size_t)s + a] = 0.0;
        }
    }
    if (MODE == 0 || !dot)
        return;
    block_sum<1>(pq);
    if (threadIdx.x == 0)
        pq_part[blockIdx.x] = pq[0];
}

// ------------------------------------------------------------------------------------------
// per configuration: atoms binned by the (x, y) lines of their base point, with their spline
// arguments; the order inside a bin is arbitrary (no result depends on it)
// ------------------------------------------------------------------------------------------
__global__ void k_xybin_count(int npad, const int* __restrict__ perm, const double4* __restrict__ pos_s, double3 kl,
                              int3 K, int* __restrict__ count)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad || perm[s] < 0)
        return;
    const double4 p = pos_s[s];
    int fx, fy;
    double u;
    grid_coord(p.x, kl.x, K.x, fx, u);
    grid_coord(p.y, kl.y, K.y, fy, u);
    atomicAdd(&count[fx * K.y + fy], 1);
}

template <typename R>
__global__ void k_xybin_fill(int npad, const int* __restrict__ perm, const double4* __restrict__ pos_s, double3 kl,
                             int3 K, const int* __restrict__ start, int* __restrict__ cursor,
                             int4* __restrict__ rec, typename PlT<R>::R4* __restrict__ wout)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad || perm[s] < 0)
        return;
    const double4 p = pos_s[s];
    int f[3];
    double u[3];
    grid_coord(p.x, kl.x, K.x, f[0], u[0]);
    grid_coord(p.y, kl.y, K.y, f[1], u[1]);
    grid_coord(p.z, kl.z, K.z, f[2], u[2]);
    const int b = f[0] * K.y + f[1];
    // the cursor starts at the bin's count and counts down to zero, which leaves the counters
    // cleared for the next binning
    const int e = start[b] + atomicSub(&cursor[b], 1) - 1;
    rec[e] = make_int4(s, f[0], f[1], f[2]);
    wout[e] = typename PlT<R>::R4{(R)u[0], (R)u[1], (R)u[2], (R)0};
}

template <typename R>
__global__ void k_plane_roots(int n, typename PlT<R>::C* __restrict__ out)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n)
        return;
    double s, c;
    sincospi(-2.0 * (double)k / (double)n, &s, &c);
    out[k] = typename PlT<R>::C{(R)c, (R)s};
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static inline int nblk(size_t n, int b) { return (int)((n + b - 1) / b); }
static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

static int min_radix(const PlaneDim& d) { return *std::min_element(d.rad, d.rad + d.nr); }

// The radices of length n: as few as possible (at least two), and of those the split whose
// smallest radix is largest (the fewest butterflies, so the fewest threads, in a stage); the two
// largest at the ends, the others (at most 9) between them.  Returns false where a prime factor
// above 7 is left or a stage would need more than 256 butterflies.
static bool plane_factor(int n, PlaneDim& d)
{
    static const int radices[] = {18, 16, 15, 14, 12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
    d.n = n;
    d.nr = 0;
    for (int nr = 2; nr <= 8 && d.nr == 0; ++nr) {
        int cur[8], best = 0;
        auto split = [&](auto&& self, int left, int at, int most) -> void {
            if (at == nr) {
                if (left == 1 && cur[nr - 1] > best && (nr < 3 || cur[2] <= 9)) {
                    best = cur[nr - 1];  // non-increasing: the last is the smallest
                    d.nr = nr;
                    d.rad[0] = cur[0];
                    d.rad[nr - 1] = cur[1];
                    std::copy(cur + 2, cur + nr, d.rad + 1);
                }
                return;
            }
            for (int r : radices)
                if (r <= most && left % r == 0) {
                    cur[at] = r;
                    self(self, left / r, at + 1, r);
                }
        };
        split(split, n, 0, 18);
    }
    return d.nr > 0 && n / min_radix(d) <= 256;
}

// threads of a column pass: every butterfly of its widest stage for kc columns, in whole waves
static int col_threads(const PlaneDim& d, int kc) { return cdiv(kc * (d.n / min_radix(d)), 64) * 64; }

static size_t lds_spread(const PlaneGeom& g, size_t cs) { return 16 * (size_t)g.Pc * g.S + cs * g.K2; }
static size_t lds_gather(const PlaneGeom& g, size_t cs) { return cs * ((size_t)(g.Pc + 2) * g.S + g.K2); }
static size_t lds_force(const PlaneGeom& g, size_t cs) { return cs * ((size_t)(2 * g.Pf + 4) * g.S + g.K2); }
static size_t lds_lines(int N, int kc, size_t cs) { return cs * ((size_t)N * (kc | 1) + N); }

// Threads of the one-launch y-x-y pass, 0 where it does not serve the grid: a column of at most
// kPlYxyPoints points, both lengths of two stages, one butterfly per thread.  The pass reads 8 or 16
// bytes of each 128-byte line, so it gains only where launches cost more than bytes: y + x + y 14.2
// against 9.5 us at 24^3, 14.8 / 11.9 at 36^3, 15.4 / 15.2 at 48^3 and 17.0 / 24.2 at 64^3 in FP32
// (15.2 / 10.1, 15.4 / 13.2, 18.3 / 19.4, 23.4 / 30.7 in FP64); at 48^3 the launches saved decide.
constexpr int kPlYxyPoints = 2304;
static size_t lds_yxy(const PlaneGeom& g, size_t cs) { return cs * ((size_t)g.K0 * (g.K1 | 1) + g.K0 + g.K1); }
static int yxy_threads(const PlaneGeom& g, const PlaneDim& dy, const PlaneDim& dx, size_t cs)
{
    if (g.K0 * g.K1 > kPlYxyPoints || dy.nr != 2 || dx.nr != 2 || lds_yxy(g, cs) > kPlLdsMax)
        return 0;
    const int nt = std::max(g.K0 * (g.K1 / min_radix(dy)), g.K1 * (g.K0 / min_radix(dx)));
    return nt <= kPlYxyThreads ? cdiv(nt, 64) * 64 : 0;
}

// Geometry and factorisations of a context's grid, worked out once.
struct PlanePlan {
    PlaneGeom g;
    PlaneDim d[3];
    bool factors;  // every length has a factorisation (else g is not filled)
    int yxy;       // threads of the one-launch y-x-y pass, 0: the three passes
};

static PlaneGeom make_geom(const amoeba_ctx* c, const PlaneDim (&d)[3])
{
    PlaneGeom g;
    g.npad = c->npad;
    g.K0 = c->K[0];
    g.K1 = c->K[1];
    g.K2 = c->K[2];
    g.kh = g.K2 / 2 + 1;
    const size_t cs = c->mixed ? sizeof(float2) : sizeof(double2);
    // rows of G start on 128-byte lines and column chunks are whole lines, so the column passes
    // move whole lines (unaligned rows of a chunk cost about twice the bytes: measured)
    const int line = (int)(128 / cs);
    g.ks = cdiv(g.kh, line) * line;
    g.S = 2 * g.kh;
    g.P = (g.K1 + 1) / 2;
    // row chunks: about kPlTargetWG workgroups of 512 threads, within the LDS and conversion
    // limits; a grid that needs more than kPlLargeWG of them (two 512-thread workgroups fit a CU)
    // takes 256-thread workgroups on smaller chunks, so that more of them are resident at once
    // and the chip is not left with a partial last round (measured at 216^3)
    const int zb = g.K2 / min_radix(d[2]);
    auto one_round = [&]() { return g.Pc * zb <= g.nt; };  // the spread's first stage: a thread for every butterfly
    auto rows = [&](int target) {
        g.nyc = std::min(g.P, std::max(1, cdiv(target, g.K0)));
        g.Pc = cdiv(g.P, g.nyc);
        while (g.Pc > 1 && (lds_spread(g, cs) > kPlLdsMax || lds_gather(g, cs) > kPlLdsMax || !one_round()))
            g.Pc = cdiv(g.Pc, 2);
        g.nyc = cdiv(g.P, g.Pc);
    };
    g.nt = kPlThreads;
    rows(kPlTargetWG);
    if (g.K0 * g.nyc > kPlLargeWG) {
        g.nt = kPlThreadsLarge;
        rows(kPlTargetWGLarge);
        if (!one_round()) {
            g.nt = kPlThreads;
            rows(kPlTargetWG);
        }
    }
    // the gradient's interpolation holds a line per row: row chunks of at most half the pairs
    g.Pf = cdiv(g.Pc, 2);
    while (g.Pf > 1 && lds_force(g, cs) > kPlLdsMax)
        g.Pf = cdiv(g.Pf, 2);
    g.nyf = cdiv(g.P, g.Pf);
    // column chunks of one line, fewer columns where a pass would exceed the threads or the LDS of
    // a workgroup (lengths far above those of the plane path's usual grids)
    g.kc = line;
    while (g.kc > 1 && (col_threads(d[0], g.kc) > kPlColThreads || col_threads(d[1], g.kc) > kPlColThreads ||
                        lds_lines(g.K0, g.kc, cs) > kPlLdsMax || lds_lines(g.K1, g.kc, cs) > kPlLdsMax))
        g.kc /= 2;
    g.kcs = 0;
    while ((1 << g.kcs) < g.kc)
        ++g.kcs;
    g.nty = col_threads(d[1], g.kc);
    g.ntx = col_threads(d[0], g.kc);
    g.nkc = cdiv(g.kh, g.kc);
    g.kl = g.kc | 1;
    g.klx = c->K[0] / c->prm.box[0];
    g.kly = c->K[1] / c->prm.box[1];
    g.klz = c->K[2] / c->prm.box[2];
    return g;
}

static const PlanePlan& plane_plan(const amoeba_ctx* c)
{
    if (!c->plane_plan) {
        auto p = std::make_shared<PlanePlan>();
        p->factors = true;
        p->yxy = 0;
        for (int a = 0; a < 3; ++a)
            p->factors = plane_factor(c->K[a], p->d[a]) && p->factors;
        if (p->factors) {
            p->g = make_geom(c, p->d);
            p->yxy = yxy_threads(p->g, p->d[1], p->d[0], c->mixed ? sizeof(float2) : sizeof(double2));
        }
        c->plane_plan = p;
    }
    return *c->plane_plan;
}

int plane_row_stride(const amoeba_ctx* c) { return plane_plan(c).g.ks; }

void plane_column_chunks(const amoeba_ctx* c, int* kc, int* nkc)
{
    const PlaneGeom& g = plane_plan(c).g;
    *kc = g.kc;
    *nkc = g.nkc;
}

bool plane_eligible(const amoeba_ctx* c)
{
    const PlanePlan& p = plane_plan(c);
    if (!p.factors)
        return false;
    const PlaneGeom& g = p.g;
    const size_t cs = c->mixed ? sizeof(float2) : sizeof(double2);
    return lds_spread(g, cs) <= kPlLdsMax && lds_gather(g, cs) <= kPlLdsMax &&
           g.Pc * (g.K2 / min_radix(p.d[2])) <= g.nt && lds_lines(g.K0, g.kc, cs) <= kPlLdsMax &&
           lds_lines(g.K1, g.kc, cs) <= kPlLdsMax && g.nty <= kPlColThreads && g.ntx <= kPlColThreads && (size_t)g.K0 * g.K1 <= 65536;
}

// Whether the gradient's interpolation fits a workgroup's LDS (a line per row and the halo).
bool plane_force_fits(const amoeba_ctx* c)
{
    return lds_force(plane_plan(c).g, c->mixed ? sizeof(float2) : sizeof(double2)) <= kPlLdsMax;
}

int plane_setup(amoeba_ctx* c)
{
    c->plane_ok = plane_eligible(c);
    if (!c->plane_ok)
        return AMOEBA_OK;
    const size_t rs = c->mixed ? sizeof(float) : sizeof(double);
    const int nb2 = c->K[0] * c->K[1];
    int rc;
    if ((rc = ctx_alloc(c, (void**)&c->xb_start, sizeof(int) * (nb2 + 1))) ||
        (rc = ctx_alloc(c, (void**)&c->xb_count, sizeof(int) * (nb2 + 1))) ||
        (rc = ctx_alloc(c, (void**)&c->xb_rec, sizeof(int4) * c->npad)) ||
        (rc = ctx_alloc(c, &c->xb_w, 4 * rs * c->npad)) ||
        (rc = ctx_alloc(c, &c->rec_part, 4 * rs * 5 * (size_t)c->npad)))
        return rc;
    for (int a = 0; a < 3; ++a) {
        if ((rc = ctx_alloc(c, &c->pl_roots[a], 2 * rs * c->K[a])))
            return rc;
        if (c->mixed)
            hipLaunchKernelGGL(k_plane_roots<float>, dim3(nblk(c->K[a], 256)), dim3(256), 0, c->stream, c->K[a],
                               (float2*)c->pl_roots[a]);
        else
            hipLaunchKernelGGL(k_plane_roots<double>, dim3(nblk(c->K[a], 256)), dim3(256), 0, c->stream, c->K[a],
                               (double2*)c->pl_roots[a]);
    }
    return AMOEBA_OK;
}

int plane_bin_atoms(amoeba_ctx* c)
{
    if (!c->plane_ok)
        return AMOEBA_OK;
    hipStream_t st = c->stream;
    const int nb2 = c->K[0] * c->K[1];
    int3 K = make_int3(c->K[0], c->K[1], c->K[2]);
    double3 kl = make_double3(c->K[0] / c->prm.box[0], c->K[1] / c->prm.box[1], c->K[2] / c->prm.box[2]);
    // xb_count is zero between binnings (zeroed at allocation; the fill counts it back down)
    hipLaunchKernelGGL(k_xybin_count, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm, c->pos_s, kl, K,
                       c->xb_count);
    int rc = device_scan(c, nb2, c->xb_count, c->xb_start);
    if (rc) {
        hipMemsetAsync(c->xb_count, 0, sizeof(int) * (nb2 + 1), st);
        return rc;
    }
    if (c->mixed)
        hipLaunchKernelGGL(k_xybin_fill<float>, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm,
                           c->pos_s, kl, K, c->xb_start, c->xb_count, c->xb_rec, (float4*)c->xb_w);
    else
        hipLaunchKernelGGL(k_xybin_fill<double>, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm,
                           c->pos_s, kl, K, c->xb_start, c->xb_count, c->xb_rec, (double4*)c->xb_w);
    return AMOEBA_OK;
}

// The passes of one reciprocal field, for the two entry points below and the gradient.
template <typename R> struct PlanePasses {
    using C = typename PlT<R>::C;
    using R4 = typename PlT<R>::R4;
    static constexpr bool FIX = std::is_same<R, float>::value;
    amoeba_ctx* c;
    const PlaneGeom& g;
    const PlaneDim (&d)[3];
    const int yxy;
    const C* const* roots;
    explicit PlanePasses(amoeba_ctx* ctx)
        : c(ctx), g(plane_plan(ctx).g), d(plane_plan(ctx).d), yxy(plane_plan(ctx).yxy),
          roots((const C* const*)ctx->pl_roots)
    {
    }
    bool small() const { return g.nt == kPlThreads; }
    void spread(const R4* src, int sstride, bool perm, C* gc, int ud) const
    {
        auto k = perm ? (small() ? k_pme_spread_z<R, FIX, true, kPlThreads>
                                 : k_pme_spread_z<R, FIX, true, kPlThreadsLarge>)
                      : (small() ? k_pme_spread_z<R, FIX, false, kPlThreads>
                                 : k_pme_spread_z<R, FIX, false, kPlThreadsLarge>);
        hipLaunchKernelGGL(k, dim3(g.K0 * g.nyc), dim3(g.nt), lds_spread(g, sizeof(C)), c->stream, g, d[2],
                           c->xb_start, c->xb_rec, (const R4*)c->xb_w, src, sstride, roots[2], gc, c->sc, ud);
    }
    // y, x with the influence function and y back, of gc (and gc1 when given); reduce: the
    // real-space reduction of a small system's product in the same launch
    void transforms(C* gc, C* gc1, int ud, bool reduce = false) const
    {
        const int ng = gc1 ? 2 : 1;
        const RealReduceArgs<R> rr{reduce ? c->npad : 0, c->eipart, (const R*)c->jbuf, c->rev_ptr, c->rev_idx,
                                   c->ereal};
        if (const int nt = yxy) {
            hipLaunchKernelGGL(k_pme_yxy<R>, dim3(g.kh + (reduce ? cdiv(4 * c->npad, nt) : 0), ng), dim3(nt),
                               lds_yxy(g, sizeof(C)), c->stream, g, d[1], d[0], gc, gc1, (const R*)c->theta_pl,
                               roots[1], roots[0], rr, c->sc, ud);
            return;
        }
        const size_t ly = lds_lines(g.K1, g.kc, sizeof(C)), lx = lds_lines(g.K0, g.kc, sizeof(C));
        hipLaunchKernelGGL((k_pme_ylines<R, -1>), dim3(g.K0 * g.nkc + (reduce ? cdiv(4 * c->npad, g.nty) : 0), ng),
                           dim3(g.nty), ly, c->stream, g, d[1], gc, gc1, roots[1], rr, c->sc, ud);
        hipLaunchKernelGGL(k_pme_xconv<R>, dim3(g.K1 * g.nkc, ng), dim3(g.ntx), lx, c->stream, g, d[0], gc, gc1,
                           (const R*)c->theta_pl, roots[0], c->sc, ud);
        hipLaunchKernelGGL((k_pme_ylines<R, 1>), dim3(g.K0 * g.nkc, ng), dim3(g.nty), ly, c->stream, g, d[1], gc,
                           gc1, roots[1], RealReduceArgs<R>{}, c->sc, ud);
    }
    void gather(const C* gc, int ud) const
    {
        auto k = small() ? k_pme_z_gather<R, kPlThreads> : k_pme_z_gather<R, kPlThreadsLarge>;
        hipLaunchKernelGGL(k, dim3(g.K0 * g.nyc), dim3(g.nt), lds_gather(g, sizeof(C)), c->stream, g, d[2], gc,
                           c->xb_start, c->xb_rec, (const R4*)c->xb_w, roots[2], (R4*)c->rec_part, c->sc, ud);
    }
};

// part 1: the spread pass; part 2: the transforms and the interpolation; 3: both.  perm: spread
// the permanent multipoles (mp) instead of the direction, all stages timed as AMOEBA_T_PERM.
template <typename R> static void plane_field_t(amoeba_ctx* c, bool use_done, int parts, bool perm)
{
    using P = PlanePasses<R>;
    const P p(c);
    const int ud = use_done ? 1 : 0;
    typename P::C* gc = (typename P::C*)c->grid_c;
    if (parts & 1) {
        StageTimer tm(c, perm ? AMOEBA_T_PERM : AMOEBA_T_SPREAD);
        const void* src = perm ? (c->mixed ? (const void*)c->mp_f : (const void*)c->mp_d)
                               : (c->mixed ? (const void*)c->pv_f : (const void*)c->pv_d);
        p.spread((const typename P::R4*)src, perm ? 3 : 1, perm, gc, perm ? 0 : ud);
    }
    if (!(parts & 2))
        return;
    {
        StageTimer tm(c, perm ? AMOEBA_T_PERM : AMOEBA_T_FFT);
        p.transforms(gc, nullptr, ud);
    }
    StageTimer tm(c, perm ? AMOEBA_T_PERM : AMOEBA_T_GATHER);
    p.gather(gc, ud);
}

// A small system: at most small_blocks() blocks, row passes of the 512-thread workgroups.  Its dipole
// product is enqueued as one launch for tiles and spread, with the real-space reduction beside the
// transforms, on the context stream, unless stage timers want the stages by themselves.
bool plane_small_system(const amoeba_ctx* c)
{
    return pme_use_planes(c) && c->ntiles > 0 && c->nb <= small_blocks(c) && plane_plan(c).g.nt == kPlThreads;
}
bool plane_small_product(const amoeba_ctx* c) { return plane_small_system(c) && !c->timing && !c->timing_live; }

// The product up to its combine: E_real in ereal, the reciprocal shares in rec_part.
template <typename R> static void small_product_t(amoeba_ctx* c, bool use_done)
{
    using C = typename PlT<R>::C;
    const PlanePasses<R> p(c);
    const int ud = use_done ? 1 : 0;
    launch_product_head(c, HeadSpread<R>{p.g, p.d[2], p.roots[2], (C*)c->grid_c, lds_spread(p.g, sizeof(C)), ud});
    p.transforms((C*)c->grid_c, nullptr, ud, true);
    p.gather((const C*)c->grid_c, ud);
}

void plane_small_product_fields(amoeba_ctx* c, bool use_done)
{
    if (c->mixed)
        small_product_t<float>(c, use_done);
    else
        small_product_t<double>(c, use_done);
}

// Complex values of one half grid of the plane path (a second one is the gradient's workspace).
size_t plane_grid_bytes(const amoeba_ctx* c)
{
    return (size_t)c->K[0] * c->K[1] * plane_row_stride(c) * 2 * (c->mixed ? sizeof(float) : sizeof(double));
}

// Reciprocal shares of the polarization gradient (part[5][npad], FP64): both potentials, then
// their interpolation.  src: [npad][4] (R4) multipoles and dipoles (the ForceKind records); grid1:
// a second half grid.
template <typename R> static void plane_force_t(amoeba_ctx* c, const void* src, void* grid1, double4* part)
{
    using P = PlanePasses<R>;
    using C = typename P::C;
    const P p(c);
    const typename P::R4* s4 = (const typename P::R4*)src;
    C *gp = (C*)c->grid_c, *gm = (C*)grid1;
    p.spread(s4, 4, true, gp, 0);
    p.spread(s4 + 3, 4, false, gm, 0);
    p.transforms(gp, gm, 0);
    hipLaunchKernelGGL((k_pme_z_force<R, kPlThreadsLarge>), dim3(p.g.K0 * p.g.nyf), dim3(kPlThreadsLarge),
                       lds_force(p.g, sizeof(C)), c->stream, p.g, p.d[2], (const C*)gp, (const C*)gm, c->xb_start,
                       c->xb_rec, c->pos_s, p.roots[2], (const double4*)c->mp_d, c->v_mu, part);
}

void plane_force(amoeba_ctx* c, const void* src, void* grid1, double4* part)
{
    if (c->mixed)
        plane_force_t<float>(c, src, grid1, part);
    else
        plane_force_t<double>(c, src, grid1, part);
}

void plane_dipole_field(amoeba_ctx* c, bool use_done, int parts)
{
    if (c->mixed)
        plane_field_t<float>(c, use_done, parts, false);
    else
        plane_field_t<double>(c, use_done, parts, false);
}

void plane_perm_field(amoeba_ctx* c)
{
    if (c->mixed)
        plane_field_t<float>(c, false, 3, true);
    else
        plane_field_t<double>(c, false, 3, true);
}

void plane_gather(amoeba_ctx* c, double* out)
{
    StageTimer tm(c, AMOEBA_T_GATHER);
    double3 kl = make_double3(c->K[0] / c->prm.box[0], c->K[1] / c->prm.box[1], c->K[2] / c->prm.box[2]);
    if (c->mixed)
        hipLaunchKernelGGL((k_plane_combine<float, 0>), dim3(nblk(c->npad, 256)), dim3(256), 0, c->stream, c->npad,
                           kl, c->perm, (const float4*)c->rec_part, c->alpha_inv_s, (const double*)nullptr, 0.0,
                           (const double*)nullptr, (const float4*)nullptr, (const int*)nullptr, (const int*)nullptr,
                           (const double*)nullptr, out, c->sc, (double*)nullptr, 0, 0);
    else
        hipLaunchKernelGGL((k_plane_combine<double, 0>), dim3(nblk(c->npad, 256)), dim3(256), 0, c->stream,
                           c->npad, kl, c->perm, (const double4*)c->rec_part, c->alpha_inv_s, (const double*)nullptr, 0.0,
                           (const double*)nullptr, (const double4*)nullptr, (const int*)nullptr,
                           (const int*)nullptr, (const double*)nullptr, out, c->sc, (double*)nullptr, 0, 0);
}

int plane_combine(amoeba_ctx* c, bool use_done, bool dot_pq, bool reduced)
{
    StageTimer tm(c, AMOEBA_T_GATHER);
    double3 kl = make_double3(c->K[0] / c->prm.box[0], c->K[1] / c->prm.box[1], c->K[2] / c->prm.box[2]);
    const double self = self_coefficient(c);
    const int nwg = nblk(c->npad, 256);
    if (c->mixed) {
        auto k = reduced ? k_plane_combine<float, 2> : k_plane_combine<float, 1>;
        hipLaunchKernelGGL(k, dim3(nwg), dim3(256), 0, c->stream, c->npad, kl, c->perm, (const float4*)c->rec_part,
                           c->alpha_inv_s, c->v_p, self, c->eipart, (const float4*)c->jbuf, c->rev_ptr, c->rev_idx,
                           c->ereal, c->v_q, c->sc, c->red.part, (int)use_done, (int)dot_pq);
    } else {
        auto k = reduced ? k_plane_combine<double, 2> : k_plane_combine<double, 1>;
        hipLaunchKernelGGL(k, dim3(nwg), dim3(256), 0, c->stream, c->npad, kl, c->perm, (const double4*)c->rec_part,
                           c->alpha_inv_s, c->v_p, self, c->eipart, (const double4*)c->jbuf, c->rev_ptr, c->rev_idx,
                           c->ereal, c->v_q, c->sc, c->red.part, (int)use_done, (int)dot_pq);
    }
    return nwg;
}

}  // namespace amoeba
