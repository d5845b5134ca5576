// Real-space pair kernels over 64 x 64 block tiles (paper: "Neighbor list" block-matrix
// interaction, "List filtering" group-atom tiles, and the real-space scheme; the scaled pairs
// are corrected in a separate pass as in the paper's final real-space scheme).
//
// One workgroup (4 waves) per 64-atom i-block; the waves take the block's tiles in turn.  The
// block's i-atoms are staged in LDS once; each wave stages its tile's 64 j-atoms (positions
// relative to the i-block origin, dipoles or multipoles, damping parameters) and the tile's
// in-cutoff bitmasks.  An exclusive wave scan of the row popcounts numbers the in-cutoff pairs,
// and every lane evaluates an equal contiguous share of them by walking the set bits of the
// masks, so masked-out pair slots cost nothing.  Each pair is evaluated once (Newton's third
// law): the field at i accumulates in registers while the lane stays on a row and is then added
// to the block's LDS accumulator, which collects all tiles of the block; the field at j is added,
// per pair, to the tile's LDS accumulator.  In mixed precision every LDS addition is a 64-bit
// fixed-point integer (38 fraction bits; see LdsAcc), so the sums do not depend on the order of
// the lanes' atomics and the product is bitwise reproducible; FP64 mode accumulates in FP64.
//
// No global atomics: a block writes its i-field once (eipart) and each off-diagonal tile writes
// its 64 j-fields to its own slot of jbuf; the diagonal tile's j-field goes straight into the
// block's accumulator.  Every atom's real-space field is then the sum of its eipart and of the
// jbuf slots listed for it in the reverse index built with the list (in mixed precision an
// exact fixed-point sum, so the order of the list does not matter; see JSum).
//
// Pair math (Ewald real space, Thole damping of Ren & Ponder as used by AMOEBA):
//   B0 = erfc(beta r)/r,  B_n = ((2n-1) B_{n-1} + (2 beta^2)^n e^{-beta^2 r^2} / (beta sqrt(pi))) / r^2
//   eps = a (r / (alpha_i alpha_j)^{1/6})^3,  a = min(a_i, a_j)
//   B1' = B1 - e^{-eps} / r^3,  B2' = B2 - 3 (1+eps) e^{-eps} / r^5,
//   B3' = B3 - 15 (1 + eps + 3/5 eps^2) e^{-eps} / r^7
//   dipole field at i from mu_j:  -B1' mu_j + B2' (mu_j.r) r           (r = r_i - r_j)
//   multipole field at i from j:   q_j B1' r - B1' d_j + B2' (d_j.r) r
//                                  + (1/3) B3' (Theta_j:rr) r - (2/3) B2' Theta_j r
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "tiles.h"

namespace amoeba {

template <typename R, bool FIX, class K, bool MI, int CM, int W>
__global__ __launch_bounds__(64 * W, K::kMinWaves) void k_block_tiles(const int* __restrict__ blk_tile0,
                                                     const int* __restrict__ tile_np,
                                                     const int* __restrict__ tile_j,
                                                     const unsigned long long* __restrict__ tile_mask,
                                                     const uint16_t* __restrict__ tile_walk,
                                                     const typename V4<R>::T* __restrict__ jrel,
                                                     const typename V4<R>::T* __restrict__ off,
                                                     const typename V4<R>::T* __restrict__ par,
                                                     const typename V4<R>::T* __restrict__ src, EwaldArgs<R> ew,
                                                     double* __restrict__ eipart, R* __restrict__ jbuf,
                                                     const PcgScalars* __restrict__ sc, int use_done,
                                                     const int* __restrict__ coef_row0, long long coef_cap_rows,
                                                     typename V2<R>::T* __restrict__ coef)
{
    __shared__ TileLds<R, FIX, K, W> L;
    if (use_done && sc->done)
        return;
    block_tiles<R, FIX, K, MI, CM, W>(L, blockIdx.x, blk_tile0, tile_np, tile_j, tile_mask, tile_walk, jrel,
                                                off, par, src, ew, eipart, jbuf, coef_row0, coef_cap_rows, coef);
}

template <typename R>
__global__ void k_real_reduce(int npad, const double* __restrict__ eipart, const R* __restrict__ jbuf,
                              const int* __restrict__ rev_ptr, const int* __restrict__ rev_idx,
                              double* __restrict__ ereal, const PcgScalars* __restrict__ sc, int use_done)
{
    // latency bound and beside the reciprocal passes on the other stream: its waves issue first
    __builtin_amdgcn_s_setprio(3);
    if (use_done && sc->done)
        return;
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < npad)
        real_reduce<R>(s, eipart, jbuf, rev_ptr, rev_idx, ereal);
}

// Waves per block: four where the blocks fill the chip (a block's tiles share its staged i data and
// one row of accumulators), eight for a small system, whose blocks leave the chip idle and whose
// time is the longest wave's.
template <typename F> static void with_waves(const amoeba_ctx* c, F&& f)
{
    if (c->nb <= small_blocks(c))
        f(std::integral_constant<int, kSmallWaves>{});
    else
        f(std::integral_constant<int, kWavesPerWG>{});
}

template <typename R, bool FIX, bool MI, int CM, int W>
static void dipole_tiles(amoeba_ctx* c, bool use_done, hipStream_t st, const typename V4<R>::T* jrel,
                         const typename V4<R>::T* off, const typename V4<R>::T* par, const typename V4<R>::T* pv)
{
    hipLaunchKernelGGL((k_block_tiles<R, FIX, DipoleKind<R>, MI, CM, W>), dim3(c->nb), dim3(64 * W), 0, st,
                       c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask, c->tile_walk, jrel, off, par, pv,
                       make_ewald<R>(c),
                       c->eipart, (R*)c->jbuf, c->sc, (int)use_done, c->coef_row0, (long long)c->coef_cap_rows,
                       (typename V2<R>::T*)c->coef);
}

template <typename R, bool FIX, bool MI, int W>
static void dipole_tiles_cm(amoeba_ctx* c, int cm, bool use_done, hipStream_t st, const typename V4<R>::T* jrel,
                            const typename V4<R>::T* off, const typename V4<R>::T* par,
                            const typename V4<R>::T* pv)
{
    if (cm == kCoefReplay)
        dipole_tiles<R, FIX, MI, kCoefReplay, W>(c, use_done, st, jrel, off, par, pv);
    else if (cm == kCoefRecord)
        dipole_tiles<R, FIX, MI, kCoefRecord, W>(c, use_done, st, jrel, off, par, pv);
    else
        dipole_tiles<R, FIX, MI, kCoefCompute, W>(c, use_done, st, jrel, off, par, pv);
}

// Whether the dipole products use the store.  AUTO: in FP64, where the pair functions cost far
// more than reading 16 bytes per pair back; not in mixed precision, where the FP32 tiles are
// bound by their LDS traffic (the field atomics and the j-data reads), which the store leaves as
// it is, so that replay measured no faster than evaluation.
bool coef_store_on(const amoeba_ctx* c)
{
    return c->pair_store == AMOEBA_PAIRS_STORED || (c->pair_store == AMOEBA_PAIRS_AUTO && !c->mixed);
}

// Coefficient mode of the next dipole product: the store needs the refresh's row scan and a
// buffer; the first product of a configuration records, the later ones replay.
int next_coef_mode(const amoeba_ctx* c)
{
    if (!coef_store_on(c) || !c->coef_rows_ok || !c->coef)
        return kCoefCompute;
    return c->coef_ready ? kCoefReplay : kCoefRecord;
}

// The mode of a dipole product about to be enqueued; the next one then replays what it records.
int begin_coef_mode(amoeba_ctx* c, bool* use_done)
{
    const int cm = next_coef_mode(c);
    // a recording product runs even when a converged PCG skips the rest of its iteration, so
    // that the store is whole for the products that replay it
    if (cm == kCoefRecord) {
        *use_done = false;
        c->coef_ready = true;
    }
    c->coef_last_stored = cm != kCoefCompute;
    return cm;
}

template <bool MI> static void mutual_tiles(amoeba_ctx* c, bool use_done, hipStream_t st)
{
    if (c->ntiles == 0)
        return;
    StageTimer tm(c, AMOEBA_T_REAL, st);
    const int cm = begin_coef_mode(c, &use_done);
    auto go = [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        if (c->mixed)
            dipole_tiles_cm<float, true, MI, W>(c, cm, use_done, st, c->jrel_f, c->off_f, c->par_f, c->pv_f);
        else
            dipole_tiles_cm<double, false, MI, W>(c, cm, use_done, st, c->jrel_d, c->off_d, c->par_d, c->pv_d);
    };
    with_waves(c, go);
}

void coef_invalidate(amoeba_ctx* c) { c->coef_ready = false; }

// Frees the store (hipFree waits for the device, so no queued product still reads it).
void coef_release(amoeba_ctx* c)
{
    if (!c->coef)
        return;
    hipFree(c->coef);
    c->coef = nullptr;
    c->ws_bytes -= c->coef_bytes;
    c->coef_bytes = 0;
    c->coef_cap_rows = 0;
    coef_invalidate(c);
}

// Called with the context stream synchronized: grows the store to the rows of the last mask
// refresh (read back with that synchronization) plus an eighth, or to what the workspace cap
// leaves.  A store smaller than the rows is still used: the tiles beyond it evaluate their
// coefficients.
int coef_reserve(amoeba_ctx* c)
{
    if (!c->coef_rows_pending || !coef_store_on(c))
        return AMOEBA_OK;
    c->coef_rows_pending = false;
    const int64_t rows = (int64_t)(unsigned)c->flags_host[10];
    if (rows <= c->coef_cap_rows)
        return AMOEBA_OK;
    const int64_t row_bytes = (int64_t)kBlock * (c->mixed ? sizeof(float2) : sizeof(double2));
    int64_t want = rows + rows / 8 + 64;
    const int64_t others = c->ws_bytes - c->coef_bytes;
    if (c->prm.max_workspace_bytes > 0)
        want = std::min(want, (c->prm.max_workspace_bytes - others) / row_bytes);
    if (want <= c->coef_cap_rows)
        return AMOEBA_OK;  // the cap leaves no more room: keep the store it has
    coef_release(c);
    void* q = nullptr;
    if (want < 64 || hipMalloc(&q, (size_t)(want * row_bytes)) != hipSuccess) {
        (void)hipGetLastError();
        return AMOEBA_OK;  // no store: the products evaluate the coefficients
    }
    c->coef = q;
    c->coef_bytes = want * row_bytes;
    c->ws_bytes += c->coef_bytes;
    c->coef_cap_rows = want;
    return AMOEBA_OK;
}

void launch_mutual_tiles(amoeba_ctx* c, bool use_done, hipStream_t st)
{
    if (!st)
        st = c->stream;
    if (c->skip_mimg)
        mutual_tiles<false>(c, use_done, st);
    else
        mutual_tiles<true>(c, use_done, st);
}

void launch_real_reduce(amoeba_ctx* c, double* ereal, hipStream_t st, bool use_done)
{
    if (!st)
        st = c->stream;
    if (c->mixed)
        hipLaunchKernelGGL(k_real_reduce<float>, dim3((c->npad + 255) / 256), dim3(256), 0, st, c->npad,
                           c->eipart, (const float*)c->jbuf, c->rev_ptr, c->rev_idx, ereal, c->sc, (int)use_done);
    else
        hipLaunchKernelGGL(k_real_reduce<double>, dim3((c->npad + 255) / 256), dim3(256), 0, st, c->npad,
                           c->eipart, (const double*)c->jbuf, c->rev_ptr, c->rev_idx, ereal, c->sc, (int)use_done);
}

template <bool MI, int W> static void perm_tiles(amoeba_ctx* c, hipStream_t st)
{
    StageTimer tm(c, AMOEBA_T_PERM, st);
    if (c->mixed)
        hipLaunchKernelGGL((k_block_tiles<float, true, MultipoleKind<float>, MI, kCoefCompute, W>), dim3(c->nb), dim3(64 * W), 0,
                           st, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask, c->tile_walk, c->jrel_f,
                           c->off_f, c->par_f,
                           (const float4*)c->mp_f, make_ewald<float>(c), c->eipart, (float*)c->jbuf, c->sc, 0,
                           (const int*)nullptr, 0ll, (float2*)nullptr);
    else
        hipLaunchKernelGGL((k_block_tiles<double, false, MultipoleKind<double>, MI, kCoefCompute, W>), dim3(c->nb), dim3(64 * W), 0,
                           st, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask, c->tile_walk, c->jrel_d,
                           c->off_d, c->par_d,
                           (const double4*)c->mp_d, make_ewald<double>(c), c->eipart, (double*)c->jbuf, c->sc, 0,
                           (const int*)nullptr, 0ll, (double2*)nullptr);
}

template <bool MI, int W> static void force_tiles(amoeba_ctx* c, const void* src, hipStream_t st)
{
    if (c->mixed)
        hipLaunchKernelGGL((k_block_tiles<float, true, ForceKind<float>, MI, kCoefCompute, W>), dim3(c->nb), dim3(64 * W), 0,
                           st, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask, c->tile_walk,
                           c->jrel_f, c->off_f,
                           c->par_f, (const float4*)src, make_ewald<float>(c), c->eipart, (float*)c->jbuf, c->sc, 0,
                           (const int*)nullptr, 0ll, (float2*)nullptr);
    else
        hipLaunchKernelGGL((k_block_tiles<double, false, ForceKind<double>, MI, kCoefCompute, W>), dim3(c->nb), dim3(64 * W), 0,
                           st, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask, c->tile_walk,
                           c->jrel_d, c->off_d,
                           c->par_d, (const double4*)src, make_ewald<double>(c), c->eipart, (double*)c->jbuf, c->sc,
                           0, (const int*)nullptr, 0ll, (double2*)nullptr);
}

// Real-space pair sums of the polarization gradient, sum_j G_ij per slot, into out (FP64 N x 3);
// src: [npad][4] (R4) multipoles and dipoles in the ForceKind layout.
void launch_force_tiles(amoeba_ctx* c, const void* src, double* out, hipStream_t st)
{
    if (c->ntiles > 0) {
        with_waves(c, [&](auto waves) {
            constexpr int W = decltype(waves)::value;
            if (c->skip_mimg)
                force_tiles<false, W>(c, src, st);
            else
                force_tiles<true, W>(c, src, st);
        });
        launch_real_reduce(c, out, st);
    } else {
        hipMemsetAsync(out, 0, sizeof(double) * 3 * (size_t)c->npad, st);
    }
}

// Radial neighbour sums of the learned guess into out (FP64 N x 3, slot order): the pair walk and the
// reduction of the fields, each pair once, lanes level in their pair counts.  Evaluating each pair for
// its row and again for its column took 88 us at 96,000 atoms in mixed precision, this takes 35 us.
template <bool MI, int W> static void radial_tiles(amoeba_ctx* c)
{
    if (c->mixed)
        hipLaunchKernelGGL((k_block_tiles<float, true, RadialKind<float>, MI, kCoefCompute, W>), dim3(c->nb),
                           dim3(64 * W), 0, c->stream, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask,
                           c->tile_walk, c->jrel_f, c->off_f, c->par_f, (const float4*)nullptr, make_ewald<float>(c),
                           c->eipart, (float*)c->jbuf, c->sc, 0, (const int*)nullptr, 0ll, (float2*)nullptr);
    else
        hipLaunchKernelGGL((k_block_tiles<double, false, RadialKind<double>, MI, kCoefCompute, W>), dim3(c->nb),
                           dim3(64 * W), 0, c->stream, c->blk_tile0, c->tile_np, c->tile_j, c->tile_mask,
                           c->tile_walk, c->jrel_d, c->off_d, c->par_d, (const double4*)nullptr,
                           make_ewald<double>(c), c->eipart, (double*)c->jbuf, c->sc, 0, (const int*)nullptr, 0ll,
                           (double2*)nullptr);
}

void launch_radial_sums(amoeba_ctx* c, double* out)
{
    if (c->ntiles == 0) {
        hipMemsetAsync(out, 0, sizeof(double) * 3 * (size_t)c->npad, c->stream);
        return;
    }
    {
        StageTimer tm(c, AMOEBA_T_GUESS);
        with_waves(c, [&](auto waves) {
            constexpr int W = decltype(waves)::value;
            if (c->skip_mimg)
                radial_tiles<false, W>(c);
            else
                radial_tiles<true, W>(c);
        });
    }
    launch_real_reduce(c, out);
}

void launch_perm_tiles(amoeba_ctx* c, hipStream_t st)
{
    if (c->ntiles == 0)
        return;
    if (!st)
        st = c->stream;
    with_waves(c, [&](auto waves) {
        constexpr int W = decltype(waves)::value;
        if (c->skip_mimg)
            perm_tiles<false, W>(c, st);
        else
            perm_tiles<true, W>(c, st);
    });
    launch_real_reduce(c, c->ereal, st);
}

// ------------------------------------------------------------------------------------------
// K4 + final assembly of E_perm (FP64): real-space field + reciprocal field + dipole self
// field + the scaled-pair correction of every listed pair (at any separation):
//   inside rc:  delta B_n = -c_n (1 - s) lambda_{2n+1} / r^{2n+1}   (tiles used s = 1)
//   beyond rc:  delta B_n = -c_n (1 - s lambda_{2n+1}) / r^{2n+1}   (tiles skipped the pair)
// ------------------------------------------------------------------------------------------
__global__ void k_perm_assemble(int npad, const int* __restrict__ perm, const double4* __restrict__ pos_s,
                                const double4* __restrict__ par, const double4* __restrict__ mp,
                                const int* __restrict__ sc_ptr, const int* __restrict__ sc_j,
                                const double* __restrict__ sc_s, const double* __restrict__ ereal,
                                const double* __restrict__ erec, double3 box, double3 binv, double rc2, double self,
                                double* __restrict__ out, int* __restrict__ flags)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    if (perm[s] < 0) {
        out[3 * s] = out[3 * s + 1] = out[3 * s + 2] = 0.0;
        return;
    }
    double e[3];
    for (int a = 0; a < 3; ++a)
        e[a] = ereal[3 * (size_t)s + a] + erec[3 * (size_t)s + a];
    double4 m0 = mp[3 * (size_t)s];
    e[0] += self * m0.y;
    e[1] += self * m0.z;
    e[2] += self * m0.w;
    double4 pi = pos_s[s], pari = par[s];
    for (int k = sc_ptr[s]; k < sc_ptr[s + 1]; ++k) {
        int j = sc_j[k];
        double sf = sc_s[k];
        double4 pj = pos_s[j], parj = par[j];
        double dx = mimg_fp64(pi.x - pj.x, box.x, binv.x), dy = mimg_fp64(pi.y - pj.y, box.y, binv.y),
               dz = mimg_fp64(pi.z - pj.z, box.z, binv.z);
        double r2 = dx * dx + dy * dy + dz * dz;
        bool in = r2 < rc2;
        double r = sqrt(r2);
        double rinv = 1.0 / r, rinv2 = rinv * rinv;
        double rinv3 = rinv * rinv2, rinv5 = rinv3 * rinv2, rinv7 = rinv5 * rinv2;
        double a = fmin(pari.w, parj.w);
        double u = r * pari.z * parj.z;
        double eps = a * u * u * u;
        double ex = exp(-eps);
        double l3 = 1.0 - ex, l5 = 1.0 - (1.0 + eps) * ex, l7 = 1.0 - (1.0 + eps + 0.6 * eps * eps) * ex;
        double f3 = in ? (1.0 - sf) * l3 : 1.0 - sf * l3;
        double f5 = in ? (1.0 - sf) * l5 : 1.0 - sf * l5;
        double f7 = in ? (1.0 - sf) * l7 : 1.0 - sf * l7;
        double b1 = -f3 * rinv3, b2 = -3.0 * f5 * rinv5, b3 = -15.0 * f7 * rinv7;
        double4 j0 = mp[3 * (size_t)j], j1 = mp[3 * (size_t)j + 1], j2 = mp[3 * (size_t)j + 2];
        double tdx = j1.x * dx + j1.y * dy + j1.z * dz;
        double tdy = j1.y * dx + j1.w * dy + j2.x * dz;
        double tdz = j1.z * dx + j2.x * dy + j2.y * dz;
        double tdd = tdx * dx + tdy * dy + tdz * dz;
        double dd = j0.y * dx + j0.z * dy + j0.w * dz;
        double rad = j0.x * b1 + b2 * dd + b3 * tdd / 3.0;
        double c2 = 2.0 * b2 / 3.0;
        e[0] += rad * dx - b1 * j0.y - c2 * tdx;
        e[1] += rad * dy - b1 * j0.z - c2 * tdy;
        e[2] += rad * dz - b1 * j0.w - c2 * tdz;
    }
    for (int a = 0; a < 3; ++a) {
        if (!isfinite(e[a]))
            atomicOr(flags, kFlagNonFinite);
        out[3 * (size_t)s + a] = e[a];
    }
}

void launch_perm_assemble(amoeba_ctx* c, double* out_slot, const double* scales)
{
    StageTimer tm(c, AMOEBA_T_PERM);
    double3 box = make_double3(c->prm.box[0], c->prm.box[1], c->prm.box[2]);
    double b = c->prm.ewald_alpha;
    double self = 4.0 * b * b * b / (3.0 * sqrt(kPi));
    hipLaunchKernelGGL(k_perm_assemble, dim3((c->npad + 255) / 256), dim3(256), 0, c->stream, c->npad, c->perm,
                       c->pos_s, c->par_d, (const double4*)c->mp_d, c->sc_ptr, c->sc_j, scales, c->ereal, c->erec,
                       box, make_double3(1.0 / box.x, 1.0 / box.y, 1.0 / box.z), c->prm.cutoff * c->prm.cutoff, self,
                       out_slot, c->flags);
}

}  // namespace amoeba
