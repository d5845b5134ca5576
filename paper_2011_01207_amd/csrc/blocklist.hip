// Blocked neighbour list of the real-space pair kernels (paper: "Neighbor list", "Box
// partitioning", "List filtering").
//
// Build (once per list):
//   1. atoms get a key along a column-serpentine cell order: the box is cut into ny x nz
//      columns along x whose cross-section holds about one block's worth of atoms per block
//      length, odd columns / odd z-slabs run backwards, so consecutive atoms stay spatially
//      adjacent across column ends; the atoms are ordered by key (with the atom index as
//      tie-break, so all distinct) through buckets of about two atoms, ranked within their
//      bucket, which gives a deterministic order;
//   2. the sorted order is cut into 64-atom blocks (one block = one wave64); the last block is
//      padded with phantom atoms;
//   3. every block gets a bounding box; block pairs whose boxes come within cutoff + buffer
//      are candidates (the adjacency of the paper's block matrix; each unordered pair once,
//      block I taking the J with J - I mod nb in 1 .. nb/2).  The blocks are binned by their
//      box centres into a grid whose cells are at least twice the largest half-extent plus
//      cutoff + buffer wide, so the candidates of a block lie in the 27 cells around its own;
//      a box too small for three cells per axis scans all blocks J = I + 1 .. I + nb/2;
//   4. list filtering: the atoms of candidate blocks that lie within cutoff + buffer of ANY
//      atom of block I are kept, in a fixed order (neighbour cell, J, slot; or J, slot), and
//      packed into 64-atom tiles; each block also owns its diagonal tile (I, I).
// Per configuration (every call that takes positions):
//   5. positions are gathered into slot order, checked for NaN and for list staleness, each
//      block gets an FP64 origin and FP32/FP64 offsets, and every tile gets its in-cutoff
//      bitmasks (bit k of row i: |r_i - r_jk| < rc) and the j positions relative to the
//      i-block origin, computed in FP64.
#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>

#include <type_traits>

#include "common.h"
#include "sort_key.h"

namespace amoeba {

__device__ __forceinline__ double mimg(double d, double L) { return mimg_fp64(d, L, 1.0 / L); }

// Sort key of atom a: column (cz, cy) in a serpentine order, then x within the column (also
// serpentine) quantised to kXBits bits (box / 4096, far below the block size); packed as
// col | xq.  Equal keys keep index order, so the order is deterministic.  The order is built from
// buckets key >> shift, at most one per slot (about two atoms each at an even density): k_sort_keys
// counts them and notes each atom's arrival in its bucket, k_sort_place writes the entries (key,
// atom) bucket by bucket, k_sort_rank ranks each entry among its bucket's.  These and a scan, five
// launches, take 34 us at 288,000 atoms, positions included; a merge sort took 21 launches and 135 us,
// the order and positions after it 18 us more.
// Non-finite positions go to a last bucket of their own, which is not ranked (the build reports them).
// A bucket may hold all atoms of a column within a few 4096ths of the box: with even matter the two
// above, with matter in a small part of a large box many, which the index alone then orders.  The
// ranking's time grows with the square of the largest bucket (about 4 ms for kRankMax atoms in one), so
// larger ones, which take a box of tens of thousands of Angstrom or all atoms in one place, are left in the
// order of arrival: a valid list where its capacity holds it, but not the same one every time.
// Also clears the build's error flags.
constexpr int kRankMax = 1 << 18;

__global__ void k_sort_keys(int n, const double* __restrict__ pos, double3 box, int ny, int nz, int shift,
                            int nbucket, unsigned* __restrict__ keys, int* __restrict__ arrival,
                            int* __restrict__ count, int* __restrict__ flags)
{
    int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a == 0)
        flags[0] = 0;
    if (a >= n)
        return;
    const unsigned key = sort_key(wrap_box(pos[3 * a], box.x), wrap_box(pos[3 * a + 1], box.y),
                                  wrap_box(pos[3 * a + 2], box.z), box.x, box.y, box.z, ny, nz);
    keys[a] = key;
    arrival[a] = atomicAdd(&count[bucket_of(key, shift, nbucket)], 1);
}

__global__ void k_sort_place(int n, int shift, int nbucket, const unsigned* __restrict__ keys,
                             const int* __restrict__ arrival, const int* __restrict__ start,
                             int* __restrict__ count, unsigned long long* __restrict__ entry)
{
    const int a = blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= n)
        return;
    const unsigned key = keys[a];
    const int b = bucket_of(key, shift, nbucket), r = arrival[a];
    entry[start[b] + r] = (unsigned long long)key << 32 | (unsigned)a;
    if (r == 0)
        count[b] = 0;  // the counters are zero between their uses
}

// The order (perm, slot), and each atom's position (wrapped into the box) at its slot, also as the
// reference of the staleness test.  Phantom slots (perm < 0) hold zeros.
__global__ __launch_bounds__(256) void k_sort_rank(int n, int npad, int shift, int nbucket,
                                                   const unsigned long long* __restrict__ entry,
                                                   const int* __restrict__ start, const double* __restrict__ pos,
                                                   double3 box, int* __restrict__ perm, int* __restrict__ slot,
                                                   double4* __restrict__ pos_s, double4* __restrict__ pos_ref,
                                                   int* __restrict__ flags)
{
    __shared__ int s_f;
    if (threadIdx.x == 0)
        s_f = 0;
    __syncthreads();
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p < npad) {
        int dst = p, a = -1;
        double x = 0.0, y = 0.0, z = 0.0;
        if (p < n) {
            const unsigned long long e = entry[p];
            const unsigned key = (unsigned)(e >> 32);
            a = (int)(unsigned)e;
            x = pos[3 * (size_t)a];
            y = pos[3 * (size_t)a + 1];
            z = pos[3 * (size_t)a + 2];
            const int b = bucket_of(key, shift, nbucket), s0 = start[b], s1 = start[b + 1];
            if (key != kKeyNonFinite && s1 - s0 <= kRankMax) {
                dst = s0;
                for (int q = s0; q < s1; ++q)
                    dst += entry[q] < e ? 1 : 0;
            }
            if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
                atomicOr(&s_f, kFlagNonFinite);
                x = y = z = 0.0;
            }
            x = wrap_box(x, box.x);
            y = wrap_box(y, box.y);
            z = wrap_box(z, box.z);
            slot[a] = dst;
        }
        perm[dst] = a;
        pos_s[dst] = pos_ref[dst] = make_double4(x, y, z, 0.0);
    }
    __syncthreads();
    if (threadIdx.x == 0 && s_f != 0)
        atomicOr(flags, s_f);
}

// Two-phase exclusive scan for long arrays: block sums (1024 per workgroup), then block-local
// scans, each offset by the sum of the block sums before it.
__global__ __launch_bounds__(256) void k_scan_blocksum(int n, const int* __restrict__ in, int* __restrict__ bsum)
{
    __shared__ int sh[256];
    int base = blockIdx.x * 1024, t = threadIdx.x;
    int s = 0;
    for (int u = 0; u < 4; ++u) {
        int i = base + t * 4 + u;
        s += i < n ? in[i] : 0;
    }
    sh[t] = s;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if (t < off)
            sh[t] += sh[t + off];
        __syncthreads();
    }
    if (t == 0)
        bsum[blockIdx.x] = sh[0];
}

__global__ __launch_bounds__(256) void k_scan_apply(int n, const int* __restrict__ in, const int* __restrict__ bsum,
                                                    int* __restrict__ out, int* __restrict__ total_copy)
{
    __shared__ int sh[256];
    __shared__ int s_boff;
    int base = blockIdx.x * 1024, t = threadIdx.x;
    {
        // this workgroup's offset: the sum of the block sums before it (fixed order)
        int b = 0;
        for (int k = t; k < (int)blockIdx.x; k += 256)
            b += bsum[k];
        sh[t] = b;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if (t < off)
                sh[t] += sh[t + off];
            __syncthreads();
        }
        if (t == 0)
            s_boff = sh[0];
        __syncthreads();
    }
    int v[4], s = 0;
    for (int u = 0; u < 4; ++u) {
        int i = base + t * 4 + u;
        v[u] = i < n ? in[i] : 0;
        s += v[u];
    }
    sh[t] = s;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        int y = t >= off ? sh[t - off] : 0;
        __syncthreads();
        sh[t] += y;
        __syncthreads();
    }
    int run = s_boff + sh[t] - s;
    for (int u = 0; u < 4; ++u) {
        int i = base + t * 4 + u;
        if (i < n)
            out[i] = run;
        run += v[u];
    }
    if (blockIdx.x == gridDim.x - 1 && t == 255) {
        out[n] = run;
        if (total_copy)
            *total_copy = run;
    }
}


// Per-slot parameters and the slot's count of scaled pairs (the CSR in slot order).  The Thole
// factor also goes into w of the dipole tiles' source copy pv (the vector kernels that fill it
// write x, y, z only), so that the tiles read a j atom's dipole and factor in one load.
template <typename R>
__global__ void k_params(int npad, const int* __restrict__ perm, const double* __restrict__ alpha,
                         const double* __restrict__ thole, double4* __restrict__ pd, float4* __restrict__ pf,
                         double* __restrict__ as, double* __restrict__ ais, const int* __restrict__ ptr_in,
                         int* __restrict__ cnt, R* __restrict__ pv)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    int a = perm[s];
    pv[4 * (size_t)s + 3] = a >= 0 ? (R)thole[a] : (R)0;
    cnt[s] = a >= 0 ? ptr_in[a + 1] - ptr_in[a] : 0;
    double al = a >= 0 ? alpha[a] : 1.0;
    double th = a >= 0 ? thole[a] : 0.0;
    double dinv = pow(al, -1.0 / 6.0);
    pd[s] = make_double4(al, 1.0 / al, dinv, th);
    as[s] = al;
    ais[s] = 1.0 / al;
    pf[s] = make_float4((float)al, (float)(1.0 / al), (float)dinv, (float)th);
}

// Single-workgroup exclusive scan: out[i] = sum_{k<i} in[i], out[n] = total.
// Exclusive scan of n values in one workgroup, out[n] = total (also written to *total_copy when
// given).
__global__ __launch_bounds__(1024) void k_scan_excl(int n, const int* __restrict__ in, int* __restrict__ out,
                                                    int* __restrict__ total_copy)
{
    // tiles of 4096: four consecutive values per thread (coalesced), a wave scan by shuffles,
    // the sixteen wave totals scanned by wave 0, and the running total carried across tiles
    __shared__ int wsum[16];
    __shared__ int carry_s;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int carry = 0;
    for (int base = 0; base < n; base += 4096) {
        int v[4], s = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + 4 * t + u;
            v[u] = i < n ? in[i] : 0;
            s += v[u];
        }
        int incl = s;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(incl, d);
            if (lane >= d)
                incl += y;
        }
        if (lane == 63)
            wsum[w] = incl;
        __syncthreads();
        if (w == 0) {
            const int x = lane < 16 ? wsum[lane] : 0;
            int wi = x;
#pragma unroll
            for (int d = 1; d < 16; d <<= 1) {
                const int y = __shfl_up(wi, d);
                if (lane >= d)
                    wi += y;
            }
            if (lane < 16)
                wsum[lane] = wi - x;   // exclusive over waves
            if (lane == 15)
                carry_s = wi;          // tile total
        }
        __syncthreads();
        int run = carry + wsum[w] + incl - s;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + 4 * t + u;
            if (i < n)
                out[i] = run;
            run += v[u];
        }
        carry += carry_s;
        __syncthreads();   // wsum and carry_s are rewritten by the next tile
    }
    if (t == 0) {
        out[n] = carry;
        if (total_copy)
            *total_copy = carry;
    }
}

__global__ void k_csr_fill(int npad, const int* __restrict__ perm, const int* __restrict__ slot,
                           const int* __restrict__ ptr_in, const int* __restrict__ j_in,
                           const double* __restrict__ s_in, const int* __restrict__ ptr_out,
                           int* __restrict__ j_out, double* __restrict__ s_out)
{
    int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    int a = perm[s];
    if (a < 0)
        return;
    int o = ptr_out[s];
    for (int k = ptr_in[a]; k < ptr_in[a + 1]; ++k, ++o) {
        j_out[o] = slot[j_in[k]];
        s_out[o] = s_in[k];
    }
}

// Block origin = FP64 position of the block's first atom; per-atom minimum-image offsets.  Called by
// all 64 lanes of a wave, lane l with slot l of one block (its position, and whether it is an atom);
// returns the lane's offset.
__device__ __forceinline__ double lane0(double v)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                            __builtin_amdgcn_readfirstlane(__double2loint(v)));
}

__device__ __forceinline__ double3 block_frame(int s, bool real, double x, double y, double z, double3 box,
                                               double4* __restrict__ org, double4* __restrict__ off_d,
                                               float4* __restrict__ off_f)
{
    const double ox = lane0(x), oy = lane0(y), oz = lane0(z);
    if ((s & (kBlock - 1)) == 0)
        org[s / kBlock] = make_double4(ox, oy, oz, 0.0);
    double dx = 0.0, dy = 0.0, dz = 0.0;
    if (real) {
        dx = mimg(x - ox, box.x);
        dy = mimg(y - oy, box.y);
        dz = mimg(z - oz, box.z);
    }
    off_d[s] = make_double4(dx, dy, dz, 0.0);
    off_f[s] = make_float4((float)dx, (float)dy, (float)dz, 0.0f);
    return make_double3(dx, dy, dz);
}

// Caller positions into slot order (one thread per slot: the slot's reads and writes are
// coalesced, the only scattered access is the read of its atom's caller-order position), wrapped
// into the box; flags NaN/Inf, a changed configuration and (if a reference exists) atoms that
// moved more than buffer/2 since the list build.  Phantom slots (perm < 0) hold zeros.  A wave's 64
// slots are a block, whose frame is written along (block_frame).
// Flags go to one device word that every workgroup may set; same-address device atomics are
// serialized, so each workgroup ORs its flags in LDS first and issues at most one atomic, and
// the grid is capped at kScatterWG workgroups (grid-stride loop).
constexpr int kScatterWG = 1024;

__global__ __launch_bounds__(256) void k_gather_pos(int npad, const int* __restrict__ perm,
                                                    const double* __restrict__ pos, double3 box,
                                                    double4* __restrict__ pos_s, const double4* __restrict__ ref,
                                                    double half_buf2, int* __restrict__ flags,
                                                    double4* __restrict__ org, double4* __restrict__ off_d,
                                                    float4* __restrict__ off_f)
{
    __shared__ int s_f;
    if (threadIdx.x == 0)
        s_f = 0;
    __syncthreads();
    int f = 0;
    // four slots per thread and round, every round's loads issued before they are used (the
    // caller-order reads wait on the slot's atom index)
    constexpr int U = 4;
    const int stride = gridDim.x * blockDim.x;
    for (int s0 = blockIdx.x * blockDim.x + threadIdx.x; s0 < npad; s0 += U * stride) {
        int a[U];
        double4 old[U], r0[U];
        double p[U][3];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u * stride;
            a[u] = s < npad ? perm[s] : -1;
            old[u] = s < npad ? pos_s[s] : make_double4(0.0, 0.0, 0.0, 0.0);
            r0[u] = (ref && s < npad) ? ref[s] : make_double4(0.0, 0.0, 0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                p[u][k] = a[u] >= 0 ? pos[3 * (size_t)a[u] + k] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + u * stride;
            if (s >= npad)
                break;
            double x = 0.0, y = 0.0, z = 0.0;
            if (a[u] >= 0) {
                x = p[u][0];
                y = p[u][1];
                z = p[u][2];
                if (!isfinite(x) || !isfinite(y) || !isfinite(z)) {
                    f |= kFlagNonFinite;
                    x = y = z = 0.0;
                }
                x = wrap_box(x, box.x);
                y = wrap_box(y, box.y);
                z = wrap_box(z, box.z);
                if (old[u].x != x || old[u].y != y || old[u].z != z)
                    f |= kFlagChanged;
                if (ref) {
                    const double dx = mimg(x - r0[u].x, box.x), dy = mimg(y - r0[u].y, box.y),
                                 dz = mimg(z - r0[u].z, box.z);
                    if (dx * dx + dy * dy + dz * dz > half_buf2)
                        f |= kFlagStale;
                }
            }
            pos_s[s] = make_double4(x, y, z, 0.0);
            block_frame(s, a[u] >= 0, x, y, z, box, org, off_d, off_f);
        }
    }
    if (f != 0)
        atomicOr(&s_f, f);
    __syncthreads();
    if (threadIdx.x == 0 && s_f != 0)
        atomicOr(flags, s_f);
}

// Frame of each block, and its bounding box in coordinates unwrapped around its first atom (one
// block per wave).
__global__ __launch_bounds__(256) void k_bbox(int nb, const int* __restrict__ perm,
                                              const double4* __restrict__ pos_s, double3 box,
                                              double4* __restrict__ bc, double4* __restrict__ bh,
                                              double4* __restrict__ org, double4* __restrict__ off_d,
                                              float4* __restrict__ off_f)
{
    const int lane = threadIdx.x & 63;
    const int I = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (I >= nb)
        return;
    int s = I * kBlock + lane;
    const double4 p = pos_s[s];
    const double4 o = make_double4(lane0(p.x), lane0(p.y), lane0(p.z), 0.0);
    const double3 r = block_frame(s, perm[s] >= 0, p.x, p.y, p.z, box, org, off_d, off_f);
    const double rx = r.x, ry = r.y, rz = r.z;
    double mnx = rx, mny = ry, mnz = rz, mxx = rx, mxy = ry, mxz = rz;
    for (int off = 32; off > 0; off >>= 1) {
        mnx = fmin(mnx, __shfl_xor(mnx, off));
        mny = fmin(mny, __shfl_xor(mny, off));
        mnz = fmin(mnz, __shfl_xor(mnz, off));
        mxx = fmax(mxx, __shfl_xor(mxx, off));
        mxy = fmax(mxy, __shfl_xor(mxy, off));
        mxz = fmax(mxz, __shfl_xor(mxz, off));
    }
    if (lane == 0) {
        const double hx = 0.5 * (mxx - mnx), hy = 0.5 * (mxy - mny), hz = 0.5 * (mxz - mnz);
        bc[I] = make_double4(o.x + 0.5 * (mnx + mxx), o.y + 0.5 * (mny + mxy), o.z + 0.5 * (mnz + mxz), 0.0);
        bh[I] = make_double4(hx, hy, hz, 0.0);
    }
}

// Exclusive prefix sum over the 64 lanes of a wave (all lanes active) and the wave total, by
// data-parallel primitives: shifts by 1, 2, 4, 8 lanes within each row of 16, then row 0's total
// into row 1 and row 2's into row 3 (broadcast of lane 15 of the row before), then the first two
// rows' total into rows 2 and 3 (broadcast of lane 31).  Lanes a shift or broadcast does not
// reach add 0.
__device__ __forceinline__ int wave_excl_scan_i(int x, int& total)
{
    int v = x;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 -> rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 -> rows 2, 3
    total = __builtin_amdgcn_readlane(v, 63);
    return v - x;
}

// Block grid of the candidate search.  grid[0] = 1 when it is used, grid[1..3] = cells per
// axis.  A cell is at least 2 h_max + rcb (+ a margin) wide on every axis, h_max the largest
// block half-extent on that axis, so two blocks whose boxes come within rcb have centres
// closer than one cell (periodically) and sit in the same or adjacent cells; with three or more
// cells per axis the 27 cells around a block are distinct.
constexpr double kCellMargin = 0.01;  // A

__device__ __forceinline__ int cell_of(double v, double L, int n)
{
    // rounding may take a centre at a cell's face to the cell beside it: the width's margin covers that
    const double f = v * (1.0 / L), y = (f - floor(f)) * (double)n;
    const int c = (y == y) ? (int)y : 0;  // a non-finite centre (reported by the build) goes to cell 0
    return min(max(c, 0), n - 1);
}

// One workgroup: the largest half-extent per axis (ext_out, read by the host after the build), the
// grid shape, and the blocks counted into cells: cell_start[c] = first entry of cell c.  The
// counters (at most kGridCells cells) are in LDS; `entry` keeps each block's cell and arrival there,
// `unranked` the blocks cell by cell, which k_cell_rank puts in index order within their cell.
// 10 and 5 us for 4,500 blocks; a merge sort of the cells and a search for their starts took eight
// launches and 30 us.
constexpr int kGridCells = 12288;

__global__ __launch_bounds__(1024) void k_block_grid(int nb, const double4* __restrict__ bc,
                                                     const double4* __restrict__ bh, double3 box, double rcb,
                                                     int3 ncap, double* __restrict__ ext_out,
                                                     int* __restrict__ grid, int2* __restrict__ entry,
                                                     int* __restrict__ unranked, int* __restrict__ cell_start)
{
    __shared__ double s_m[3][16];
    __shared__ int s_n[4];
    __shared__ int s_w[16];
    __shared__ int s_cnt[kGridCells];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    double m[3] = {0.0, 0.0, 0.0};
    constexpr int U = 4;  // blocks per thread and round, their loads in flight together
    for (int b0 = tid; b0 < nb; b0 += U * 1024) {
        double4 h[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            h[u] = bh[min(b0 + u * 1024, nb - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            m[0] = fmax(m[0], h[u].x);
            m[1] = fmax(m[1], h[u].y);
            m[2] = fmax(m[2], h[u].z);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int off = 32; off > 0; off >>= 1)
            m[a] = fmax(m[a], __shfl_xor(m[a], off));
        if (lane == 0)
            s_m[a][w] = m[a];
    }
    __syncthreads();
    if (tid == 0) {
        const double L[3] = {box.x, box.y, box.z};
        const int cap[3] = {ncap.x, ncap.y, ncap.z};
        bool use = true;
        for (int a = 0; a < 3; ++a) {
            double e = 0.0;
            for (int k = 0; k < 16; ++k)
                e = fmax(e, s_m[a][k]);
            ext_out[a] = e;
            const double cells = floor(L[a] / (2.0 * e + rcb + kCellMargin));
            const int nc = cells >= (double)cap[a] ? cap[a] : (int)fmax(cells, 1.0);
            grid[1 + a] = s_n[1 + a] = nc;
            use = use && nc >= 3;
        }
        grid[0] = s_n[0] = use ? 1 : 0;
    }
    __syncthreads();
    if (!s_n[0])
        return;
    const int nx = s_n[1], ny = s_n[2], nz = s_n[3], ncell = nx * ny * nz;
    for (int k = tid; k < ncell; k += 1024)
        s_cnt[k] = 0;
    __syncthreads();
    for (int b0 = tid; b0 < nb; b0 += U * 1024) {
        double4 c[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            c[u] = bc[min(b0 + u * 1024, nb - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + u * 1024;
            if (b < nb) {
                const int key = (cell_of(c[u].z, box.z, nz) * ny + cell_of(c[u].y, box.y, ny)) * nx +
                                cell_of(c[u].x, box.x, nx);
                entry[b] = make_int2(key, atomicAdd(&s_cnt[key], 1));
            }
        }
    }
    __syncthreads();
    // exclusive scan of the counters, thread t holding P consecutive ones
    const int P = (ncell + 1023) / 1024;
    int sum = 0;
    for (int u = 0; u < P; ++u)
        sum += tid * P + u < ncell ? s_cnt[tid * P + u] : 0;
    int tot;
    const int ex = wave_excl_scan_i(sum, tot);
    if (lane == 0)
        s_w[w] = tot;
    __syncthreads();
    int run = ex;
    for (int k = 0; k < w; ++k)
        run += s_w[k];
    for (int u = 0; u < P; ++u)
        if (tid * P + u < ncell) {
            const int v = s_cnt[tid * P + u];
            s_cnt[tid * P + u] = run;
            cell_start[tid * P + u] = run;
            run += v;
        }
    if (tid == 0)
        cell_start[ncell] = nb;
    __syncthreads();
    for (int b0 = tid; b0 < nb; b0 += U * 1024) {
        int2 e[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            e[u] = entry[min(b0 + u * 1024, nb - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b0 + u * 1024 < nb)
                unranked[s_cnt[e[u].x] + e[u].y] = b0 + u * 1024;
    }
}

__global__ void k_cell_rank(int nb, const int* __restrict__ grid, const int2* __restrict__ entry,
                            const int* __restrict__ unranked, const int* __restrict__ cell_start,
                            int* __restrict__ cell_blk)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= nb || !grid[0])
        return;
    const int key = entry[b].x, s0 = cell_start[key], s1 = cell_start[key + 1];
    int dst = s0;
#pragma unroll 4
    for (int q = s0; q < s1; ++q)
        dst += unranked[q] < b ? 1 : 0;
    cell_blk[dst] = b;
}

// Position of the r-th set bit (from 0) of m, r < popcount(m).
__device__ __forceinline__ int nth_set_bit(unsigned long long m, int r)
{
    unsigned v = (unsigned)m;
    int base = 0, c = __popc(v);
    if (r >= c) {
        r -= c;
        v = (unsigned)(m >> 32);
        base = 32;
    }
#pragma unroll
    for (int width = 16; width >= 1; width >>= 1) {
        c = __popc(v & ((1u << width) - 1u));
        if (r >= c) {
            r -= c;
            v >>= width;
            base += width;
        }
    }
    return base;
}

// List filtering: for block I, the atoms of the blocks J with J - I mod nb = d in 1 .. nb/2
// (d = nb/2 only for I < nb/2) that lie within rcb of any atom of I.  Every unordered block
// pair is examined exactly once.  The candidate blocks J are those of the 27 grid cells around
// I's cell (k_block_grid), in (cell, J) order, or all J = I + 1 .. I + nb/2 in d order when
// the grid is not used.  Each thread tests one block's bounding box; the ones within reach are
// collected, in order, until a round of boxes might not fit any more (most blocks: once), and a wave
// takes one candidate at a time: lane l holds its atom l, atoms out of reach of I's box drop out, and
// the squared distances of 16 of them at a time to the 64 atoms of I are four matrix instructions,
// |q|^2 + (-2 q, 1) . (j, |j|^2), taken to the least over I's atoms.  The filter only has to keep a
// superset, the masks of every configuration decide at rc in FP64: the reach has a margin of 1e-3 A, or
// twice the rounding of a component of the difference form where that is more (offsets in thousands of
// A).  The matrix form cancels: with S >= |q|^2 + |j|^2 its rounding is below S 2^-19 (as in
// k_tile_refresh), and where that is above the margin, or the minimum image is needed (twice the
// largest half-extent plus rcb reaches half an edge), the block's pairs are taken as differences on the
// vector units: blocks of some 70 A and more, in dilute systems or across a void.  The kept atoms are
// written at offsets from an ordered scan, so the list does not depend on scheduling, and counted for
// the reverse index.
// 76 us for 4,500 blocks; testing the queued atoms one per thread against the block's atoms on the
// vector units, in rounds of 256 boxes, took 163 us.
constexpr int kFiltCap = 512;  // candidates of a round

typedef float f4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256, 6) void k_filter(int nb, int n, const double4* __restrict__ pos_s,
                                                const double4* __restrict__ bc, const double4* __restrict__ bh,
                                                const double* __restrict__ ext_in, const int* __restrict__ grid,
                                                const int* __restrict__ cell_blk,
                                                const int* __restrict__ cell_start, double3 box, double3 binv,
                                                double rcb, int* __restrict__ row_count, int* __restrict__ row_j,
                                                int* __restrict__ tpb, int* __restrict__ rev_cnt,
                                                int* __restrict__ flags)
{
    __shared__ float4 s_i[kBlock];                      // i atoms relative to the block centre, w = |.|^2
    __shared__ __align__(16) float s_j[4][4 * kBlock];  // each wave's candidate, likewise
    __shared__ unsigned long long s_keep[kFiltCap];     // kept atoms of each candidate
    __shared__ int s_cand[kFiltCap];
    __shared__ int s_off[kFiltCap + 1];
    __shared__ int s_wn[4];
    __shared__ int s_cs[27], s_cp[28];                  // neighbour cells: first entry, prefix of sizes
    const int I = blockIdx.x, tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const double4 ci = bc[I], hi = bh[I];
    const bool cells = grid[0] != 0;
    if (cells && tid < 27) {
        const int nx = grid[1], ny = grid[2], nz = grid[3];
        const int cx = cell_of(ci.x, box.x, nx), cy = cell_of(ci.y, box.y, ny), cz = cell_of(ci.z, box.z, nz);
        int x = cx + tid % 3 - 1, y = cy + (tid / 3) % 3 - 1, z = cz + tid / 9 - 1;
        x += x < 0 ? nx : (x >= nx ? -nx : 0);
        y += y < 0 ? ny : (y >= ny ? -ny : 0);
        z += z < 0 ? nz : (z >= nz ? -nz : 0);
        const int c = (z * ny + y) * nx + x;
        const int a = cell_start[c];
        s_cs[tid] = a;
        s_cp[tid + 1] = cell_start[c + 1] - a;
    }
    if (tid < kBlock) {
        const int si = I * kBlock + tid;
        const double4 pi = pos_s[si];
        const float x = (float)mimg_fp64(pi.x - ci.x, box.x, binv.x), y = (float)mimg_fp64(pi.y - ci.y, box.y, binv.y),
                    z = (float)mimg_fp64(pi.z - ci.z, box.z, binv.z);
        // a phantom slot is far from everything
        s_i[tid] = si < n ? make_float4(x, y, z, x * x + y * y + z * z) : make_float4(0.0f, 0.0f, 0.0f, 1e30f);
    }
    const float Lx = (float)box.x, Ly = (float)box.y, Lz = (float)box.z;
    const float Lix = (float)binv.x, Liy = (float)binv.y, Liz = (float)binv.z;
    // largest block half-extents; pair offsets |q - j| <= h_I + (h_I + rcb + margins) <= 2 h_max + rcb
    const double ext[3] = {ext_in[0], ext_in[1], ext_in[2]};
    const bool mi = !(2.0 * ext[0] + rcb + 0.01 < 0.5 * box.x && 2.0 * ext[1] + rcb + 0.01 < 0.5 * box.y &&
                      2.0 * ext[2] + rcb + 0.01 < 0.5 * box.z);
    // a component of a difference of FP32 offsets, each up to D, is off by at most 2 D 2^-24, and by
    // 3 edges' 2^-24 more where an image is taken off; the distance by less than twice that
    const float D = 2.0f * (float)fmax(ext[0], fmax(ext[1], ext[2])) + (float)rcb;
    const float margin = fmaxf(1e-3f, (2.0f * D + (mi ? 3.0f * fmaxf(Lx, fmaxf(Ly, Lz)) : 0.0f)) * 1.1920929e-7f);
    const double rcb2 = rcb * rcb;
    const float rf2 = (float)((rcb + margin) * (rcb + margin));
    const float hxf = (float)hi.x + margin, hyf = (float)hi.y + margin, hzf = (float)hi.z + margin;
    const float reach = (float)rcb + margin, Jx = hxf + reach, Jy = hyf + reach, Jz = hzf + reach;
    const float S = hxf * hxf + hyf * hyf + hzf * hzf + Jx * Jx + Jy * Jy + Jz * Jz;
    const bool direct = mi || !(S * 1.9073486e-6f < 2.0f * margin * (float)rcb);
    const int dmax = (nb % 2 == 0 && I < nb / 2) ? nb / 2 : (nb - 1) / 2;
    __syncthreads();
    if (cells && w == 0) {
        int tot;
        const int v = lane < 27 ? s_cp[lane + 1] : 0;
        const int ex = wave_excl_scan_i(v, tot);
        if (lane < 27)
            s_cp[lane + 1] = ex + v;
        if (lane == 0)
            s_cp[0] = 0;
    }
    // the matrix operands of the block's atoms: row lr of tile m is atom 16 m + lr, column lg its
    // component; the accumulator's register v of tile m starts at |q|^2 of atom 16 m + 4 lg + v
    const int lr = lane & 15, lg = lane >> 4;
    float qa[4];
    f4 qq[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const float4 q = s_i[16 * m + lr];
        qa[m] = lg == 3 ? 1.0f : -2.0f * (lg == 0 ? q.x : lg == 1 ? q.y : q.z);
#pragma unroll
        for (int v = 0; v < 4; ++v)
            qq[m][v] = s_i[16 * m + 4 * lg + v].w;
    }
    __syncthreads();
    const int ncand = cells ? s_cp[27] : dmax;
    int count = 0;
    for (int g0 = 0; g0 < ncand;) {
        int nc = 0;
        for (; g0 < ncand && nc + 256 <= kFiltCap; g0 += 256) {
            const int g = g0 + tid;
            int J = 0;
            bool inwin = false;
            if (g < ncand) {
                if (cells) {
                    int lo = 0, up = 26;  // the last cell whose entries start at or before g
                    while (lo < up) {
                        const int mid = (lo + up + 1) >> 1;
                        if (s_cp[mid] <= g)
                            lo = mid;
                        else
                            up = mid - 1;
                    }
                    J = cell_blk[s_cs[lo] + g - s_cp[lo]];
                    const int d = J - I + (J < I ? nb : 0);
                    inwin = d >= 1 && d <= dmax;
                } else {
                    J = I + 1 + g;
                    J -= J >= nb ? nb : 0;
                    inwin = true;
                }
            }
            bool cand = false;
            if (inwin) {
                const double4 cj = bc[J], hj = bh[J];
                double dx = fabs(mimg_fp64(ci.x - cj.x, box.x, binv.x)) - hi.x - hj.x;
                double dy = fabs(mimg_fp64(ci.y - cj.y, box.y, binv.y)) - hi.y - hj.y;
                double dz = fabs(mimg_fp64(ci.z - cj.z, box.z, binv.z)) - hi.z - hj.z;
                dx = fmax(dx, 0.0);
                dy = fmax(dy, 0.0);
                dz = fmax(dz, 0.0);
                cand = dx * dx + dy * dy + dz * dz < rcb2;
            }
            const unsigned long long cm = __ballot(cand);
            if (lane == 0)
                s_wn[w] = __popcll(cm);
            __syncthreads();
            const int wbase = nc + (w > 0 ? s_wn[0] : 0) + (w > 1 ? s_wn[1] : 0) + (w > 2 ? s_wn[2] : 0);
            if (cand)
                s_cand[wbase + __popcll(cm & ((1ull << lane) - 1ull))] = J;
            nc += s_wn[0] + s_wn[1] + s_wn[2] + s_wn[3];
            __syncthreads();
        }
        double4 next = pos_s[w < nc ? s_cand[w] * kBlock + lane : 0];
        for (int k = w; k < nc; k += 4) {
            const double4 pj = next;
            const bool real = s_cand[k] * kBlock + lane < n;
            if (k + 4 < nc)
                next = pos_s[s_cand[k + 4] * kBlock + lane];
            const float jx = (float)mimg_fp64(pj.x - ci.x, box.x, binv.x);
            const float jy = (float)mimg_fp64(pj.y - ci.y, box.y, binv.y);
            const float jz = (float)mimg_fp64(pj.z - ci.z, box.z, binv.z);
            const float bx = fmaxf(fabsf(jx) - hxf, 0.0f), by = fmaxf(fabsf(jy) - hyf, 0.0f),
                        bz = fmaxf(fabsf(jz) - hzf, 0.0f);
            // an atom outside the reach of the block's box is outside that of every atom in it
            const bool inb = real && bx * bx + by * by + bz * bz < rf2;
            const unsigned long long m = __ballot(inb);
            unsigned long long near = 0ull;
            if (direct) {
                if (m) {
                    float r2 = 3e38f;
#pragma unroll 4
                    for (int i = 0; i < kBlock; ++i) {
                        const float4 q = s_i[i];
                        float dx = q.x - jx, dy = q.y - jy, dz = q.z - jz;
                        dx -= Lx * rintf(dx * Lix);
                        dy -= Ly * rintf(dy * Liy);
                        dz -= Lz * rintf(dz * Liz);
                        const float d2 = dx * dx + dy * dy + dz * dz;
                        r2 = fminf(r2, q.w < 1e30f ? d2 : 3e38f);
                    }
                    near = __ballot(r2 < rf2);
                }
            } else if (m) {
                float* sj = &s_j[w][4 * lane];
                sj[0] = jx;
                sj[1] = jy;
                sj[2] = jz;
                sj[3] = jx * jx + jy * jy + jz * jz;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    if (!((m >> (16 * t)) & 0xffffull))
                        continue;
                    const float b = s_j[w][4 * (16 * t + lr) + lg];
                    float r2 = 3e38f;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const f4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(qa[u], b, qq[u], 0, 0, 0);
                        r2 = fminf(r2, fminf(fminf(d[0], d[1]), fminf(d[2], d[3])));
                    }
                    unsigned long long hit = __ballot(r2 < rf2);  // lane (lr, lg): atom 16 t + lr
                    hit |= hit >> 32;
                    hit |= hit >> 16;
                    near |= (hit & 0xffffull) << (16 * t);
                }
                __builtin_amdgcn_wave_barrier();
            }
            if (lane == 0)
                s_keep[k] = near & m;
        }
        __syncthreads();
        {
            // ordered exclusive scan of the kept counts (thread t holds candidates 2t and 2t + 1)
            const int k = 2 * tid;
            const int n0 = k < nc ? __popcll(s_keep[k]) : 0, n1 = k + 1 < nc ? __popcll(s_keep[k + 1]) : 0;
            int tot;
            const int ex = wave_excl_scan_i(n0 + n1, tot);
            if (lane == 0)
                s_wn[w] = tot;
            __syncthreads();
            const int wbase = (w > 0 ? s_wn[0] : 0) + (w > 1 ? s_wn[1] : 0) + (w > 2 ? s_wn[2] : 0);
            s_off[k] = wbase + ex;
            s_off[k + 1] = wbase + ex + n0;
            if (tid == 255)
                s_off[kFiltCap] = wbase + tot;
        }
        __syncthreads();
        for (int k = w; k < nc; k += 4) {
            const unsigned long long km = s_keep[k];
            if ((km >> lane) & 1ull) {
                const int pos = count + s_off[k] + __popcll(km & ((1ull << lane) - 1ull));
                if (pos < kMaxFiltered) {
                    const int sj = s_cand[k] * kBlock + lane;
                    row_j[(size_t)I * kMaxFiltered + pos] = sj;
                    atomicAdd(&rev_cnt[sj], 1);
                }
            }
        }
        count += s_off[kFiltCap];
        __syncthreads();
    }
    if (tid == 0) {
        const int kept = min(count, kMaxFiltered);
        row_count[I] = kept;
        tpb[I] = 1 + (kept + kBlock - 1) / kBlock;  // the diagonal tile and the filtered j-atoms
        if (count > kMaxFiltered)
            atomicOr(flags, kFlagFilterOverflow);
    }
}

// The tiles of block I (a workgroup): its diagonal tile and its filtered j-atoms, and their entries
// (tile, lane) in the reverse index: for every slot those where it is a j-atom, in the order the
// counters' atomics give (the sums over them do not depend on it: exact fixed point in mixed
// precision, see JSum).  Does nothing when the tiles exceed the arrays (the host then launches it
// again).
__global__ __launch_bounds__(256) void k_fill_tiles(int nb, int tile_cap, const int* __restrict__ tile0,
                                                    const int* __restrict__ row_count,
                                                    const int* __restrict__ row_j, const int* __restrict__ rev_ptr,
                                                    int* __restrict__ rev_cnt, int* __restrict__ tile_blk,
                                                    int* __restrict__ tile_j, int* __restrict__ rev_idx)
{
    if (tile0[nb] > tile_cap)
        return;
    const int I = blockIdx.x, t0 = tile0[I], nt = tile0[I + 1] - t0, cnt = row_count[I];
    for (int t = threadIdx.x; t < nt; t += 256)
        tile_blk[t0 + t] = I;
    for (int e = threadIdx.x; e < nt * kBlock; e += 256) {
        const int r = e - kBlock;
        int sj = I * kBlock + e;  // diagonal tile
        if (r >= 0) {
            sj = r < cnt ? row_j[(size_t)I * kMaxFiltered + r] : -1;
            if (sj >= 0)  // the counter counts down from the slot's count: zero again afterwards
                rev_idx[rev_ptr[sj] + atomicSub(&rev_cnt[sj], 1) - 1] = t0 * kBlock + e;
        }
        tile_j[(size_t)t0 * kBlock + e] = sj;
    }
}

// Per configuration: in-cutoff bitmasks (strict r < rc, decided as in FP64) and j positions
// relative to the i-block origin.  The diagonal tile keeps only k > i.  One tile per wave.
// The squared distances less rc^2 of 16 i-atoms to the 64 j-atoms are four FP32 matrix
// instructions, |j|^2 - rc^2 + (-2 j, 1) . (q, |q|^2): lane (lr, lg) then holds those of i-atom
// 16 t + lr to the j-atoms 16 m + 4 lg + v, shifts their signs into 16 bits and takes the least
// magnitude of either sign (two vector instructions a pair); an exchange through LDS and a transpose of
// 4 x 4 groups of four bits make them rows.  With S >= |q|^2 + |j|^2 the offsets' rounding moves a
// squared distance by at most 4 S 2^-24, that of the squares and of the five sums by less than
// 28 S 2^-24 (also if they are cut off): where the least magnitude is above S 2^-19, every sign is
// that of the exact value.  Otherwise (one tile in ten or so) the 16 i-atoms' pairs are classified
// anew from the differences of their FP32 offsets, and those near rc^2 by the FP64 distance, so every
// bit equals the FP64 test.  Near is within a relative 1e-5, or 4 rc d where that is more (dilute
// systems), d = 2^-24 (2 sqrt(S/2) + 3 edges with MI) bounding the rounding of a component of a difference.
// MI: minimum image per pair offset, all pairs classified from the differences; without it the
// block-relative offsets are used as they are (valid when the list build proved that no tile offset
// can reach half the box, as for the pair kernels).
// 54 us for 42,600 tiles (69 us with a vector subtraction and comparison per pair and component).
__device__ __forceinline__ unsigned long long transpose_nibbles(unsigned long long x)
{
    unsigned long long y = (x ^ (x >> 12)) & 0x0000f0f00000f0f0ull;
    x ^= y ^ (y << 12);
    y = (x ^ (x >> 24)) & 0x00000000ff00ff00ull;
    return x ^ y ^ (y << 24);
}

// largest of a wave's non-negative floats (their order is that of their bits)
__device__ __forceinline__ float wave_max_pos(float x)
{
    int v = __float_as_int(x);
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));  // row_bcast:15, :31
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));
    return __int_as_float(__builtin_amdgcn_readlane(v, 63));
}

template <typename R, bool MI>
__global__ __launch_bounds__(256, 6) void k_tile_refresh(int ntiles, int ngroup, const int* __restrict__ tile_blk,
                                                      const int* __restrict__ tile_j, int n,
                                                      const double4* __restrict__ pos_s,
                                                      const double4* __restrict__ org,
                                                      const float4* __restrict__ off_f,
                                                      const typename V4<R>::T* __restrict__ par, double3 box,
                                                      double3 binv, double rc2,
                                                      unsigned long long* __restrict__ mask,
                                                      typename V4<R>::T* __restrict__ jrel,
                                                      int* __restrict__ tile_np, int* __restrict__ tile_rows,
                                                      uint16_t* __restrict__ walk,
                                                      unsigned long long* __restrict__ pair_part,
                                                      const int* __restrict__ flags)
{
    // launched ahead of the host's look at the flags: only for a changed and valid configuration
    if (flags && (flags[0] & (kFlagChanged | kFlagNonFinite | kFlagStale)) != kFlagChanged)
        return;
    using R4 = typename V4<R>::T;
    __shared__ __align__(16) float s_i[4][4 * kBlock];  // i offsets and |.|^2
    __shared__ __align__(16) float s_j[4][4 * kBlock];  // j likewise
    __shared__ __align__(16) float s_jn[4][kBlock];     // |j|^2 - rc^2
    __shared__ uint16_t s_p[4][4 * kBlock];
    __shared__ unsigned long long s_cnt[4];
    __shared__ unsigned long long s_m[4][kBlock];
    __shared__ int s_off[4][kBlock];
    // one tile per wave: its index and everything derived from it are wave-uniform
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int group = blockIdx.x; group < ngroup; group += gridDim.x) {
        const int t = group * 4 + w;
        const bool act = t < ntiles;
        const int I = act ? tile_blk[t] : 0;
        const int si = I * kBlock + lane;
        const int sj = act ? tile_j[(size_t)t * kBlock + lane] : -1;
        unsigned long long m = 0;
        int P = 0;
        if (act) {  // uniform: one tile per wave
            const double4 o = org[I];
            const bool jvalid = sj >= 0 && sj < n;
            const double4 pj = sj >= 0 ? pos_s[sj] : o;
            const R wj = sj >= 0 ? par[sj].z : (R)0;  // the j atom's polarizability factor
            const float4 oi = off_f[si];
            const double jx = mimg_fp64(pj.x - o.x, box.x, binv.x), jy = mimg_fp64(pj.y - o.y, box.y, binv.y),
                         jz = mimg_fp64(pj.z - o.z, box.z, binv.z);
            jrel[(size_t)t * kBlock + lane] = R4{(R)jx, (R)jy, (R)jz, wj};
            const float rcf = (float)rc2;
            const float Lx = (float)box.x, Ly = (float)box.y, Lz = (float)box.z;
            const float Lix = (float)binv.x, Liy = (float)binv.y, Liz = (float)binv.z;
            // absent atoms (no i-atom, no j-atom, phantom slots) lie at the origin with a square that
            // puts every sum with them far out of reach
            constexpr float kFar = 1e30f;
            const float qx = (float)jx, qy = (float)jy, qz = (float)jz;
            const float jn = qx * qx + qy * qy + qz * qz, in2 = oi.x * oi.x + oi.y * oi.y + oi.z * oi.z;
            const bool ivalid = si < n;
            float* wi = &s_i[w][4 * lane];
            wi[0] = ivalid ? oi.x : 0.0f;
            wi[1] = ivalid ? oi.y : 0.0f;
            wi[2] = ivalid ? oi.z : 0.0f;
            wi[3] = ivalid ? in2 : kFar;
            float* wp = &s_j[w][4 * lane];
            wp[0] = jvalid ? qx : 0.0f;
            wp[1] = jvalid ? qy : 0.0f;
            wp[2] = jvalid ? qz : 0.0f;
            wp[3] = jvalid ? jn : kFar;
            s_jn[w][lane] = jvalid ? jn - rcf : kFar;
            // S: twice the largest square of the tile
            const float M = wave_max_pos(fmaxf(ivalid ? in2 : 0.0f, jvalid ? jn : 0.0f));
            const float thr = M * 3.814697265625e-6f;  // 2^-18
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int lr = lane & 15, lg = lane >> 4;
            float ja[4];
            f4 jq[4];
            if constexpr (!MI) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    ja[k] = lg == 3 ? 1.0f : -2.0f * s_j[w][4 * (16 * k + lr) + lg];
                    jq[k] = *(const f4*)&s_jn[w][16 * k + 4 * lg];
                }
            }
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                unsigned bits = 0;
                bool redo = MI;
                if constexpr (!MI) {
                    const float b = s_i[w][4 * (16 * tt + lr) + lg];
                    // the bits of the least positive value, and those of the negative one nearest to 0
                    // (a positive value's bits are the smaller the less it is; a negative one's, as a
                    // signed number, too)
                    unsigned above = __float_as_uint(kFar);
                    int below = __float_as_int(-kFar);
#pragma unroll
                    for (int k = 3; k >= 0; --k) {
                        const f4 d = __builtin_amdgcn_mfma_f32_16x16x4f32(ja[k], b, jq[k], 0, 0, 0);
#pragma unroll
                        for (int v = 3; v >= 0; --v)  // bits << 1 | sign of d
                            bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(d[v]), 31);
#pragma unroll
                        for (int v = 0; v < 4; v += 2) {
                            above = min(above, min(__float_as_uint(d[v]), __float_as_uint(d[v + 1])));
                            below = min(below, min(__float_as_int(d[v]), __float_as_int(d[v + 1])));
                        }
                    }
                    redo = __any(__uint_as_float(above) <= thr || -__int_as_float(below) <= thr);
                }
                if (redo) {  // uniform
                    bits = 0;
                    const float rc = sqrtf(rcf);
                    const float band = fmaxf(1e-5f * rcf, rc * (4.7683716e-7f * sqrtf(M) +
                                                                (MI ? 7.1525574e-7f * fmaxf(Lx, fmaxf(Ly, Lz)) : 0.0f)));
                    const float lo2 = rcf - band, hi2 = rcf + band;
                    const float* pi = &s_i[w][4 * (16 * tt + lr)];
#pragma unroll MI ? 4 : 1
                    for (int e = 0; e < 16; ++e) {
                        const int k = 16 * (e >> 2) + 4 * lg + (e & 3);
                        const float* q = &s_j[w][4 * k];
                        float dx = pi[0] - q[0], dy = pi[1] - q[1], dz = pi[2] - q[2];
                        if (MI) {
                            dx -= Lx * rintf(dx * Lix);
                            dy -= Ly * rintf(dy * Liy);
                            dz -= Lz * rintf(dz * Liz);
                        }
                        const float r2 = dx * dx + dy * dy + dz * dz;
                        bool in = r2 < hi2 && pi[3] < kFar && q[3] < kFar;
                        if (in && !(r2 < lo2)) {  // rare: decided by the FP64 distance
                            const double4 p = pos_s[I * kBlock + 16 * tt + lr];
                            const double4 pk = pos_s[tile_j[(size_t)t * kBlock + k]];
                            const double ex = mimg_fp64(p.x - pk.x, box.x, binv.x),
                                         ey = mimg_fp64(p.y - pk.y, box.y, binv.y),
                                         ez = mimg_fp64(p.z - pk.z, box.z, binv.z);
                            in = ex * ex + ey * ey + ez * ez < rc2;
                        }
                        bits |= in ? 1u << e : 0u;
                    }
                }
                s_p[w][4 * (16 * tt + lr) + lg] = (uint16_t)bits;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            // row `lane`: bits 16 lg + 4 m + v of its four parts are the columns 16 m + 4 lg + v
            const uint16_t* pp = &s_p[w][4 * lane];
            m = transpose_nibbles((unsigned long long)pp[0] | (unsigned long long)pp[1] << 16 |
                                  (unsigned long long)pp[2] << 32 | (unsigned long long)pp[3] << 48);
            if (tile_j[(size_t)t * kBlock] == I * kBlock)  // the block with itself
                m &= lane == kBlock - 1 ? 0ull : ~0ull << (lane + 1);
            mask[(size_t)t * kBlock + lane] = m;
        }
        // The pair kernels split a tile's in-cutoff pairs (row-major) among the 64 lanes of a wave,
        // lane l taking pairs [l B, (l + 1) B) with B = ceil(P / 64).  Its first pair, row i (the
        // last row whose exclusive pair offset is <= l B) and that row's bit, is found here once
        // per configuration instead of by every product.
        {
            const int off = wave_excl_scan_i(__popcll(m), P);
            s_off[w][lane] = off;
            s_m[w][lane] = m;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (act) {
                const int Bs = (P + 63) >> 6, p0 = lane * Bs;
                uint16_t ws = 0xffff;
                if (p0 < P) {
                    int lo = 0, hi = kBlock - 1;
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (s_off[w][mid] <= p0)
                            lo = mid;
                        else
                            hi = mid - 1;
                    }
                    ws = (uint16_t)(lo | nth_set_bit(s_m[w][lo], p0 - s_off[w][lo]) << 8);
                }
                walk[(size_t)t * kBlock + lane] = ws;
            }
        }
        // pairs of the workgroup's tiles: one partial per workgroup, summed in order by
        // k_sum_pairs (no global atomics)
        if (lane == 0) {
            s_cnt[w] = (unsigned long long)P;
            if (act) {
                tile_np[t] = P;               // the pair kernels balance their waves by it
                tile_rows[t] = (P + 63) >> 6;  // rows of the tile's stored coefficients
            }
        }
        __syncthreads();
        if (threadIdx.x == 0)
            pair_part[group] = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
        __syncthreads();  // s_cnt is free for the next group
    }
}

__global__ __launch_bounds__(1024) void k_sum_pairs(int n, const unsigned long long* __restrict__ part,
                                                    unsigned long long* __restrict__ total)  // pinned host word
{
    // integer sums: exact in any order; eight loads in flight per thread
    __shared__ unsigned long long sh[16];
    unsigned long long a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 1024) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * 1024;
            if (i < n)
                a[u] += part[i];
        }
    }
    unsigned long long s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    for (int off = 32; off > 0; off >>= 1)
        s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0)
        sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long tot = 0;
        for (int k = 0; k < 16; ++k)
            tot += sh[k];
        total[0] = tot;
    }
}

static inline int nblk(long n, int b) { return (int)((n + b - 1) / b); }

constexpr int kScanOneWG = 8192;  // longest array scanned by one workgroup (measured)

int device_scan(amoeba_ctx* c, int n, const int* in, int* out, int* total_copy)
{
    // one workgroup walks short arrays in tiles of 4096; longer ones take the two launches
    // (block sums, then block-local scans), whose latency does not grow with the length
    hipStream_t st = c->stream;
    const int cap = c->npad / 1024 + 2;
    const int nbk = nblk(n, 1024);
    if (n <= kScanOneWG || (n <= 65536 && nbk + 1 > cap)) {
        hipLaunchKernelGGL(k_scan_excl, dim3(1), dim3(1024), 0, st, n, in, out, total_copy);
        return AMOEBA_OK;
    }
    if (nbk + 1 > cap)
        return set_error(c, AMOEBA_E_INVALID, "device_scan: scratch too small");
    int* bsum = c->b_scan;
    hipLaunchKernelGGL(k_scan_blocksum, dim3(nbk), dim3(256), 0, st, n, in, bsum);
    hipLaunchKernelGGL(k_scan_apply, dim3(nbk), dim3(256), 0, st, n, in, bsum, out, total_copy);
    return AMOEBA_OK;
}

int sort_params(amoeba_ctx* c)
{
    hipStream_t st = c->stream;
    coef_invalidate(c);  // the coefficients depend on the polarizabilities and Thole factors
    // parameters and the scaled-pair CSR in slot order
    int* cnt = c->b_cnt;
    auto params = [&](auto* pv) {
        using R = std::remove_pointer_t<decltype(pv)>;
        hipLaunchKernelGGL(k_params<R>, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm, c->alpha_in,
                           c->thole_in, c->par_d, c->par_f, c->alpha_s, c->alpha_inv_s, c->sc_ptr_in, cnt, pv);
    };
    if (c->mixed)
        params((float*)c->pv_f);
    else
        params((double*)c->pv_d);
    int rcs = device_scan(c, c->npad, cnt, c->sc_ptr);
    if (rcs)
        return rcs;
    if (c->n_scaled > 0)
        hipLaunchKernelGGL(k_csr_fill, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm, c->slot,
                           c->sc_ptr_in, c->sc_j_in, c->sc_s_in, c->sc_ptr, c->sc_j, c->sc_s);
    if (c->n_scaled > 0 && c->dscales_set)  // the same pairs, their direct scales (sc_j rewritten alike)
        hipLaunchKernelGGL(k_csr_fill, dim3(nblk(c->npad, 256)), dim3(256), 0, st, c->npad, c->perm, c->slot,
                           c->sc_ptr_in, c->sc_j_in, c->sc_sd_in, c->sc_ptr, c->sc_j, c->sc_sd);
    // the tiles' j records carry the slots' polarizability factors: refresh them before the
    // next product
    c->cfg_valid = false;
    return AMOEBA_OK;
}

// Rows of the stored pair coefficients of the current masks; their total reaches the host with
// its next wait.
void coef_scan_rows(amoeba_ctx* c)
{
    const bool scan_fits = c->ntiles <= 65536 || nblk(c->ntiles, 1024) + 1 <= c->npad / 1024 + 2;
    if (c->ntiles > 0 && scan_fits && device_scan(c, c->ntiles, c->tile_rows, c->coef_row0) == AMOEBA_OK) {
        hipMemcpyAsync(c->flags_host + 10, c->coef_row0 + c->ntiles, sizeof(int), hipMemcpyDeviceToHost, c->stream);
        c->coef_rows_ok = true;
        c->coef_rows_pending = true;
    }
}

// Sum of the mask refresh's per-workgroup pair counts, written to pinned host memory (read by
// amoeba_get_info after ev_pairs).
void launch_sum_pairs(amoeba_ctx* c)
{
    hipLaunchKernelGGL(k_sum_pairs, dim3(1), dim3(1024), 0, c->stream, c->pair_nwg, c->pair_part, c->pairs_host_dev);
    hipEventRecord(c->ev_pairs, c->stream);
}

// Workgroups of the refresh at most: one that the flags end at once costs its dispatch (16 us of a
// product at 288,000 atoms with all 10,600).
constexpr int kRefreshWG = 4096;

// The mask refresh; with `flags`, unless they say that the configuration is the same or not valid.
static void launch_refresh(amoeba_ctx* c, const int* flags)
{
    hipStream_t st = c->stream;
    double3 box = make_double3(c->prm.box[0], c->prm.box[1], c->prm.box[2]);
    double3 binv = make_double3(1.0 / box.x, 1.0 / box.y, 1.0 / box.z);
    const int nwg = nblk((long)c->ntiles * kBlock, 256);
    auto refresh = [&](auto* kernel, auto* par, auto* jrel) {
        hipLaunchKernelGGL(kernel, dim3(std::min(nwg, kRefreshWG)), dim3(256), 0, st, c->ntiles, nwg, c->tile_blk, c->tile_j, c->n, c->pos_s,
                           c->blk_org, c->off_f, par, box, binv, c->prm.cutoff * c->prm.cutoff, c->tile_mask, jrel,
                           c->tile_np, c->tile_rows, c->tile_walk, c->pair_part, flags);
    };
    // the pair kernels of the context's precision read one of the two j records
    if (c->mixed)
        refresh(c->skip_mimg ? k_tile_refresh<float, false> : k_tile_refresh<float, true>, c->par_f, c->jrel_f);
    else
        refresh(c->skip_mimg ? k_tile_refresh<double, false> : k_tile_refresh<double, true>, c->par_d, c->jrel_d);
    c->pair_nwg = nwg;
}

// What follows from refreshed masks.
static void after_refresh(amoeba_ctx* c)
{
    launch_sum_pairs(c);
    c->pairs_pending = true;  // read by amoeba_get_info
    coef_invalidate(c);
    c->coef_rows_ok = false;
    if (coef_store_on(c))
        coef_scan_rows(c);
    c->pme_bins_stale = true;
}

static void refresh_tiles(amoeba_ctx* c)
{
    StageTimer tm(c, AMOEBA_T_LIST);
    launch_refresh(c, nullptr);
    after_refresh(c);
}

// Steps 1-4 of the build (everything before the first mask refresh).
static int build_tiles(amoeba_ctx* c, const double* pos)
{
    hipStream_t st = c->stream;
    const int n = c->n, nb = c->nb, npad = c->npad;
    double3 box = make_double3(c->prm.box[0], c->prm.box[1], c->prm.box[2]);
    // column cross-section: about one block per (edge x edge x edge) at the mean density
    double vol = box.x * box.y * box.z;
    double edge = cbrt(kBlock * vol / n);
    int ny = (int)fmin(255.0, fmax(1.0, floor(box.y / edge + 0.5)));
    int nz = (int)fmin(255.0, fmax(1.0, floor(box.z / edge + 0.5)));
    // at most npad buckets, the last one for non-finite positions
    const long long nkeys = (long long)ny * nz << kXBits;
    int shift = 0;
    while (((nkeys - 1) >> shift) + 2 > npad)
        ++shift;
    const int nbucket = (int)((nkeys - 1) >> shift) + 2;

    int rc = AMOEBA_OK;
    if (!c->b_keys) {
        // block grid: at most floor(L / rcb) cells per axis (the cell width is at least rcb),
        // and not many more cells than blocks (nor than the grid kernel has counters)
        const double rcb = c->prm.cutoff + c->prm.buffer;
        for (int a = 0; a < 3; ++a)
            c->b_ncap[a] = (int)std::max(1.0, std::min(1024.0, std::floor(c->prm.box[a] / rcb)));
        auto ncells = [&]() { return (long long)c->b_ncap[0] * c->b_ncap[1] * c->b_ncap[2]; };
        while (ncells() > std::min(2ll * nb + 27, (long long)kGridCells)) {
            int* big = std::max_element(c->b_ncap, c->b_ncap + 3);
            if (*big <= 3)
                break;
            --*big;
        }
        c->b_ncell_cap = (int)ncells();
        if ((rc = ctx_alloc_all(c, {{&c->b_keys, sizeof(unsigned) * n},
                                    {&c->b_entry, sizeof(unsigned long long) * n},
                                    {&c->b_cell_blk, sizeof(int) * nb},
                                    {&c->b_bc, sizeof(double4) * nb},
                                    {&c->b_bh, sizeof(double4) * nb},
                                    {&c->b_rowc, sizeof(int) * nb},
                                    {&c->b_rowj, sizeof(int) * (size_t)nb * kMaxFiltered},
                                    {&c->b_tpb, sizeof(int) * (nb + 1)},
                                    {&c->rev_cnt, sizeof(int) * (npad + 1)},
                                    {&c->b_cell_start, sizeof(int) * ((size_t)c->b_ncell_cap + 1)}})))
            return rc;
    }
    double4 *bc = c->b_bc, *bh = c->b_bh;
    int *row_count = c->b_rowc, *row_j = c->b_rowj, *tpb = c->b_tpb, *t0 = c->blk_tile0;
    // build status words, read back with one copy: flags[0] error flags, flags[1] the tile
    // count, flags[4..9] the largest block half-extents (b_extent); flags[16..19] the block grid
    // (device only)
    int* grid = c->flags + 16;
    // rev_cnt, zero between its uses, counts the buckets; rev_ptr and b_cnt serve until their own use
    int *arrival = c->b_cnt, *start = c->rev_ptr;
    hipLaunchKernelGGL(k_sort_keys, dim3(nblk(n, 256)), dim3(256), 0, st, n, pos, box, ny, nz, shift, nbucket,
                       c->b_keys, arrival, c->rev_cnt, c->flags);
    if ((rc = device_scan(c, nbucket, c->rev_cnt, start))) {
        hipMemsetAsync(c->rev_cnt, 0, sizeof(int) * (npad + 1), st);
        return rc;
    }
    hipLaunchKernelGGL(k_sort_place, dim3(nblk(n, 256)), dim3(256), 0, st, n, shift, nbucket, c->b_keys, arrival,
                       start, c->rev_cnt, c->b_entry);
    hipLaunchKernelGGL(k_sort_rank, dim3(nblk(npad, 256)), dim3(256), 0, st, n, npad, shift, nbucket, c->b_entry,
                       start, pos, box, c->perm, c->slot, c->pos_s, c->pos_ref, c->flags);
    if (c->atoms_set && (rc = sort_params(c)) != AMOEBA_OK)
        return rc;

    hipLaunchKernelGGL(k_bbox, dim3(nblk(nb, 4)), dim3(256), 0, st, nb, c->perm, c->pos_s, box, bc, bh, c->blk_org,
                       c->off_d, c->off_f);
    const double rcb = c->prm.cutoff + c->prm.buffer;
    // the entries' space serves as the blocks' (key, arrival) and the keys' as the unranked order
    hipLaunchKernelGGL(k_block_grid, dim3(1), dim3(1024), 0, st, nb, bc, bh, box, rcb,
                       make_int3(c->b_ncap[0], c->b_ncap[1], c->b_ncap[2]), c->b_extent, grid, (int2*)c->b_entry,
                       (int*)c->b_keys, c->b_cell_start);
    hipLaunchKernelGGL(k_cell_rank, dim3(nblk(nb, 256)), dim3(256), 0, st, nb, grid, (const int2*)c->b_entry,
                       (const int*)c->b_keys, c->b_cell_start, c->b_cell_blk);
    double3 binv = make_double3(1.0 / box.x, 1.0 / box.y, 1.0 / box.z);
    // the counters are zero again after every complete build: counted up here, down by the fill
    auto fail = [&](int code) {
        hipMemsetAsync(c->rev_cnt, 0, sizeof(int) * (npad + 1), st);
        return code;
    };
    hipLaunchKernelGGL(k_filter, dim3(nb), dim3(256), 0, st, nb, n, c->pos_s, bc, bh, c->b_extent, grid,
                       c->b_cell_blk, c->b_cell_start, box, binv, rcb, row_count, row_j, tpb, c->rev_cnt, c->flags);
    if ((rc = device_scan(c, nb, tpb, t0, c->flags + 1)))
        return fail(rc);
    hipMemcpyAsync(c->flags_host, c->flags, 4 * sizeof(int) + 3 * sizeof(double), hipMemcpyDeviceToHost, st);
    hipEventRecord(c->ev_build, st);
    // the fill runs while the host waits for the counts, if the tiles fit the arrays there are
    auto fill = [&] {
        hipLaunchKernelGGL(k_fill_tiles, dim3(nb), dim3(256), 0, st, nb, (int)c->tile_cap, t0, row_count, row_j,
                           c->rev_ptr, c->rev_cnt, c->tile_blk, c->tile_j, c->rev_idx);
    };
    if ((rc = device_scan(c, npad, c->rev_cnt, c->rev_ptr)))
        return fail(rc);
    const int filled_cap = c->tile_cap;
    if (filled_cap > 0)
        fill();
    if ((rc = hip_check(c, hipEventSynchronize(c->ev_build), "build_blocklist")))
        return fail(rc);
    const int total = c->flags_host[1];
    {
        // Every j-atom of a tile lies within cutoff + buffer of an atom of the i-block at the
        // build, and atoms move at most buffer/2 before the list goes stale, so a tile
        // displacement component is at most rc + 3 buffer + 4 h (h the largest block
        // half-extent on that axis).  Below half the box edge the block-relative offsets
        // already give the minimum image and the pair kernels skip it.
        const double* ext = (const double*)(c->flags_host + 4);
        bool ok = true;
        for (int a = 0; a < 3; ++a) {
            const double bound = c->prm.cutoff + 3.0 * c->prm.buffer + 4.0 * ext[a];
            ok = ok && std::isfinite(ext[a]) && bound < 0.5 * c->prm.box[a] * (1.0 - 1e-3);
        }
        c->skip_mimg = ok;
    }
    if (*c->flags_host & kFlagNonFinite) {
        set_error(c, AMOEBA_E_NUMERIC, "build_blocklist: non-finite position");
        return fail(AMOEBA_E_NUMERIC);
    }
    if (*c->flags_host & kFlagFilterOverflow) {
        set_error(c, AMOEBA_E_INVALID, "build_blocklist: more than 2048 atoms within cutoff+buffer of a block "
                                       "(density too high for the list capacity)");
        return fail(AMOEBA_E_INVALID);
    }
    if (total > c->tile_cap) {
        // grow the tile arrays (earlier, smaller ones stay allocated until destroy)
        size_t tb = (size_t)total * kBlock;
        size_t rs = c->mixed ? sizeof(float) : sizeof(double);
        // the j records of the context's precision
        const AllocReq jrel = c->mixed ? AllocReq(&c->jrel_f, sizeof(float4) * tb) : AllocReq(&c->jrel_d, sizeof(double4) * tb);
        if ((rc = ctx_alloc_all(c, {{&c->tile_blk, sizeof(int) * total},
                                    {&c->tile_j, sizeof(int) * tb},
                                    {&c->tile_mask, sizeof(unsigned long long) * tb},
                                    {&c->tile_np, sizeof(int) * total},
                                    {&c->tile_walk, sizeof(uint16_t) * tb},
                                    {&c->tile_rows, sizeof(int) * total},
                                    {&c->coef_row0, sizeof(int) * (total + 1)},
                                    jrel,
                                    {&c->jbuf, rs * 4 * tb},
                                    {&c->rev_idx, sizeof(int) * tb},
                                    {&c->pair_part, sizeof(unsigned long long) * ((size_t)total / 4 + 1)}})))
            return fail(rc);
        c->tile_cap = total;
        c->rev_cap = (int64_t)tb;
    }
    c->ntiles = total;
    if (total > filled_cap)
        fill();
    return AMOEBA_OK;
}

int build_blocklist(amoeba_ctx* c, const double* pos)
{
    int rc;
    {
        StageTimer tm(c, AMOEBA_T_LIST);
        rc = build_tiles(c, pos);
    }
    if (rc != AMOEBA_OK)
        return rc;
    refresh_tiles(c);   // the pair count is read when amoeba_get_info asks for it
    pme_bins_current(c);
    c->list_built = true;
    c->cfg_valid = true;
    return AMOEBA_OK;
}

// The device flags, and the rows of the stored coefficients where the host waits for them, to the
// host without a copy and a wait for the whole stream: a kernel writes them and then the sequence
// number to coherent host memory, which the host watches.
__global__ void k_post_flags(const int* __restrict__ flags, const int* __restrict__ rows, int* __restrict__ post,
                             int seq)
{
    __hip_atomic_store(&post[1], flags[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (rows)
        __hip_atomic_store(&post[2], rows[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&post[0], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

int post_flags(amoeba_ctx* c)
{
    c->post_seq = c->post_seq == INT_MAX ? 1 : c->post_seq + 1;
    const int* rows = c->coef_rows_pending ? c->coef_row0 + c->ntiles : nullptr;
    hipLaunchKernelGGL(k_post_flags, dim3(1), dim3(1), 0, c->stream, c->flags, rows, c->post_dev, c->post_seq);
    return c->post_seq;
}

// The host watches the word for kWatch at most (every wait of a call on an idle stream is shorter), then
// waits for the stream as the device's schedule flags say: behind a long queue it does not hold a core.
constexpr std::chrono::milliseconds kWatch(5);

int wait_flags(amoeba_ctx* c, int seq, int* f, const char* who)
{
    int rc = AMOEBA_OK;
    const auto t0 = std::chrono::steady_clock::now();
    for (unsigned spin = 1; __atomic_load_n(&c->post_host[0], __ATOMIC_ACQUIRE) != seq; ++spin) {
        if (spin % 4096)
            continue;
        // the stream ended or failed: its own word on it
        if (hipStreamQuery(c->stream) == hipErrorNotReady) {
            if (hipPeekAtLastError() == hipErrorNotReady)
                (void)hipGetLastError();  // not an error to leave behind
            if (std::chrono::steady_clock::now() - t0 < kWatch)
                continue;
        }
        if ((rc = hip_check(c, hipStreamSynchronize(c->stream), who)))
            return rc;
        if (__atomic_load_n(&c->post_host[0], __ATOMIC_ACQUIRE) != seq)
            return set_error(c, AMOEBA_E_DEVICE, std::string(who) + ": flags not received");
    }
    *f = c->post_host[1];
    if (c->coef_rows_pending)
        c->flags_host[10] = c->post_host[2];
    return AMOEBA_OK;
}

int prepare_config(amoeba_ctx* c, const double* pos)
{
    hipStream_t st = c->stream;
    double3 box = make_double3(c->prm.box[0], c->prm.box[1], c->prm.box[2]);
    double hb = 0.5 * c->prm.buffer;
    hipMemsetAsync(c->flags, 0, sizeof(int), st);
    hipLaunchKernelGGL(k_gather_pos, dim3(std::min(nblk(c->npad, 256), kScatterWG)), dim3(256), 0, st, c->npad,
                       c->perm, pos, box, c->pos_s, (const double4*)c->pos_ref, hb * hb, c->flags, c->blk_org,
                       c->off_d, c->off_f);
    // The masks are refreshed while the host waits for the flags, on the flags' own say where the
    // present masks may still be right (the stage timers want the refresh by itself).  A copy of the
    // flags and a wait for the stream before the refresh left the GPU idle for some 10 us: a permanent
    // field at 96,000 atoms 222 -> 206 us.
    const int seq = post_flags(c);
    const bool early = !c->timing && c->ntiles > 0;
    if (early)
        launch_refresh(c, c->flags);
    int f = 0;
    int rc = wait_flags(c, seq, &f, "prepare_config");
    if (rc) {
        c->cfg_valid = false;
        return rc;
    }
    coef_reserve(c);
    if (f & kFlagNonFinite) {
        c->cfg_valid = false;
        return set_error(c, AMOEBA_E_NUMERIC, "non-finite position");
    }
    if (f & kFlagStale) {
        c->cfg_valid = false;
        return set_error(c, AMOEBA_E_LIST, "block list is stale: an atom moved more than buffer/2 since "
                                           "amoeba_build_blocklist");
    }
    if (c->cfg_valid && !(f & kFlagChanged))
        return AMOEBA_OK;  // same configuration as the last refresh: masks, frames and bins are current
    // the pair count is read when amoeba_get_info asks for it
    if (early && (f & kFlagChanged))
        after_refresh(c);
    else
        refresh_tiles(c);
    c->cfg_valid = true;
    return AMOEBA_OK;
}

}  // namespace amoeba
