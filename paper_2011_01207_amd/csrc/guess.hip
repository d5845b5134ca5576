// Learned initial guess of the induced dipoles: bases, features, the per-atom network and its
// training (forward, backward, Adam).  This is an addition to the paper's method, which starts
// its PCG from a plain guess; PCG still converges to the same tolerance from any start.
//
// Bases (slot order, FP64): v0 = alpha E_perm, v_{k+1} = alpha (R[v_k] + c v_k), with R the
// real-space dipole field of the pair kernel (the same tiles and precision as a PCG product)
// and c the Ewald self coefficient.  Invariant features: alpha, Thole a, |v_k| in Debye, the
// three cosines between the bases, and three Gaussian-weighted neighbour counts over the
// in-cutoff pairs of the tile list.  Network: SiLU MLP NFEAT -> 64 -> 64 -> NBASIS in FP32,
// mu0 = sum_k (s_k + y_k) v_k with s = (1, 1, 1).
//
// Delta kind, for a configuration that follows a solved one (converged dipoles mu_ref and
// permanent field E_ref of that one, held by the context in caller order): v0 = mu_ref,
// v1 = alpha (E_perm - E_ref), v2 = alpha E_perm, s = (1, 0, 0), the radial sums left out (zero).
// The untrained network returns mu_ref, the previous-step guess; trained, it adds the local
// response to the change of the permanent field, with no real-space product and no tile walk.
//
// Both dense layers, forward and backward, and the weight gradients are matrix products on the
// matrix cores in FP32.  Training gives every tile of 16 samples to a fixed wave and sums waves and
// workgroups in a fixed order, so gradients, losses and updates are bitwise reproducible.
#include <algorithm>
#include <cmath>
#include <map>
#include <mutex>
#include <type_traits>
#include <vector>

#include "common.h"
#include "reduce.h"

namespace amoeba {

template <typename R4T> struct Cast4G;
template <> struct Cast4G<float4> {
    __device__ static float4 make(double x, double y, double z, double w)
    {
        return make_float4((float)x, (float)y, (float)z, (float)w);
    }
};
template <> struct Cast4G<double4> {
    __device__ static double4 make(double x, double y, double z, double w) { return make_double4(x, y, z, w); }
};

constexpr int kNF = AMOEBA_GUESS_NFEAT;
constexpr int kNB = AMOEBA_GUESS_NBASIS;
constexpr int kH = AMOEBA_GUESS_HIDDEN;
constexpr int kNP = AMOEBA_GUESS_NPARAM;
constexpr int kNM = AMOEBA_GUESS_NMODEL;
constexpr int kOffB1 = kH * kNF;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + kNB * kH;
constexpr int kOffMean = kNP;
constexpr int kOffInv = kNP + kNF;
static_assert(kOffB3 + kNB == kNP, "parameter layout");
static_assert(kNP + 2 * kNF == kNM, "model layout");
constexpr int kGuessWG = 256;          // workgroups of the gradient kernel (at most)

// Scratch of amoeba_guess_gradient_noalloc: per-workgroup gradient and loss partials, the loss
// and the flag word, for batches of at most AMOEBA_GUESS_NOALLOC_MAX_BATCH samples, in one file-scope
// device array (each device holds its own copy until the process ends).  Host code never uses
// the array's name as an address: guess_scratch_init looks up each device's address once.
constexpr int kScratchWG = 128;  // 64 samples to a workgroup (guess_grad)
static_assert(kScratchWG * 64 >= AMOEBA_GUESS_NOALLOC_MAX_BATCH, "scratch partials");
constexpr size_t kScratchPart = sizeof(float) * (size_t)kNP * kScratchWG;
constexpr size_t kScratchLoss = kScratchPart;
constexpr size_t kScratchScal = kScratchLoss + sizeof(double) * kScratchWG;
constexpr size_t kScratchFlags = kScratchScal + sizeof(double) * 4;
constexpr size_t kScratchBytes = (kScratchFlags + sizeof(int) + 255) / 256 * 256;
static_assert(kScratchLoss % 8 == 0, "scratch layout");
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// fixed offsets s_k of mu0 = sum_k (s_k + y_k) v_k
struct GuessOffsets {
    float s[kNB];
};

// logistic function with the hardware reciprocal (1 ulp) instead of an IEEE division sequence
__device__ __forceinline__ float sigm(float a) { return __builtin_amdgcn_rcpf(1.0f + __expf(-a)); }

static inline int nblk64(int64_t n, int b) { return (int)((n + b - 1) / b); }

// next basis vector: v = alpha (ereal + cself vprev), or v0 = alpha e when ereal is NULL; the
// pair kernel's copy of it is written to pv for the following real-space product
template <typename R4T>
__global__ void k_guess_basis(int npad, const double4* __restrict__ par, const double* __restrict__ ereal,
                              const double* __restrict__ vprev, double cself, double* __restrict__ vnext,
                              R4T* __restrict__ pv)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    const double al = par[s].x;
    double v[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const double x = vprev[3 * (size_t)s + c];
        v[c] = ereal ? al * (ereal[3 * (size_t)s + c] + cself * x) : al * x;
        vnext[3 * (size_t)s + c] = v[c];
    }
    pv[s] = Cast4G<R4T>::make(v[0], v[1], v[2], par[s].w);  // w: Thole factor, read by the dipole tiles
}

// delta bases: on entry v1 holds E_ref and v0 mu_ref in slot order (e the permanent field);
// v1 = alpha (e - E_ref), v2 = alpha e
__global__ void k_guess_delta_bases(int npad, const double4* __restrict__ par, const double* __restrict__ e,
                                    double* __restrict__ v1, double* __restrict__ v2)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    const double al = par[s].x;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const size_t i = 3 * (size_t)s + c;
        const double x = e[i];
        v1[i] = al * (x - v1[i]);
        v2[i] = al * x;
    }
}

// features and FP32 bases of every real atom, written at its slot (perm_out NULL) or at its
// caller index (perm_out = perm); phantom slots get zeros in slot order
__global__ void k_guess_features(int npad, const int* __restrict__ perm, const double4* __restrict__ par,
                                 const double* __restrict__ v, const double* __restrict__ radial, int caller_order,
                                 float* __restrict__ feat, float* __restrict__ basis)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= npad)
        return;
    const int a = perm[s];
    if (a < 0) {
        if (!caller_order) {
            for (int f = 0; f < kNF; ++f)
                feat[(size_t)s * kNF + f] = 0.0f;
            for (int f = 0; f < kNB * 3; ++f)
                basis[(size_t)s * kNB * 3 + f] = 0.0f;
        }
        return;
    }
    const size_t d = caller_order ? (size_t)a : (size_t)s;
    const size_t n3 = 3 * (size_t)npad;
    double b[kNB][3], nn[kNB];
#pragma unroll
    for (int k = 0; k < kNB; ++k) {
        nn[k] = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            b[k][c] = v[k * n3 + 3 * (size_t)s + c];
            nn[k] += b[k][c] * b[k][c];
            basis[d * kNB * 3 + k * 3 + c] = (float)b[k][c];
        }
    }
    const double4 p = par[s];
    float* x = feat + d * kNF;
    x[0] = (float)p.x;
    x[1] = (float)p.w;
#pragma unroll
    for (int k = 0; k < kNB; ++k)
        x[2 + k] = (float)(kDebye * sqrt(nn[k]));
    const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int i = pa[q], j = pb[q];
        const double dot = b[i][0] * b[j][0] + b[i][1] * b[j][1] + b[i][2] * b[j][2];
        x[5 + q] = (float)(dot / sqrt(nn[i] * nn[j] + 1e-20));
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
        x[8 + c] = radial ? (float)radial[3 * (size_t)s + c] : 0.0f;
}

// ------------------------------------------------------------------------------------------
// Sum over the 16 lanes of a row (lanes with the same lane / 16), in every lane: data-parallel
// additions with the neighbour, the neighbouring pair, and the mirrored half row and row (the
// partial sums are uniform in the halves that they mirror).
__device__ __forceinline__ float row_sum(float x)
{
    auto add = [](float v, auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), C, 0xf, 0xf, true));
    };
    x = add(x, std::integral_constant<int, 0xb1>{});   // quad_perm [1, 0, 3, 2]
    x = add(x, std::integral_constant<int, 0x4e>{});   // quad_perm [2, 3, 0, 1]
    x = add(x, std::integral_constant<int, 0x141>{});  // row_half_mirror
    x = add(x, std::integral_constant<int, 0x140>{});  // row_mirror
    return x;
}

// Inference over many samples (the whole box per configuration): the two dense layers are
// matrix products over tiles of 16 samples on the matrix cores (FP32 in and out,
// v_mfma_f32_16x16x4f32: A 16x4 with lane l holding A[l mod 16][l div 16], B 4x16 with lane l
// holding B[l div 16][l mod 16], D 16x16 with lane l holding D[4 (l div 16) + v][l mod 16] in
// its v-th register).  Layer 1: A = normalised features (11 padded to 12), B = W1^T (in
// registers).  Its output goes through LDS to become the A operand of layer 2 (B = W2^T, read
// from LDS, which keeps the register count at three waves per SIMD).  The output layer and the
// basis combination run on the vector units, each lane summing its units and the 16 lanes of a
// group adding their partial sums (row_sum).  The next tile's inputs are loaded during the current one.
typedef float mfma_f4 __attribute__((ext_vector_type(4)));
constexpr int kFwdTile = 16;        // samples per tile (one wave)
constexpr int kFwdMaxWG = 768;      // workgroups at most (grid-stride over the tiles; measured)

__global__ __launch_bounds__(256) void k_guess_forward(int64_t n, const float* __restrict__ w,
                                                       const float* __restrict__ feat,
                                                       const float* __restrict__ basis, GuessOffsets so,
                                                       const int* __restrict__ perm, double* __restrict__ out64,
                                                       float* __restrict__ out32)
{
    static_assert(kH == 64 && kNF <= 12 && kNB == 3, "tile shapes of the matrix-core forward");
    __shared__ float s_h[4][kFwdTile][kH + 1];
    __shared__ float s_w2t[kH][72];  // W2 transposed: [input unit][output unit]
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    // operands that every tile uses: B of layer 1 (k = feature 4 s + lg, n = unit 16 nt + lr),
    // W2 for B of layer 2 (k = input unit 4 s + lg, n = unit 16 nt + lr), biases and output
    // weights of this lane's units, normalisation of its features
    float w1b[4][3], bias1[4], bias2[4], w3l[kNB][4], mean[3], inv[3];
    for (int i = threadIdx.x; i < kH * kH; i += 256)
        s_w2t[i % kH][i / kH] = w[kOffW2 + i];
#pragma unroll
    for (int s3 = 0; s3 < 3; ++s3) {
        const int f = 4 * s3 + lg;
        mean[s3] = f < kNF ? w[kOffMean + f] : 0.0f;
        inv[s3] = f < kNF ? w[kOffInv + f] : 0.0f;
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int u = 16 * nt + lr;
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const int f = 4 * s3 + lg;
            w1b[nt][s3] = f < kNF ? w[u * kNF + f] : 0.0f;
        }
        bias1[nt] = w[kOffB1 + u];
        bias2[nt] = w[kOffB2 + u];
#pragma unroll
        for (int c = 0; c < kNB; ++c)
            w3l[c][nt] = w[kOffW3 + c * kH + u];
    }
    __syncthreads();
    const int64_t ntiles = (n + kFwdTile - 1) / kFwdTile;
    const int64_t stride = (int64_t)gridDim.x * 4;
    // this lane's inputs of a tile: features (A of layer 1) and, for the lanes that write an
    // output component, the basis vectors and the slot's phantom flag; the next tile's are
    // loaded while the current one is computed
    const int ov = lr / kNB, oc = lr - (lr / kNB) * kNB;  // output sample 4 lg + ov, component oc
    auto load_tile = [&](int64_t tile, float (&x)[3], float (&bs)[kNB], bool& live) {
        const int64_t ai = tile * kFwdTile + lr, ao = tile * kFwdTile + 4 * lg + ov;
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const int f = 4 * s3 + lg;
            x[s3] = (tile < ntiles && ai < n && f < kNF) ? feat[ai * kNF + f] : 0.0f;
        }
        live = tile < ntiles && lr < 4 * kNB && ao < n && !(perm && perm[ao] < 0);
#pragma unroll
        for (int k = 0; k < kNB; ++k)
            bs[k] = live ? basis[ao * kNB * 3 + k * 3 + oc] : 0.0f;
    };
    float xn[3], bn[kNB];
    bool ln;
    load_tile((int64_t)blockIdx.x * 4 + wv, xn, bn, ln);
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wv; tile < ntiles; tile += stride) {
        const int64_t a0 = tile * kFwdTile;
        float xc[3], bc[kNB];
        const bool lc = ln;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            xc[k] = xn[k];
            bc[k] = bn[k];
        }
        load_tile(tile + stride, xn, bn, ln);
        // layer 1
        mfma_f4 d1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            d1[nt] = mfma_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const float xa = (xc[s3] - mean[s3]) * inv[s3];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                d1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa, w1b[nt][s3], d1[nt], 0, 0, 0);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float a = d1[nt][v] + bias1[nt];
                s_h[wv][4 * lg + v][16 * nt + lr] = a * sigm(a);
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // layer 2
        mfma_f4 d2[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            d2[nt] = mfma_f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s16 = 0; s16 < 16; ++s16) {
            const float ha = s_h[wv][lr][4 * s16 + lg];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                d2[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ha, s_w2t[4 * s16 + lg][16 * nt + lr], d2[nt], 0, 0, 0);
        }
        // output layer: partial sums over this lane's units for the samples 4 lg + v
        float y[4][kNB];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                y[v][c] = 0.0f;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float a = d2[nt][v] + bias2[nt];
                const float h = a * sigm(a);
#pragma unroll
                for (int c = 0; c < kNB; ++c)
                    y[v][c] = fmaf(w3l[c][nt], h, y[v][c]);
            }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                y[v][c] = row_sum(y[v][c]);
        // lane lr < 12 of group lg writes component oc of sample 4 lg + ov (phantom slots: 0)
        const int64_t a = a0 + 4 * lg + ov;
        if (lr < 4 * kNB && a < n) {
            float yk[kNB];
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                yk[c] = ov == 0 ? y[0][c] : ov == 1 ? y[1][c] : ov == 2 ? y[2][c] : y[3][c];
            float mu = 0.0f;
            if (lc) {
#pragma unroll
                for (int k = 0; k < kNB; ++k)
                    mu = fmaf(so.s[k] + (w[kOffB3 + k] + yk[k]), bc[k], mu);
            }
            if (out64)
                out64[3 * a + oc] = (double)mu;
            else
                out32[3 * a + oc] = mu;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

static unsigned forward_grid(int64_t n)
{
    const int64_t tiles = (n + kFwdTile - 1) / kFwdTile;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((tiles + 3) / 4, kFwdMaxWG));
}

// ------------------------------------------------------------------------------------------
// Loss and gradient on the matrix cores (FP32 16x16x4, layouts as in k_guess_forward).  Workgroups
// of four waves; tile q of 16 samples belongs to wave q mod (4 G) of the launch.  A wave keeps a
// layer's values where its product leaves them, lane (lr, lg) holding samples 4 lg .. 4 lg + 3 of unit
// 16 nt + lr:
//   forward   a1 = x W1^T, a2 = h1 W2^T          (h1 through LDS to become an A operand)
//   backward  d2 = (d3 W3) silu'(a2), d1 = (d2 W2) silu'(a1)            (d2 through LDS)
//   weights   gW2 += d2^T h1, gW1 += d1^T x: the sum runs over samples, so register v of the layer
//             values is an operand as it stands (k index lg = sample 4 lg + v), with no transposition
// and the rest (output layer, biases, loss) on the vector units.  The weight gradients stay in 96
// registers over the wave's tiles; at the end the waves of the workgroup add theirs in LDS, in wave
// order, and the workgroup writes one partial.  Samples past the batch end contribute exactly zero.
// 220 matrix instructions (12 us for 65,536 samples) and about 700 vector ones to a tile.  One wave
// to a SIMD: the gradients and a tile's layers need 348 registers (two waves in 256 spilled: 53 us).
// For 65,536 samples 48 us; one wave per workgroup on the vector units, a sample to a lane, took
// 209 us.
// ------------------------------------------------------------------------------------------
constexpr int kGradWaves = 4;
constexpr int kPadA = kH + 4;    // LDS row strides that keep the operand reads free of bank conflicts:
constexpr int kPadB = kH + 16;   // [16 nt + lr][4 s + lg] and [4 s + lg][16 nt + lr]

struct GradWeights {
    float w2a[kH][kPadA];                    // W2, read as the B operand of h1 W2^T
    float w2b[kH][kPadB];                    // W2, read as the B operand of d2 W2
    float w1[kH][12], w3[kNB][kH], b1[kH], b2[kH];  // kept here rather than in registers
    float h[kGradWaves][kFwdTile][kPadA];    // a wave's h1, then its d2
};
constexpr int kGradSums = kGradWaves / 2;
static_assert(kGradWaves == 4 && kFwdTile * kGradWaves == 64, "the sums written out, and the scratch array's size");
union GradLds {
    GradWeights w;
    float sum[kGradSums][kNP];               // at the end: sums of the waves' gradients
};

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__global__ __launch_bounds__(64 * kGradWaves) void k_guess_grad(int64_t n_batch, int64_t n_rows,
                                                                const int* __restrict__ idx,
                                                                const float* __restrict__ w,
                                                                const float* __restrict__ feat,
                                                                const float* __restrict__ basis, GuessOffsets so,
                                                                const float* __restrict__ target, float lscale,
                                                                float* __restrict__ part, double* __restrict__ lossp,
                                                                int* __restrict__ flags)
{
    static_assert(kH == 64 && kNF <= 12 && kNB == 3, "tile shapes of the matrix-core gradient");
    __shared__ GradLds lds;
    __shared__ double s_loss[kGradWaves];
    GradWeights& L = lds.w;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, lr = lane & 15, lg = lane >> 4;
    for (int i = tid; i < kH * kH; i += 64 * kGradWaves) {
        const float v = w[kOffW2 + i];
        L.w2a[i / kH][i % kH] = v;
        L.w2b[i / kH][i % kH] = v;
    }
    for (int i = tid; i < kH * 12; i += 64 * kGradWaves)
        L.w1[i / 12][i % 12] = i % 12 < kNF ? w[(i / 12) * kNF + i % 12] : 0.0f;
    if (tid < kNB * kH)
        L.w3[tid / kH][tid % kH] = w[kOffW3 + tid];
    if (tid < kH) {
        L.b1[tid] = w[kOffB1 + tid];
        L.b2[tid] = w[kOffB2 + tid];
    }
    float mean[3], inv[3], bias3[kNB];
    const float mean_x = lr < kNF ? w[kOffMean + lr] : 0.0f, inv_x = lr < kNF ? w[kOffInv + lr] : 0.0f;
#pragma unroll
    for (int c = 0; c < kNB; ++c)
        bias3[c] = w[kOffB3 + c];
#pragma unroll
    for (int s3 = 0; s3 < 3; ++s3) {
        const int f = 4 * s3 + lg;
        mean[s3] = f < kNF ? w[kOffMean + f] : 0.0f;
        inv[s3] = f < kNF ? w[kOffInv + f] : 0.0f;
    }
    const mfma_f4 zero{0.0f, 0.0f, 0.0f, 0.0f};
    mfma_f4 gW2[4][4], gW1[4];
    float gW3[kNB][4], gb1[4], gb2[4], gb3[kNB];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gW1[a] = zero;
        gb1[a] = gb2[a] = 0.0f;
#pragma unroll
        for (int b = 0; b < 4; ++b)
            gW2[a][b] = zero;
#pragma unroll
        for (int c = 0; c < kNB; ++c)
            gW3[c][a] = 0.0f;
    }
#pragma unroll
    for (int c = 0; c < kNB; ++c)
        gb3[c] = 0.0f;
    double lacc = 0.0;
    const int64_t ntiles = (n_batch + kFwdTile - 1) / kFwdTile;
    float(&sh)[kFwdTile][kPadA] = L.h[wv];
    // the row of sample m of a tile, -1 past the batch end and for an index outside the data
    auto row_of = [&](int64_t tile, int m) -> int64_t {
        const int64_t b = tile * kFwdTile + m;
        if (b >= n_batch)
            return -1;
        const int64_t r = idx ? (int64_t)idx[b] : b;
        return r < 0 || r >= n_rows ? -1 : r;
    };
    // a tile's inputs: features as the A operand of layer 1 (sample lr) and as the B operand of gW1
    // (samples 4 lg + v), basis and target of sample 4 lg + lr mod 4.  The next tile's are loaded
    // while the current one is computed, and its row (of sample lr) one tile before that, so that no
    // load waits for another.
    struct In {
        float xa[3], xb[4], bs[kNB][3], tg[3];
    };
    auto load = [&](int64_t tile, int64_t ra, In& in) {
        const int64_t rs = __shfl((long long)ra, 4 * lg + (lr & 3));
        if (lg == 0 && ra < 0 && tile * kFwdTile + lr < n_batch)
            atomicOr(flags, kFlagBadIndex);
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3) {
            const int f = 4 * s3 + lg;
            in.xa[s3] = ra >= 0 && f < kNF ? (feat[ra * kNF + f] - mean[s3]) * inv[s3] : 0.0f;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t rv = __shfl((long long)ra, 4 * lg + v);
            in.xb[v] = rv >= 0 && lr < kNF ? (feat[rv * kNF + lr] - mean_x) * inv_x : 0.0f;
        }
#pragma unroll
        for (int k = 0; k < kNB; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                in.bs[k][c] = rs >= 0 ? basis[rs * kNB * 3 + k * 3 + c] : 0.0f;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            in.tg[c] = rs >= 0 ? target[rs * 3 + c] : 0.0f;
    };
    const int64_t stride = (int64_t)gridDim.x * kGradWaves, tile0 = (int64_t)blockIdx.x * kGradWaves + wv;
    In in;
    int64_t row_next = row_of(tile0 + stride, lr);
    load(tile0, row_of(tile0, lr), in);
    __syncthreads();  // the weights are in LDS
    for (int64_t tile = tile0; tile < ntiles; tile += stride) {
        float xa[3], xb[4], bs[kNB][3], tg[3];
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3)
            xa[s3] = in.xa[s3];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            xb[v] = in.xb[v];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            tg[c] = in.tg[c];
#pragma unroll
            for (int k = 0; k < kNB; ++k)
                bs[k][c] = in.bs[k][c];
        }
        load(tile + stride, row_next, in);
        row_next = row_of(tile + 2 * stride, lr);
        // layer 1
        mfma_f4 h1[4], s1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            h1[nt] = zero;
#pragma unroll
        for (int s3 = 0; s3 < 3; ++s3)
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                h1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[s3], L.w1[16 * nt + lr][4 * s3 + lg], h1[nt], 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const float bias = L.b1[16 * nt + lr];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float a = h1[nt][v] + bias, sg = sigm(a);
                h1[nt][v] = a * sg;
                s1[nt][v] = sg * (1.0f + a * (1.0f - sg));
                sh[4 * lg + v][16 * nt + lr] = h1[nt][v];
            }
        }
        wave_sync();
        // layer 2
        mfma_f4 h2[4], d2[4];  // d2: silu'(a2) until the delta replaces it
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            h2[nt] = zero;
#pragma unroll
        for (int s16 = 0; s16 < 16; ++s16) {
            const float ha = sh[lr][4 * s16 + lg];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                h2[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ha, L.w2a[16 * nt + lr][4 * s16 + lg], h2[nt], 0, 0, 0);
        }
        float y[4][kNB];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                y[v][c] = 0.0f;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int u = 16 * nt + lr;
            const float bias = L.b2[u], w3[kNB] = {L.w3[0][u], L.w3[1][u], L.w3[2][u]};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float a = h2[nt][v] + bias, sg = sigm(a);
                h2[nt][v] = a * sg;
                d2[nt][v] = sg * (1.0f + a * (1.0f - sg));
#pragma unroll
                for (int c = 0; c < kNB; ++c)
                    y[v][c] = fmaf(w3[c], h2[nt][v], y[v][c]);
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                y[v][c] = row_sum(y[v][c]);
        // loss and d3 of sample 4 lg + lr mod 4 (four lanes hold the same), then of all four
        float d3[4][kNB], l = 0.0f;
        {
            const int vs = lr & 3;
            float yk[kNB], gm[3], dk[kNB];
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                yk[c] = so.s[c] + (bias3[c] + (vs == 0 ? y[0][c] : vs == 1 ? y[1][c] : vs == 2 ? y[2][c] : y[3][c]));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                float m = 0.0f;
#pragma unroll
                for (int k = 0; k < kNB; ++k)
                    m = fmaf(yk[k], bs[k][c], m);
                const float dlt = m - tg[c];
                l = fmaf(dlt, dlt, l);
                gm[c] = 2.0f * lscale * dlt;
            }
#pragma unroll
            for (int k = 0; k < kNB; ++k) {
                dk[k] = gm[0] * bs[k][0] + gm[1] * bs[k][1] + gm[2] * bs[k][2];
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    d3[v][k] = __shfl(dk[k], (lane & 48) + v);
            }
            l = lr < 4 ? l * lscale : 0.0f;
            l = row_sum(l);
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            lacc += (double)l;
        }
        // delta of layer 2, and what it and the output layer add to their gradients
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            const int u = 16 * nt + lr;
            const float w3[kNB] = {L.w3[0][u], L.w3[1][u], L.w3[2][u]};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                float g = 0.0f;
#pragma unroll
                for (int c = 0; c < kNB; ++c) {
                    g = fmaf(w3[c], d3[v][c], g);
                    gW3[c][nt] = fmaf(d3[v][c], h2[nt][v], gW3[c][nt]);
                }
                d2[nt][v] *= g;
                gb2[nt] += d2[nt][v];
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int c = 0; c < kNB; ++c)
                gb3[c] += d3[v][c];
        wave_sync();  // h1 has been read from LDS
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                sh[4 * lg + v][16 * nt + lr] = d2[nt][v];
        wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int nt = 0; nt < 4; ++nt)
                    gW2[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(d2[mt][v], h1[nt][v], gW2[mt][nt], 0, 0, 0);
        mfma_f4 d1[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
            d1[nt] = zero;
#pragma unroll
        for (int s16 = 0; s16 < 16; ++s16) {
            const float da = sh[lr][4 * s16 + lg];
#pragma unroll
            for (int nt = 0; nt < 4; ++nt)
                d1[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(da, L.w2b[4 * s16 + lg][16 * nt + lr], d1[nt], 0, 0, 0);
        }
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                d1[nt][v] *= s1[nt][v];
                gb1[nt] += d1[nt][v];
            }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
                gW1[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(d1[mt][v], xb[v], gW1[mt], 0, 0, 0);
        wave_sync();  // d2 has been read from LDS
    }
    // sums over the four row groups of the vector-unit gradients (every lane)
    auto groups = [](float x) {
        x += __shfl_xor(x, 16);
        return x + __shfl_xor(x, 32);
    };
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        gb1[nt] = groups(gb1[nt]);
        gb2[nt] = groups(gb2[nt]);
#pragma unroll
        for (int c = 0; c < kNB; ++c)
            gW3[c][nt] = groups(gW3[c][nt]);
    }
#pragma unroll
    for (int c = 0; c < kNB; ++c)
        gb3[c] = groups(gb3[c]);
    if (lane == 0)
        s_loss[wv] = lacc;
    __syncthreads();  // the weights in LDS are no longer read
    // the first half of the waves into a sum each, the second half added to them, the sums added
    // where they are written out
    for (int r = 0; r < 2; ++r) {
        if (wv / kGradSums == r) {
            float* sum = lds.sum[wv % kGradSums];
            auto add = [&](int p, float v) { sum[p] = r ? sum[p] + v : v; };
#pragma unroll
            for (int mt = 0; mt < 4; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int k = 16 * mt + 4 * lg + v;
                    if (lr < kNF)
                        add(k * kNF + lr, gW1[mt][v]);
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt)
                        add(kOffW2 + k * kH + 16 * nt + lr, gW2[mt][nt][v]);
                }
            if (lg == 0) {
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) {
                    add(kOffB1 + 16 * nt + lr, gb1[nt]);
                    add(kOffB2 + 16 * nt + lr, gb2[nt]);
#pragma unroll
                    for (int c = 0; c < kNB; ++c)
                        add(kOffW3 + c * kH + 16 * nt + lr, gW3[c][nt]);
                }
                if (lr == 0)
#pragma unroll
                    for (int c = 0; c < kNB; ++c)
                        add(kOffB3 + c, gb3[c]);
            }
        }
        __syncthreads();
    }
    float* p = part + (size_t)blockIdx.x * kNP;
    for (int i = tid; i < kNP; i += 64 * kGradWaves)
        p[i] = lds.sum[0][i] + lds.sum[1][i];
    if (tid == 0) {
        double l = 0.0;
        for (int q = 0; q < kGradWaves; ++q)
            l += s_loss[q];
        lossp[blockIdx.x] = l;
    }
}

// Sum of the workgroup partials per parameter in FP64, in a fixed order: 64 parameters per
// workgroup, sixteen groups of partials per parameter (g, g+16, ...) combined in LDS in group
// order.  Then the gradient is written out and/or an Adam step is applied -- skipped when the
// gradient kernel flagged an index outside the data, so a rejected step changes nothing.  The
// loss is summed by the first wave of workgroup 0.  (Four groups over 512 partials took 52 us, a
// chain of 128 loads a thread.)
constexpr int kRedGroups = 16;
__global__ __launch_bounds__(64 * kRedGroups) void k_guess_reduce(int nwg, const float* __restrict__ part,
                                                      const double* __restrict__ lossp, float* __restrict__ grad,
                                                      float* __restrict__ w, float* __restrict__ m,
                                                      float* __restrict__ v, int adam, float lr, float bc1,
                                                      float bc2, double* __restrict__ loss,
                                                      const int* __restrict__ flags)
{
    __shared__ double s_sum[kRedGroups][64];
    const int tid = threadIdx.x, g = tid >> 6, pl = tid & 63;
    const int p = blockIdx.x * 64 + pl;
    if (blockIdx.x == 0 && g == 0) {
        double l = 0.0;
        for (int q = pl; q < nwg; q += 64)
            l += lossp[q];
        for (int off = 32; off > 0; off >>= 1)
            l += __shfl_xor(l, off);
        if (pl == 0)
            loss[0] = l;
    }
    double acc = 0.0;
    if (p < kNP) {
        // four loads in flight
        for (int q = g; q < nwg; q += 4 * kRedGroups) {
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                x[u] = q + u * kRedGroups < nwg ? part[(size_t)(q + u * kRedGroups) * kNP + p] : 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u)
                acc += (double)x[u];
        }
    }
    s_sum[g][pl] = acc;
    __syncthreads();
    if (g != 0 || p >= kNP)
        return;
    double tot = s_sum[0][pl];
#pragma unroll
    for (int q = 1; q < kRedGroups; ++q)
        tot += s_sum[q][pl];
    const float gr = (float)tot;
    if (grad)
        grad[p] = gr;
    if (adam && !(flags[0] & kFlagBadIndex)) {
        const float mm = 0.9f * m[p] + 0.1f * gr;
        const float vv = 0.999f * v[p] + 0.001f * gr * gr;
        m[p] = mm;
        v[p] = vv;
        w[p] -= lr * (mm * bc1) / (sqrtf(vv * bc2) + 1e-8f);
    }
}

// Feature statistics: pass 0 sums x, pass 1 sums (x - mean)^2; FP64 partials per workgroup.
__global__ __launch_bounds__(256) void k_guess_norm_partial(int64_t n, const float* __restrict__ feat, int pass,
                                                            const double* __restrict__ mean,
                                                            double* __restrict__ part)
{
    double acc[kNF];
#pragma unroll
    for (int f = 0; f < kNF; ++f)
        acc[f] = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
#pragma unroll
        for (int f = 0; f < kNF; ++f) {
            const double x = (double)feat[i * kNF + f];
            const double d = pass ? x - mean[f] : x;
            acc[f] += pass ? d * d : d;
        }
    block_sum<kNF>(acc);
    if (threadIdx.x < kNF)
        part[(size_t)blockIdx.x * kNF + threadIdx.x] = acc[threadIdx.x];
}

__global__ __launch_bounds__(256) void k_guess_norm_final(int nparts, int64_t n, const double* __restrict__ part,
                                                          int pass, double* __restrict__ mean, float* __restrict__ w)
{
    double tot[kNF];
    sum_partials<kNF>(part, nparts, tot);
    if (threadIdx.x < kNF) {
        const int f = threadIdx.x;
        if (pass == 0) {
            mean[f] = tot[f] / (double)n;
            w[kOffMean + f] = (float)mean[f];
        } else {
            const double sd = sqrt(tot[f] / (double)n);
            w[kOffInv + f] = sd > 1e-6 ? (float)(1.0 / sd) : 0.0f;
        }
    }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
static int guess_alloc_config(amoeba_ctx* c)
{
    if (c->g_v)
        return AMOEBA_OK;
    const size_t n3 = 3 * (size_t)c->npad;
    return ctx_alloc_all(c, {{&c->g_v, sizeof(double) * 3 * n3},
                             {&c->g_radial, sizeof(double) * n3},
                             {&c->g_feat, sizeof(float) * kNF * (size_t)c->npad},
                             {&c->g_basis, sizeof(float) * kNB * 3 * (size_t)c->npad},
                             {&c->g_save_mu, sizeof(double) * n3},
                             {&c->g_save_q, sizeof(double) * n3}});
}

static GuessOffsets guess_offsets(const amoeba_ctx* c)
{
    if (c->g_kind == AMOEBA_GUESS_KIND_DELTA)
        return GuessOffsets{{1.0f, 0.0f, 0.0f}};
    return GuessOffsets{{1.0f, 1.0f, 1.0f}};
}

// Bases and features of the configuration whose permanent field is in v_e (slot order).
int guess_compute(amoeba_ctx* c)
{
    if (c->g_kind == AMOEBA_GUESS_KIND_DELTA && !c->g_ref_set)
        return set_error(c, AMOEBA_E_STATE, "learned guess of the delta kind: no reference configuration "
                                            "(amoeba_guess_set_reference)");
    int rc = guess_alloc_config(c);
    if (rc)
        return rc;
    const size_t n3 = 3 * (size_t)c->npad;
    const double cself = 4.0 * pow(c->prm.ewald_alpha, 3) / (3.0 * sqrt(kPi));
    const int g = nblk64(c->npad, 256);
    if (c->g_kind == AMOEBA_GUESS_KIND_DELTA) {
        const size_t na3 = 3 * (size_t)c->n;
        // non-finite reference entries raise the flag read with the caller's next flag read
        launch_gather_vec_checked(c, c->g_ref, c->g_v);
        launch_gather_vec_checked(c, c->g_ref + na3, c->g_v + n3);
        StageTimer tm(c, AMOEBA_T_GUESS);
        hipLaunchKernelGGL(k_guess_delta_bases, dim3(g), dim3(256), 0, c->stream, c->npad, c->par_d, c->v_e,
                           c->g_v + n3, c->g_v + 2 * n3);
    }
    for (int k = 0; k < kNB && c->g_kind == AMOEBA_GUESS_KIND_NEUMANN; ++k) {
        const double* prev = k ? c->g_v + (k - 1) * n3 : c->v_e;
        const double* er = k ? c->ereal : nullptr;
        {
            StageTimer tm(c, AMOEBA_T_GUESS);
            if (c->mixed)
                hipLaunchKernelGGL(k_guess_basis<float4>, dim3(g), dim3(256), 0, c->stream, c->npad, c->par_d, er,
                                   prev, cself, c->g_v + k * n3, c->pv_f);
            else
                hipLaunchKernelGGL(k_guess_basis<double4>, dim3(g), dim3(256), 0, c->stream, c->npad, c->par_d, er,
                                   prev, cself, c->g_v + k * n3, c->pv_d);
        }
        if (k + 1 < kNB) {
            launch_mutual_tiles(c, false);
            launch_real_reduce(c, c->ereal);
        }
    }
    // the radial sums (a walk over every tile) only for the Neumann kind; the delta kind's
    // features leave them out (zero)
    const bool radial = c->g_kind == AMOEBA_GUESS_KIND_NEUMANN;
    if (radial)
        launch_radial_sums(c, c->g_radial);
    StageTimer tm(c, AMOEBA_T_GUESS);
    hipLaunchKernelGGL(k_guess_features, dim3(g), dim3(256), 0, c->stream, c->npad, c->perm, c->par_d, c->g_v,
                       radial ? c->g_radial : nullptr, 0, c->g_feat, c->g_basis);
    return AMOEBA_OK;
}

// mu0 of every slot (FP64, phantoms zero) from the slot-order features of guess_compute.
void guess_forward_slot(amoeba_ctx* c, double* mu_slot)
{
    StageTimer tm(c, AMOEBA_T_GUESS);
    hipLaunchKernelGGL(k_guess_forward, dim3(forward_grid(c->npad)), dim3(256), 0, c->stream, (int64_t)c->npad,
                       c->g_model, c->g_feat, c->g_basis, guess_offsets(c), c->perm, mu_slot, (float*)nullptr);
}

static int guess_alloc_model(amoeba_ctx* c)
{
    if (c->g_model)
        return AMOEBA_OK;
    if (!c->g_scal_host && hipHostMalloc((void**)&c->g_scal_host, sizeof(double) * 4, hipHostMallocDefault) != hipSuccess) {
        c->g_scal_host = nullptr;
        return set_error(c, AMOEBA_E_NOMEM, "pinned host allocation failed");
    }
    return ctx_alloc_all(c, {{&c->g_model, sizeof(float) * kNM},
                             {&c->g_adam_m, sizeof(float) * kNP},
                             {&c->g_adam_v, sizeof(float) * kNP},
                             {&c->g_part, sizeof(float) * kNP * (size_t)kGuessWG},
                             {&c->g_lossp, sizeof(double) * kGuessWG},
                             {&c->g_scal, sizeof(double) * 4},
                             {&c->g_npart, sizeof(double) * kNF * kRedBlocks},
                             {&c->g_nmean, sizeof(double) * kNF}});
}

// end of a features / predict call: the flag word (cleared by the e_perm check) reports a
// non-finite reference of the delta kind
static int guess_flags(amoeba_ctx* c, const char* who)
{
    int f = 0, rc = read_flags(c, &f);
    if (rc)
        return rc;
    if (f & kFlagNonFinite)
        return set_error(c, AMOEBA_E_NUMERIC, std::string(who) + ": non-finite value in the guess reference");
    return AMOEBA_OK;
}

static int guess_ready(amoeba_ctx* c, const char* who)
{
    if (!c->guess_loaded)
        return set_error(c, AMOEBA_E_STATE, std::string(who) + ": no model loaded (amoeba_guess_set_model)");
    return AMOEBA_OK;
}

// device buffers of a gradient evaluation: the context's, or the no-allocation scratch
struct GradWork {
    float* part;     // [nwg][NPARAM]
    double* lossp;   // [nwg]
    double* scal;    // [4]
    int* flags;
    bool fill_flags; // clear the flag word with a kernel instead of a memset node
};

__global__ void k_zero_flag(int* __restrict__ flags)
{
    if (threadIdx.x == 0)
        flags[0] = 0;
}

int guess_scratch_init(amoeba_ctx* c)
{
    // once per device, with that device current (amoeba_create runs on the caller's device)
    static std::mutex mu;
    static std::map<int, void*> addr;
    std::lock_guard<std::mutex> lock(mu);
    auto it = addr.find(c->device);
    if (it == addr.end()) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return set_error(c, AMOEBA_E_DEVICE, "hipGetSymbolAddress of the guess scratch failed");
        }
        it = addr.emplace(c->device, ptr).first;
    }
    c->g_scratch = it->second;
    return AMOEBA_OK;
}

static GradWork ctx_work(amoeba_ctx* c)
{
    return GradWork{c->g_part, c->g_lossp, c->g_scal, c->flags, false};
}

static GradWork scratch_work(amoeba_ctx* c)
{
    unsigned char* base = static_cast<unsigned char*>(c->g_scratch);
    return GradWork{reinterpret_cast<float*>(base), reinterpret_cast<double*>(base + kScratchLoss),
                    reinterpret_cast<double*>(base + kScratchScal), reinterpret_cast<int*>(base + kScratchFlags),
                    true};
}

// loss and gradient partials of a batch, then the reduction (Adam step when adam != 0)
static int guess_grad(amoeba_ctx* c, const float* feat, const float* basis, const float* target, int64_t n_rows,
                      const int32_t* idx, int64_t n_batch, float* grad_out, bool adam, float lr, double* loss_out,
                      const char* who, const GradWork& ws)
{
    if (!feat || !basis || !target)
        return set_error(c, AMOEBA_E_INVALID, std::string(who) + ": NULL feat, basis or target");
    if (n_batch < 1 || n_rows < 1 || (!idx && n_batch > n_rows))
        return set_error(c, AMOEBA_E_INVALID, std::string(who) + ": need 1 <= n_batch (<= n_rows without idx)");
    if (adam && !(lr > 0.0f && std::isfinite(lr)))
        return set_error(c, AMOEBA_E_INVALID, std::string(who) + ": lr must be positive");
    hipStream_t st = c->stream;
    // a tile of 16 samples to a wave
    const int64_t per_wg = (int64_t)kFwdTile * kGradWaves;
    const int nwg = (int)std::min<int64_t>((n_batch + per_wg - 1) / per_wg, kGuessWG);
    if (ws.fill_flags)
        hipLaunchKernelGGL(k_zero_flag, dim3(1), dim3(64), 0, st, ws.flags);
    else
        hipMemsetAsync(ws.flags, 0, sizeof(int), st);
    float bc1 = 1.f, bc2 = 1.f;
    if (adam) {
        const int64_t t = c->g_step + 1;
        bc1 = (float)(1.0 / (1.0 - pow(0.9, (double)t)));
        bc2 = (float)(1.0 / (1.0 - pow(0.999, (double)t)));
    }
    {
        StageTimer tm(c, AMOEBA_T_GUESS);
        const float lscale = (float)(kDebye * kDebye / (double)n_batch);
        hipLaunchKernelGGL(k_guess_grad, dim3(nwg), dim3(64 * kGradWaves), 0, st, n_batch, n_rows, idx, c->g_model, feat, basis,
                           guess_offsets(c), target, lscale, ws.part, ws.lossp, ws.flags);
        hipLaunchKernelGGL(k_guess_reduce, dim3((kNP + 63) / 64), dim3(64 * kRedGroups), 0, st, nwg, ws.part, ws.lossp,
                           grad_out, c->g_model, c->g_adam_m, c->g_adam_v, adam ? 1 : 0, lr, bc1, bc2, ws.scal,
                           ws.flags);
    }
    hipMemcpyAsync(c->flags_host, ws.flags, sizeof(int), hipMemcpyDeviceToHost, st);
    hipMemcpyAsync(c->g_scal_host, ws.scal, sizeof(double), hipMemcpyDeviceToHost, st);
    int rc = hip_check(c, hipStreamSynchronize(st), who);
    if (rc)
        return rc;
    if (c->flags_host[0] & kFlagBadIndex)
        return set_error(c, AMOEBA_E_INVALID, std::string(who) + ": idx entry outside [0, n_rows)");
    if (adam)
        c->g_step += 1;
    if (loss_out)
        *loss_out = c->g_scal_host[0];
    return AMOEBA_OK;
}

}  // namespace amoeba

using namespace amoeba;

extern "C" {

int amoeba_guess_set_model(amoeba_ctx* c, const float* model, int64_t n_floats)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!model || n_floats != kNM)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_set_model: need AMOEBA_GUESS_NMODEL floats");
    for (int64_t i = 0; i < n_floats; ++i)
        if (!std::isfinite(model[i]))
            return set_error(c, AMOEBA_E_NUMERIC, "amoeba_guess_set_model: non-finite model entry");
    int rc = guess_alloc_model(c);
    if (rc)
        return rc;
    hipStream_t st = c->stream;
    hipMemcpyAsync(c->g_model, model, sizeof(float) * kNM, hipMemcpyHostToDevice, st);
    hipMemsetAsync(c->g_adam_m, 0, sizeof(float) * kNP, st);
    hipMemsetAsync(c->g_adam_v, 0, sizeof(float) * kNP, st);
    c->g_step = 0;
    if ((rc = hip_check(c, hipStreamSynchronize(st), "amoeba_guess_set_model")))
        return rc;
    c->guess_loaded = true;
    return AMOEBA_OK;
}

int amoeba_guess_get_model(amoeba_ctx* c, float* model, int64_t n_floats)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!model || n_floats != kNM)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_get_model: need AMOEBA_GUESS_NMODEL floats");
    int rc = guess_ready(c, "amoeba_guess_get_model");
    if (rc)
        return rc;
    hipMemcpyAsync(model, c->g_model, sizeof(float) * kNM, hipMemcpyDeviceToHost, c->stream);
    return hip_check(c, hipStreamSynchronize(c->stream), "amoeba_guess_get_model");
}

int amoeba_guess_set_kind(amoeba_ctx* c, int32_t kind)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (kind != AMOEBA_GUESS_KIND_NEUMANN && kind != AMOEBA_GUESS_KIND_DELTA)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_set_kind: unknown kind");
    c->g_kind = kind;
    return AMOEBA_OK;
}

int amoeba_guess_set_reference(amoeba_ctx* c, const double* mu_ref, const double* e_ref)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!mu_ref || !e_ref)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_set_reference: NULL argument");
    const size_t n3 = 3 * (size_t)c->n;
    int rc;
    if (!c->g_ref && (rc = ctx_alloc(c, (void**)&c->g_ref, sizeof(double) * 2 * n3)))
        return rc;
    // copied on the stream, no host wait; the entries are checked for NaN/Inf where they are
    // used (AMOEBA_E_NUMERIC from that call)
    hipMemcpyAsync(c->g_ref, mu_ref, sizeof(double) * n3, hipMemcpyDeviceToDevice, c->stream);
    hipMemcpyAsync(c->g_ref + n3, e_ref, sizeof(double) * n3, hipMemcpyDeviceToDevice, c->stream);
    c->g_ref_set = true;
    return AMOEBA_OK;
}

// Checkpoint blob: header (48 bytes), model, Adam moments.
namespace {
struct GuessBlobHeader {
    char magic[8];
    uint32_t version;
    int32_t kind;
    int32_t nfeat, nbasis, hidden, nparam, nmodel, zero;
    int64_t step;
};
static_assert(sizeof(GuessBlobHeader) == 48, "blob header layout");
constexpr char kBlobMagic[8] = {'A', 'M', 'G', 'U', 'E', 'S', 'S', 0};
constexpr int64_t kBlobBytes = AMOEBA_GUESS_BLOB_BYTES;
static_assert(kBlobBytes == (int64_t)sizeof(GuessBlobHeader) + 4 * (kNM + 2 * kNP), "blob size");
}  // namespace

int amoeba_guess_save(amoeba_ctx* c, void* blob, int64_t* bytes)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!bytes)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_save: NULL bytes");
    if (!blob) {
        *bytes = kBlobBytes;
        return AMOEBA_OK;
    }
    if (*bytes < kBlobBytes)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_save: blob smaller than AMOEBA_GUESS_BLOB_BYTES");
    int rc = guess_ready(c, "amoeba_guess_save");
    if (rc)
        return rc;
    GuessBlobHeader h;
    std::copy(kBlobMagic, kBlobMagic + 8, h.magic);
    h.version = AMOEBA_GUESS_BLOB_VERSION;
    h.kind = c->g_kind;
    h.nfeat = kNF;
    h.nbasis = kNB;
    h.hidden = kH;
    h.nparam = kNP;
    h.nmodel = kNM;
    h.zero = 0;
    h.step = c->g_step;
    char* out = static_cast<char*>(blob);
    std::copy(reinterpret_cast<const char*>(&h), reinterpret_cast<const char*>(&h) + sizeof(h), out);
    float* f = reinterpret_cast<float*>(out + sizeof(h));
    hipStream_t st = c->stream;
    hipMemcpyAsync(f, c->g_model, sizeof(float) * kNM, hipMemcpyDeviceToHost, st);
    hipMemcpyAsync(f + kNM, c->g_adam_m, sizeof(float) * kNP, hipMemcpyDeviceToHost, st);
    hipMemcpyAsync(f + kNM + kNP, c->g_adam_v, sizeof(float) * kNP, hipMemcpyDeviceToHost, st);
    if ((rc = hip_check(c, hipStreamSynchronize(st), "amoeba_guess_save")))
        return rc;
    *bytes = kBlobBytes;
    return AMOEBA_OK;
}

int amoeba_guess_load(amoeba_ctx* c, const void* blob, int64_t bytes)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!blob || bytes != kBlobBytes)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: need a blob of AMOEBA_GUESS_BLOB_BYTES bytes");
    GuessBlobHeader h;
    const char* in = static_cast<const char*>(blob);
    std::copy(in, in + sizeof(h), reinterpret_cast<char*>(&h));
    if (!std::equal(kBlobMagic, kBlobMagic + 8, h.magic))
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: not a learned-guess checkpoint");
    if (h.version != AMOEBA_GUESS_BLOB_VERSION)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: unsupported checkpoint version");
    if (h.nfeat != kNF || h.nbasis != kNB || h.hidden != kH || h.nparam != kNP || h.nmodel != kNM || h.zero != 0)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: network shape differs from this library's");
    if (h.kind != AMOEBA_GUESS_KIND_NEUMANN && h.kind != AMOEBA_GUESS_KIND_DELTA)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: unknown kind");
    if (h.step < 0)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: negative step count");
    // the payload may be unaligned in the caller's buffer: copy it out before use
    std::vector<float> f(kNM + 2 * kNP);
    std::copy(in + sizeof(h), in + kBlobBytes, reinterpret_cast<char*>(f.data()));
    for (float x : f)
        if (!std::isfinite(x))
            return set_error(c, AMOEBA_E_NUMERIC, "amoeba_guess_load: non-finite entry");
    for (int i = 0; i < kNP; ++i)
        if (f[kNM + kNP + i] < 0.0f)
            return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_load: negative Adam second moment");
    int rc = guess_alloc_model(c);
    if (rc)
        return rc;
    hipStream_t st = c->stream;
    hipMemcpyAsync(c->g_model, f.data(), sizeof(float) * kNM, hipMemcpyHostToDevice, st);
    hipMemcpyAsync(c->g_adam_m, f.data() + kNM, sizeof(float) * kNP, hipMemcpyHostToDevice, st);
    hipMemcpyAsync(c->g_adam_v, f.data() + kNM + kNP, sizeof(float) * kNP, hipMemcpyHostToDevice, st);
    if ((rc = hip_check(c, hipStreamSynchronize(st), "amoeba_guess_load")))
        return rc;
    c->g_step = h.step;
    c->g_kind = h.kind;
    c->guess_loaded = true;
    return AMOEBA_OK;
}

int amoeba_guess_features(amoeba_ctx* c, const double* pos, const double* e_perm, float* feat_out, float* basis_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!e_perm || !feat_out || !basis_out)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_features: NULL argument");
    int rc = begin_config(c, pos, "amoeba_guess_features", false);
    if (rc)
        return rc;
    if ((rc = check_vec_finite(c, e_perm, 3 * (size_t)c->n, "e_perm")))
        return rc;
    launch_gather_vec(c, e_perm, c->v_e);
    if ((rc = guess_compute(c)))
        return rc;
    {
        StageTimer tm(c, AMOEBA_T_GUESS);
        hipLaunchKernelGGL(k_guess_features, dim3(nblk64(c->npad, 256)), dim3(256), 0, c->stream, c->npad, c->perm,
                           c->par_d, c->g_v, c->g_kind == AMOEBA_GUESS_KIND_NEUMANN ? c->g_radial : nullptr, 1,
                           feat_out, basis_out);
    }
    return guess_flags(c, "amoeba_guess_features");
}

int amoeba_guess_fit_norm(amoeba_ctx* c, const float* feat, int64_t n_rows)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!feat || n_rows < 1)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_fit_norm: need feat and n_rows >= 1");
    int rc = guess_ready(c, "amoeba_guess_fit_norm");
    if (rc)
        return rc;
    hipStream_t st = c->stream;
    const int nwg = (int)std::min<int64_t>(kRedBlocks, (n_rows + 255) / 256);
    StageTimer tm(c, AMOEBA_T_GUESS);
    for (int pass = 0; pass < 2; ++pass) {
        hipLaunchKernelGGL(k_guess_norm_partial, dim3(nwg), dim3(256), 0, st, n_rows, feat, pass, c->g_nmean,
                           c->g_npart);
        hipLaunchKernelGGL(k_guess_norm_final, dim3(1), dim3(256), 0, st, nwg, n_rows, c->g_npart, pass,
                           c->g_nmean, c->g_model);
    }
    return hip_check(c, hipStreamSynchronize(st), "amoeba_guess_fit_norm");
}

int amoeba_guess_forward(amoeba_ctx* c, const float* feat, const float* basis, int64_t n, float* mu_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!feat || !basis || !mu_out || n < 1)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_forward: NULL argument or n < 1");
    int rc = guess_ready(c, "amoeba_guess_forward");
    if (rc)
        return rc;
    {
        StageTimer tm(c, AMOEBA_T_GUESS);
        hipLaunchKernelGGL(k_guess_forward, dim3(forward_grid(n)), dim3(256), 0, c->stream, n,
                           c->g_model, feat, basis, guess_offsets(c), (const int*)nullptr, (double*)nullptr, mu_out);
    }
    return hip_check(c, hipStreamSynchronize(c->stream), "amoeba_guess_forward");
}

int amoeba_guess_gradient(amoeba_ctx* c, const float* feat, const float* basis, const float* target, int64_t n_rows,
                          const int32_t* idx, int64_t n_batch, float* grad_out, double* loss_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!grad_out)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_gradient: NULL grad_out");
    int rc = guess_ready(c, "amoeba_guess_gradient");
    if (rc)
        return rc;
    return guess_grad(c, feat, basis, target, n_rows, idx, n_batch, grad_out, false, 0.0f, loss_out,
                      "amoeba_guess_gradient", ctx_work(c));
}

int amoeba_guess_gradient_noalloc(amoeba_ctx* c, const float* feat, const float* basis, const float* target,
                                  int64_t n_rows, const int32_t* idx, int64_t n_batch, float* grad_out,
                                  double* loss_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!grad_out)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_gradient_noalloc: NULL grad_out");
    if (n_batch > AMOEBA_GUESS_NOALLOC_MAX_BATCH)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_gradient_noalloc: n_batch above "
                                              "AMOEBA_GUESS_NOALLOC_MAX_BATCH (8192)");
    int rc = guess_ready(c, "amoeba_guess_gradient_noalloc");
    if (rc)
        return rc;
    if (!c->g_scratch)
        return set_error(c, AMOEBA_E_STATE, "amoeba_guess_gradient_noalloc: scratch address unknown");
    return guess_grad(c, feat, basis, target, n_rows, idx, n_batch, grad_out, false, 0.0f, loss_out,
                      "amoeba_guess_gradient_noalloc", scratch_work(c));
}

int amoeba_guess_train_step(amoeba_ctx* c, const float* feat, const float* basis, const float* target,
                            int64_t n_rows, const int32_t* idx, int64_t n_batch, float lr, double* loss_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    int rc = guess_ready(c, "amoeba_guess_train_step");
    if (rc)
        return rc;
    return guess_grad(c, feat, basis, target, n_rows, idx, n_batch, nullptr, true, lr, loss_out,
                      "amoeba_guess_train_step", ctx_work(c));
}

int amoeba_guess_predict(amoeba_ctx* c, const double* pos, const double* e_perm, double* mu0_out)
{
    if (!c)
        return AMOEBA_E_INVALID;
    c->err.clear();
    if (!e_perm || !mu0_out)
        return set_error(c, AMOEBA_E_INVALID, "amoeba_guess_predict: NULL argument");
    int rc = guess_ready(c, "amoeba_guess_predict");
    if (rc)
        return rc;
    if ((rc = begin_config(c, pos, "amoeba_guess_predict", false)))
        return rc;
    if ((rc = check_vec_finite(c, e_perm, 3 * (size_t)c->n, "e_perm")))
        return rc;
    launch_gather_vec(c, e_perm, c->v_e);
    if ((rc = guess_compute(c)))
        return rc;
    guess_forward_slot(c, c->v_q);
    launch_scatter(c, c->v_q, mu0_out);
    return guess_flags(c, "amoeba_guess_predict");
}

}  // extern "C"
