// One-dimensional transforms of the plane PME passes (plane.hip): self-sorting (Stockham)
// mixed-radix FFTs whose first stage takes its points from wherever the pass finds them (global
// memory, the fixed-point sums of the spread) and whose last stage leaves its outputs in
// registers, so that a length N = A B with two supported radices crosses LDS once.  Radices up to
// 18 are nested from the small ones (2 to 7) with constant roots of unity, which gives two stages
// to every even product of 2, 3, 5 and 7 up to 180 that water boxes use, and to 192, 196, 210,
// 216, 224, 240, 252 and 256; other lengths run their middle stages in LDS.
#pragma once
#include "common.h"

namespace amoeba {

// Factorisation of a transform length (host-computed): at least two radices, those between the
// first and the last at most 9.
struct PlaneDim {
    int n, nr;
    int rad[12];
};

// Element (line l, point n) of a set of lines: l ls + n ps.
struct LineMap {
    int ls, ps;
    __device__ __forceinline__ int operator()(int l, int n) const { return l * ls + n * ps; }
};

// Quotient of non-negative integers a < 2^22 by b >= 1 through FP32: floor((a + 1/2) / b) with
// a correctly rounded reciprocal is off by at most (a + 1/2) / b * 2^-23 < 1 / (2b), less than the
// distance of (a + 1/2) / b to the nearest integer, so the truncation is exact.  Used for the
// line / point split of thread indices (an integer division is a long instruction sequence).
struct SmallDiv {
    int b;
    float inv;
    __device__ __forceinline__ explicit SmallDiv(int bb) : b(bb), inv(1.0f / (float)bb) {}
    __device__ __forceinline__ int quot(int a) const { return (int)(((float)a + 0.5f) * inv); }
};

template <typename C> __device__ __forceinline__ C cmul(C a, C b)
{
    return C{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename C> __device__ __forceinline__ C cadd(C a, C b) { return C{a.x + b.x, a.y + b.y}; }
template <typename C> __device__ __forceinline__ C csub(C a, C b) { return C{a.x - b.x, a.y - b.y}; }
// multiplication by SIGN i
template <int SIGN, typename C> __device__ __forceinline__ C mul_i(C a)
{
    return SIGN < 0 ? C{a.y, -a.x} : C{-a.y, a.x};
}

// cos and sin of 2 pi m / n for 0 <= m < n at compile time: reduced to the first octant, then
// the power series (below 1e-16 after ten terms).
struct UnitRoot {
    double c, s;
};
constexpr UnitRoot unit_root(int m, int n)
{
    // a / b turns with 0 <= a / b <= 1/8 after the symmetries
    long long a = 8LL * m, b = 8LL * n;
    bool neg_s = false, neg_c = false, swap = false;
    if (2 * a > b) {
        a = b - a;
        neg_s = true;
    }
    if (4 * a > b) {
        a = b / 2 - a;
        neg_c = true;
    }
    if (8 * a > b) {
        a = b / 4 - a;
        swap = true;
    }
    const double x = 2.0 * kPi * (double)a / (double)b;
    double c = 1.0, s = x, tc = 1.0, ts = x;
    for (int k = 1; k <= 10; ++k) {
        tc *= -x * x / ((2 * k - 1) * (2 * k));
        ts *= -x * x / ((2 * k) * (2 * k + 1));
        c += tc;
        s += ts;
    }
    const double cc = swap ? s : c, ss = swap ? c : s;
    return UnitRoot{neg_c ? -cc : cc, neg_s ? -ss : ss};
}

// The nested factors of a radix: RAD = P Q (Q = 1: a base transform).
constexpr int nest_q(int rad)
{
    switch (rad) {
    case 8: return 2;    // 4 x 2
    case 9: return 3;    // 3 x 3
    case 10: return 2;   // 5 x 2
    case 12: return 3;   // 4 x 3
    case 14: return 2;   // 7 x 2
    case 15: return 3;   // 5 x 3
    case 16: return 4;   // 4 x 4
    case 18: return 3;   // 6 x 3
    default: return 1;
    }
}

template <int RAD, int SIGN, typename C> __device__ __forceinline__ void dft(C (&v)[RAD]);

// a times exp(SIGN 2 pi i M / N)
template <int M, int N, int SIGN, typename C> __device__ __forceinline__ C root_mul(C a)
{
    using R = decltype(a.x);
    if constexpr (M % N == 0) {
        return a;
    } else if constexpr (4 * (M % N) == N) {
        return mul_i<SIGN>(a);
    } else if constexpr (2 * (M % N) == N) {
        return C{-a.x, -a.y};
    } else {
        constexpr UnitRoot w = unit_root(M % N, N);
        return cmul(a, C{(R)w.c, (R)SIGN * (R)w.s});
    }
}

template <int P, int Q, int SIGN, int I, typename C> __device__ __forceinline__ void nested_roots(C (&u)[P * Q])
{
    // u[k1 Q + n2] times w^(n2 k1)
    if constexpr (I < P * Q) {
        u[I] = root_mul<(I / Q) * (I % Q), P * Q, SIGN>(u[I]);
        nested_roots<P, Q, SIGN, I + 1>(u);
    }
}

// In-place RAD-point DFT: v[q] <- sum_r v[r] exp(SIGN 2 pi i r q / RAD).
template <int RAD, int SIGN, typename C> __device__ __forceinline__ void dft(C (&v)[RAD])
{
    using R = decltype(v[0].x);
    constexpr int Q = nest_q(RAD), P = RAD / Q;
    if constexpr (Q > 1) {
        C u[RAD];
#pragma unroll
        for (int n2 = 0; n2 < Q; ++n2) {
            C a[P];
#pragma unroll
            for (int n1 = 0; n1 < P; ++n1)
                a[n1] = v[Q * n1 + n2];
            dft<P, SIGN>(a);
#pragma unroll
            for (int k1 = 0; k1 < P; ++k1)
                u[k1 * Q + n2] = a[k1];
        }
        nested_roots<P, Q, SIGN, 0>(u);
#pragma unroll
        for (int k1 = 0; k1 < P; ++k1) {
            C b[Q];
#pragma unroll
            for (int n2 = 0; n2 < Q; ++n2)
                b[n2] = u[k1 * Q + n2];
            dft<Q, SIGN>(b);
#pragma unroll
            for (int k2 = 0; k2 < Q; ++k2)
                v[k1 + P * k2] = b[k2];
        }
    } else if constexpr (RAD == 2) {
        const C a = v[0], b = v[1];
        v[0] = cadd(a, b);
        v[1] = csub(a, b);
    } else if constexpr (RAD == 4) {
        const C a = cadd(v[0], v[2]), b = csub(v[0], v[2]), c = cadd(v[1], v[3]), d = mul_i<SIGN>(csub(v[1], v[3]));
        v[0] = cadd(a, c);
        v[2] = csub(a, c);
        v[1] = cadd(b, d);
        v[3] = csub(b, d);
    } else if constexpr (RAD == 6) {
        // pairs (r, r+3) first: even outputs are the 3-point DFT of the sums, odd outputs that of
        // the differences times exp(SIGN 2 pi i r / 6)
        C a[3], b[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            a[r] = cadd(v[r], v[r + 3]);
            b[r] = csub(v[r], v[r + 3]);
        }
        b[1] = root_mul<1, 6, SIGN>(b[1]);
        b[2] = root_mul<2, 6, SIGN>(b[2]);
        dft<3, SIGN>(a);
        dft<3, SIGN>(b);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            v[2 * r] = a[r];
            v[2 * r + 1] = b[r];
        }
    } else {
        static_assert(RAD == 3 || RAD == 5 || RAD == 7, "radix");
        // odd prime: with s_r = v_r + v_(RAD-r) and d_r = v_r - v_(RAD-r), outputs q and RAD - q are
        // v_0 + sum_r cos(2 pi r q / RAD) s_r +- SIGN i sum_r sin(2 pi r q / RAD) d_r
        constexpr int H = (RAD - 1) / 2;
        constexpr UnitRoot w[7] = {unit_root(0, RAD), unit_root(1, RAD), unit_root(2 % RAD, RAD),
                                   unit_root(3 % RAD, RAD), unit_root(4 % RAD, RAD), unit_root(5 % RAD, RAD),
                                   unit_root(6 % RAD, RAD)};
        C s[H], d[H];
#pragma unroll
        for (int r = 0; r < H; ++r) {
            s[r] = cadd(v[r + 1], v[RAD - 1 - r]);
            d[r] = csub(v[r + 1], v[RAD - 1 - r]);
        }
        const C v0 = v[0];
#pragma unroll
        for (int r = 0; r < H; ++r)
            v[0] = cadd(v[0], s[r]);
#pragma unroll
        for (int q = 1; q <= H; ++q) {
            C a = v0, b = C{(R)0, (R)0};
#pragma unroll
            for (int r = 1; r <= H; ++r) {
                const R c = (R)w[(r * q) % RAD].c, sn = (R)w[(r * q) % RAD].s;
                a.x += c * s[r - 1].x;
                a.y += c * s[r - 1].y;
                b.x += sn * d[r - 1].x;
                b.y += sn * d[r - 1].y;
            }
            const C ib = mul_i<SIGN>(b);
            v[q] = cadd(a, ib);
            v[RAD - q] = csub(a, ib);
        }
    }
}

// f(integral constant of the radix): one instantiation per supported radix.
template <int RAD> struct Radix {
    static constexpr int value = RAD;
};
template <typename F> __device__ __forceinline__ void with_small_radix(int rad, F&& f)
{
    switch (rad) {
    case 2: f(Radix<2>{}); break;
    case 3: f(Radix<3>{}); break;
    case 4: f(Radix<4>{}); break;
    case 5: f(Radix<5>{}); break;
    case 6: f(Radix<6>{}); break;
    case 7: f(Radix<7>{}); break;
    case 8: f(Radix<8>{}); break;
    default: f(Radix<9>{}); break;
    }
}
template <typename F> __device__ __forceinline__ void with_radix(int rad, F&& f)
{
    switch (rad) {
    case 2: f(Radix<2>{}); break;
    case 3: f(Radix<3>{}); break;
    case 4: f(Radix<4>{}); break;
    case 5: f(Radix<5>{}); break;
    case 6: f(Radix<6>{}); break;
    case 7: f(Radix<7>{}); break;
    case 8: f(Radix<8>{}); break;
    case 9: f(Radix<9>{}); break;
    case 10: f(Radix<10>{}); break;
    case 12: f(Radix<12>{}); break;
    case 14: f(Radix<14>{}); break;
    case 15: f(Radix<15>{}); break;
    case 16: f(Radix<16>{}); break;
    default: f(Radix<18>{}); break;
    }
}

// an opaque copy of an index: keeps the compiler from hoisting every radix's index arithmetic out
// of the switch (which would hold all of it in registers at once)
__device__ __forceinline__ int opaque(int i)
{
    asm volatile("" : "+v"(i));
    return i;
}

// The RAD points of a butterfly from get(r), point r times w^(r step) (w = exp(SIGN 2 pi i / N),
// tw[m] = exp(-2 pi i m / N)), at most kRootGroup points and roots in flight: the scheduling
// barriers keep a large radix from holding all of them in registers at once.
constexpr int kRootGroup = 6;
template <int RAD, int SIGN, typename C, typename G>
__device__ __forceinline__ void rooted_points(C (&v)[RAD], const C* tw, int step, G get)
{
#pragma unroll
    for (int r0 = 0; r0 < RAD; r0 += kRootGroup) {
#pragma unroll
        for (int r = r0; r < r0 + kRootGroup && r < RAD; ++r) {
            v[r] = get(r);
            if (r > 0) {
                C w = tw[r * step];
                if (SIGN > 0)
                    w.y = -w.y;
                v[r] = cmul(v[r], w);
            }
        }
        if (RAD > kRootGroup)
            __builtin_amdgcn_sched_barrier(0);
    }
}

// A middle stage (radix RAD, Ns points per finished sub-transform) of nl lines in buf, in place:
// butterfly j of a line reads points j + r N/RAD and writes output q to
// (j div Ns) Ns RAD + (j mod Ns) + q Ns.  Whole lines are processed per round, so each round reads
// its points into registers before the barrier and writes after it.
template <int RAD, int SIGN, typename C>
__device__ __forceinline__ void mid_stage(C* buf, int nl, int N, int Ns, const C* tw, LineMap am)
{
    const int nb = N / RAD, nt = blockDim.x;
    const int tstep = N / (Ns * RAD);
    const int lpr = max(1, nt / nb);
    const SmallDiv dnb(nb), dns(Ns);
    const int it = opaque(threadIdx.x);
    const int lq = dnb.quot(it), j = it - lq * nb;
    const int k = j - dns.quot(j) * Ns, o = (j - k) * RAD + k;
    for (int l0 = 0; l0 < nl; l0 += lpr) {
        const bool act = it < min(lpr, nl - l0) * nb;
        C v[RAD];
        if (act) {
            rooted_points<RAD, SIGN>(v, tw, k * tstep, [&](int r) { return buf[am(l0 + lq, j + r * nb)]; });
            dft<RAD, SIGN>(v);
        }
        __syncthreads();
        if (act) {
#pragma unroll
            for (int q = 0; q < RAD; ++q)
                buf[am(l0 + lq, o + q * Ns)] = v[q];
        }
        __syncthreads();
    }
}

// The stages between the first (radix ra, done) and the last (radix rb) of the radices of d in
// the given direction (1: rad[0] first, -1: rad[nr - 1] first).  Called after a barrier, ends with
// one.
template <int SIGN, typename C>
__device__ __forceinline__ void mid_stages(C* buf, int nl, const PlaneDim& d, int dir, const C* tw, LineMap am)
{
    int Ns = d.rad[dir > 0 ? 0 : d.nr - 1];
    for (int s = 1; s < d.nr - 1; ++s) {
        const int rad = d.rad[dir > 0 ? s : d.nr - 1 - s];
        with_small_radix(rad, [&](auto rc) {
            mid_stage<decltype(rc)::value, SIGN>(buf, nl, d.n, Ns, tw, am);
        });
        Ns *= rad;
    }
}

}  // namespace amoeba
