// Positions wrapped into the box, and the sort key of an atom in the list build's cell order
// (blocklist.hip).  Plain functions of numbers, so that a host test compiles them too.
#pragma once
#include <cfloat>
#include <cmath>

namespace amoeba {

// x in [0, L), periodically: x - L floor(x / L), and where the quotient's rounding leaves that outside
// (from about 1e16 L on it lies anywhere within the spacing of x; just below a multiple of L it is
// negative by a rounding) the exact remainder by repeated subtraction of L times a power of two, each
// subtraction exact.  Not finite: NaN.
__host__ __device__ __forceinline__ double wrap_box(double x, double L)
{
    double y = x - L * floor(x / L);
    y = y >= L ? y - L : y;
    if (y >= 0.0 && y < L)
        return y;
    double r = fabs(x);
    if (!(r <= DBL_MAX))
        return x - x;
    while (r >= L) {
        const double t = ldexp(L, ilogb(r) - ilogb(L));  // below 2 r
        r -= t <= r ? t : 0.5 * t;
    }
    r = x < 0.0 && r > 0.0 ? L - r : r;
    return r < L ? r : 0.0;
}

constexpr int kXBits = 12;  // of the position along a column
constexpr unsigned kKeyNonFinite = 0xffffffffu;

// Sort key of the wrapped position (x, y, z) in a box of edges bx, by, bz cut into ny x nz columns along
// x: col | xq, below ny nz 2^kXBits; kKeyNonFinite for a coordinate that is not a number.
__host__ __device__ __forceinline__ unsigned sort_key(double x, double y, double z, double bx, double by, double bz,
                                                      int ny, int nz)
{
    if (!(x == x && y == y && z == z))
        return kKeyNonFinite;
    const unsigned xmax = (1u << kXBits) - 1u;
    int cy = (int)(y / by * ny), cz = (int)(z / bz * nz);
    cy = cy < ny - 1 ? cy : ny - 1;
    cz = cz < nz - 1 ? cz : nz - 1;
    const unsigned col = (unsigned)(cz * ny + ((cz & 1) ? ny - 1 - cy : cy));
    unsigned q = (unsigned)(x / bx * (double)(1u << kXBits));
    q = q < xmax ? q : xmax;
    return (col << kXBits) | ((col & 1u) ? xmax - q : q);
}

// Bucket of a key; the last one is that of kKeyNonFinite, and no key lies beyond it.
__host__ __device__ __forceinline__ int bucket_of(unsigned key, int shift, int nbucket)
{
    const unsigned b = key == kKeyNonFinite ? (unsigned)nbucket : key >> shift;
    return b < (unsigned)nbucket ? (int)b : nbucket - 1;
}

}  // namespace amoeba
