// Root cube and Morton keys, shared by the build's kernels.  Internal to
// libtc.  Every expression here decides an integer or the cube itself, so
// all callers must compute exactly the same values (compiled without
// floating-point contraction).
#pragma once

#include "tc_internal.h"

#include <math.h>

namespace tc {
namespace keys {

// The input's bodies packed four values to a record, (x, y, z, m) with z = 0
// in 2D, in the input's order: the gather then reads one record per body
// instead of a position and a mass from two places.
template <typename T> struct Packed;
template <> struct Packed<float> { using type = float4; };
template <> struct Packed<double> { using type = double4; };

static __device__ __forceinline__ uint32_t spread3(uint32_t x) {   // bit b -> bit 3b (11 bits)
    x = (x | x << 16) & 0xff0000ffu;
    x = (x | x << 8) & 0x0f00f00fu;
    x = (x | x << 4) & 0xc30c30c3u;
    x = (x | x << 2) & 0x49249249u;
    return x;
}

static __device__ __forceinline__ uint32_t spread2(uint32_t x) {   // bit b -> bit 2b (16 bits)
    x = (x | x << 8) & 0x00ff00ffu;
    x = (x | x << 4) & 0x0f0f0f0fu;
    x = (x | x << 2) & 0x33333333u;
    x = (x | x << 1) & 0x55555555u;
    return x;
}

template <int D>
static __device__ __forceinline__ uint32_t quantise(double x, double lo, double scale) {
    constexpr int L = D == 3 ? 21 : 31;
    const double top = (double)((1ull << L) - 1ull);
    double f = floor((x - lo) * scale);
    if (!(f >= 0.0)) f = 0.0;                     // also catches NaN
    if (f > top) f = top;
    return (uint32_t)f;
}

// The key of a position: levels from the most significant digit down, x the
// highest bit of each digit.  The bits are spread in 32-bit halves (the low
// 10 bits of each coordinate and the rest in 3D, 16 and the rest in 2D):
// about a third of the instructions of 64-bit shifts, and a sample sort's
// blocks compute some keys more than once.
template <int D>
static __device__ __forceinline__ uint64_t morton(double x, double y, double z, const double* lo, double scale) {
    const uint32_t qx = quantise<D>(x, lo[0], scale), qy = quantise<D>(y, lo[1], scale);
    if (D == 3) {
        const uint32_t qz = quantise<D>(z, lo[2], scale);
        const uint32_t l = spread3(qx & 1023u) << 2 | spread3(qy & 1023u) << 1 | spread3(qz & 1023u);   // 30 bits
        const uint64_t hx = spread3(qx >> 10), hy = spread3(qy >> 10), hz = spread3(qz >> 10);          // 31 bits each
        return (hx << 32 | hy << 31 | hz << 30) | l;
    }
    const uint32_t l = spread2(qx & 0xffffu) << 1 | spread2(qy & 0xffffu);
    const uint32_t h = spread2(qx >> 16) << 1 | spread2(qy >> 16);
    return (uint64_t)h << 32 | l;
}

// The root cube from the per-axis extremes: the corner, the side (the next
// power of two at or above the largest extent, 1 if that is 0) and the
// quantisation scale 2^L / side.
struct Cube {
    double lo[3], size, scale;
};

static __device__ __forceinline__ Cube make_cube(const double* lo, const double* hi, int dim) {
    Cube c;
    const int L = dim == 3 ? 21 : 31;
    double ext = 0.0;
    for (int a = 0; a < 3; ++a) {
        if (a >= dim) {
            c.lo[a] = 0.0;
            continue;
        }
        c.lo[a] = isfinite(lo[a]) ? lo[a] : 0.0;  // else no finite coordinate on this axis
        const double e = hi[a] - lo[a];
        if (e > ext) ext = e;
    }
    c.size = 1.0;
    if (ext > 0.0 && isfinite(ext)) {
        int e2;
        const double f = frexp(ext, &e2);         // ext = f 2^e2, f in [0.5, 1)
        c.size = (f == 0.5) ? ext : ldexp(1.0, e2);
    }
    int e2;
    frexp(c.size, &e2);                           // size = 2^(e2-1)
    c.scale = ldexp(1.0, L - (e2 - 1));
    return c;
}

static __device__ __forceinline__ void store_cube(const Cube& c, bool bad, DevParams* prm) {
    for (int a = 0; a < 3; ++a) prm->lo[a] = c.lo[a];
    prm->size = c.size;
    prm->scale = c.scale;
    prm->status = bad ? kFlagNonFinite : 0u;
    prm->ncells = 0;
}

}  // namespace keys
}  // namespace tc
