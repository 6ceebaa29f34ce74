// Device helpers shared by the signing kernels (the per-unit walk and the
// shared-sample binned form): the lattice map of a draw and the exact
// crossing tests of Alg. 1's point-in-polygon step.
#pragma once

#include "internal.hpp"

namespace polymh {

// Lattice offset of a 32-bit half-draw: floor(h * W / 2^32).
template <bool POW2>
__device__ __forceinline__ uint32_t lattice(uint32_t h, uint32_t w, int32_t sh)
{
    if constexpr (POW2)
        return h >> sh;
    else
        return w ? __umulhi(h, w) : h;
}

// Edge record staged in LDS, oriented upward: (x_lo, y_lo, y_hi, x_hi - x_lo).
__device__ __forceinline__ int4 make_edge(int32_t x0, int32_t y0, int32_t x1, int32_t y1)
{
    return (y0 <= y1) ? make_int4(x0, y0, y1, x1 - x0) : make_int4(x1, y1, y0, x0 - x1);
}

// Crossing of the ray from (px, py) to +x with an upward edge, exact in FP64
// (edge endpoints and the sample lie in an MBR with sides < 2^26).
__device__ __forceinline__ bool crosses_fp64(int4 e, int32_t px, int32_t py)
{
    const bool straddle = (e.y <= py) & (py < e.z);
    const double t = (double)(px - e.x) * (double)(e.z - e.y);
    const double o = __fma_rn((double)e.w, (double)(py - e.y), -t);
    return straddle & (o > 0.0);
}

// The same test with an edge's products taken out of it: for coordinates
// relative to the MBR's corner, o = dx (py - y_lo) - (px - x_lo) dy =
// dx py - dy px + k, k = dy x_lo - dx y_lo.  With MBR sides below 2^26 every
// product and partial sum is an integer of at most 2^53 (dy px and dy x_lo
// differ by less than 2^52, as k's other product), so both forms are exact;
// this one is two fused multiply-adds and two compares.
struct __attribute__((aligned(16))) EdgeRec {
    double a, b, k;          // dx, -dy, dy x_lo - dx y_lo
    int32_t ylo;
    uint32_t h;              // y_hi - y_lo: straddled if y - y_lo, unsigned, is below
};

// `e` from make_edge; (x0, y0) the MBR's corner.
__device__ __forceinline__ EdgeRec make_edge_rec(int4 e, int32_t x0, int32_t y0)
{
    const double dx = (double)e.w, dy = (double)(e.z - e.y);
    EdgeRec r;
    r.a = dx;
    r.b = -dy;
    r.k = __fma_rn(dy, (double)(e.x - x0), -(dx * (double)(e.y - y0)));
    r.ylo = e.y - y0;
    r.h = (uint32_t)(e.z - e.y);
    return r;
}

// The lanes whose point, relative to the corner too (also as doubles), crosses
// their edge: a mask a comparison, combined as scalars (combined as lane
// values they are made numbers and compared again).
__device__ __forceinline__ uint64_t crosses_mask(const EdgeRec &e, int32_t py, double dpx, double dpy)
{
    return __ballot((uint32_t)(py - e.ylo) < e.h) & __ballot(__fma_rn(e.a, dpy, __fma_rn(e.b, dpx, e.k)) > 0.0);
}

__device__ __forceinline__ bool crosses_i128(const int32_t *v0, const int32_t *v1, int32_t px,
                                             int32_t py)
{
    int64_t xl = v0[0], yl = v0[1], xh = v1[0], yh = v1[1];
    if (yl > yh) {
        int64_t t = xl; xl = xh; xh = t;
        t = yl; yl = yh; yh = t;
    }
    if (!(yl <= py && py < yh)) return false;
    const __int128 o = (__int128)(xh - xl) * ((int64_t)py - yl) - (__int128)((int64_t)px - xl) * (yh - yl);
    return o > 0;
}

}  // namespace polymh
