// Polygons with holes and multipolygons as single rings.  Every ring of a
// shape after the first is joined to the first ring's first vertex v0 by a
// bridge walked out and back:
//   R0, v0, R1, R1[0], v0, R2, R2[0], v0, ..., Rk, Rk[0]   (closing to v0).
// The two edges of a bridge are the same segment in opposite directions, so
// they cross any ray together (the crossing parity of Alg. 1's membership
// test over all rings is unchanged), and they cancel in every boundary
// integral: the shoelace area, the centroid's fan moments and the Green's
// theorem sums of the refinement.  With filled rings counter-clockwise and
// holes clockwise, the joined ring therefore signs, refines and centres as
// the even-odd region of all the rings, and every kernel of the path takes
// it unchanged.
#include "internal.hpp"

#include <algorithm>

namespace polymh {

namespace {

struct Join {
    const int2 *__restrict__ xy;
    int64_t nv;
    const int64_t *__restrict__ roff;
    int64_t nr;
    const int64_t *__restrict__ prings;
    int64_t n;
    int2 *__restrict__ out;
    int64_t cap;
    int64_t *__restrict__ out_off;
    int32_t *__restrict__ bad;
};

// Shape p, rings r0 to r1 - 1 with vertices f0 to f1 - 1 (0 if `ok`, a range of
// rings, is false), by kRow lanes, kRow * kU vertices of a ring in flight.  Output
// offsets in closed form: shape p starts at ring_off[first ring] + 2 (first
// ring - p).  Malformed input (ring or vertex indices out of range, a shape
// without rings) raises the flag and is skipped; every write is checked
// against the output's capacity.
template <int kRow, int kU>
__device__ __forceinline__ void join_shape(const Join &g, int64_t p, int lane, bool ok, int64_t r0, int64_t r1, int64_t f0,
                                           int64_t f1)
{
    const int2 *__restrict__ xy = g.xy;
    const int64_t *__restrict__ roff = g.roff;
    int2 *__restrict__ out = g.out;
    const int64_t rings = ok ? r1 - r0 : 0;
    ok &= f0 >= 0 && f1 <= g.nv;
    int64_t first = f1, from = f0;          // end of the first ring
    for (int64_t i = 1; i < rings && ok; i++) {
        const int64_t f = roff[r0 + i];
        if (i == 1) first = f;
        ok = f >= from;
        from = f;
    }
    ok &= f1 >= from;
    const int64_t base = ok ? f0 + 2 * (r0 - p) : 0;
    if (lane == 0) {
        g.out_off[p] = base;
        if (p == g.n - 1) g.out_off[g.n] = ok ? f1 + 2 * (r1 - g.n) : 0;
    }
    if (!ok) {
        if (lane == 0 && g.bad) atomicOr(g.bad, 1);
        return;
    }
    const bool joined = r1 - r0 > 1;
    const int2 v0 = first > f0 ? xy[f0] : make_int2(0, 0);
    int64_t pos = base;
    bool short_ring = false;
    const int64_t end = base + (f1 - f0) + 2 * (r1 - r0 - 1);
    if (base < 0 || end > g.cap) {
        if (lane == 0 && g.bad) atomicOr(g.bad, 1);
        return;
    }
    int64_t a = f0;
    for (int64_t r = r0; r < r1; r++) {
        const int64_t e = r + 1 == r1 ? f1 : r == r0 ? first : roff[r + 1], len = e - a;
        short_ring |= len < 3;
        for (int64_t i0 = lane; i0 < len; i0 += kRow * kU) {
            int2 v[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) v[u] = xy[a + (i0 + kRow * u < len ? i0 + kRow * u : i0)];
#pragma unroll
            for (int u = 0; u < kU; u++)
                if (i0 + kRow * u < len) out[pos + i0 + kRow * u] = v[u];
        }
        pos += len;
        if (joined && r == r0) {
            if (lane == 0) out[pos] = v0;
            pos += 1;
        } else if (joined) {
            if (lane == 0) out[pos] = len > 0 ? xy[a] : v0;
            pos += 1;
            if (r + 1 < r1) {
                if (lane == 0) out[pos] = v0;
                pos += 1;
            }
        }
        a = e;
    }
    if (short_ring && lane == 0 && g.bad) atomicOr(g.bad, 1);
}

// `per` shapes (1 or 4) share a wavefront, a 16-lane row each; a shape whose
// rings have more than 64 vertices on average, 128 in all, is taken by the
// whole wavefront afterwards.  Bound: the latency of the chain rings ->
// offsets -> vertices.  100,000 shapes of 82 vertices take 43 us with four a
// wavefront, 79 with one; a ring of 1 M vertices 1.1 ms by the wavefront, 9.7
// by a row; four of 300,000 0.5 ms with a wavefront each, which costs nothing
// while the CUs hold them all.
__global__ __launch_bounds__(256) void k_join(Join g, int per)
{
    const int lane = threadIdx.x & 63, row = lane >> 4;
    const int64_t step = (((int64_t)gridDim.x * blockDim.x) >> 6) * per;
    for (int64_t p0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * per; p0 < g.n; p0 += step) {
        const int64_t p = p0 + row;
        const bool in = row < per && p < g.n;
        int64_t r0 = 0, r1 = 0, f0 = 0, f1 = 0;
        if (in) {
            r0 = g.prings[p];
            r1 = g.prings[p + 1];
        }
        const bool ok = 0 <= r0 && r0 < r1 && r1 <= g.nr;
        if (ok) {
            f0 = g.roff[r0];
            f1 = g.roff[r1];
        }
        // as a difference that cannot overflow, whatever the offsets are
        const uint64_t m = (uint64_t)f1 - (uint64_t)f0;
        const bool big = ok && m > 128 && m / 64 > (uint64_t)(r1 - r0);
        if (in && !big) join_shape<16, 4>(g, p, lane & 15, ok, r0, r1, f0, f1);
        uint64_t todo = __ballot(big && (lane & 15) == 0);
        while (todo) {
            const int r = __builtin_ctzll(todo);
            todo &= todo - 1;
            join_shape<64, 8>(g, p0 + (r >> 4), lane, true, (int64_t)dpp::readlane64((uint64_t)r0, r),
                              (int64_t)dpp::readlane64((uint64_t)r1, r), (int64_t)dpp::readlane64((uint64_t)f0, r),
                              (int64_t)dpp::readlane64((uint64_t)f1, r));
        }
    }
}

}  // namespace

polymh_status launch_join_rings(const int32_t *xy, int64_t nv, const int64_t *ring_off, int64_t nr,
                                const int64_t *poly_rings, int64_t n, int32_t *out_xy, int64_t out_cap,
                                int64_t *out_off, int32_t *bad, hipStream_t s)
{
    if (n == 0) return POLYMH_OK;
    const int per = n <= 16 * (int64_t)cu_count() ? 1 : 4;
    const int64_t blocks = std::min<int64_t>((n + 4 * per - 1) / (4 * per), 65536);
    const Join g{reinterpret_cast<const int2 *>(xy), nv, ring_off, nr, poly_rings, n,
                 reinterpret_cast<int2 *>(out_xy), out_cap, out_off, bad};
    hipLaunchKernelGGL(k_join, dim3((unsigned)blocks), dim3(256), 0, s, g, per);
    return check_launch("join_rings");
}

}  // namespace polymh
