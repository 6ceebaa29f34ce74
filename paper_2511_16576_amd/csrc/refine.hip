// Exact Jaccard refinement (Sec. 1: J = area(P n Q) / area(P u Q)).
//
// area(P n Q) by Green's theorem: the boundary of P n Q is made of the parts
// of P's edges inside Q and the parts of Q's edges inside P.  Along a straight
// edge (a, b) the integrand (x dy - y dx)/2 is the constant cross(a, b)/2, so
// an edge contributes cross(a, b)/2 times the fraction of it that lies inside
// the other polygon.  That fraction is w(a) + sum over crossings of
// s * (1 - t): w(a) is the membership of the edge's start, each crossing at
// parameter t enters (s = +1) or leaves (s = -1) the other polygon.  No
// sorting of crossings is needed, so every (edge, edge) pair is independent.
//
// Degenerate contacts (shared vertices, T-junctions, collinear overlaps) are
// resolved by a consistent symbolic perturbation: Q is translated by
// (eps, eps^2), eps -> 0+.  Every orientation predicate is then nonzero (its
// sign falls back to a fixed tie-break of the edge direction), crossings are
// proper, and the area is continuous in eps, so taking the combinatorics of
// the perturbed position with the parameters t and cross products at eps = 0
// gives exactly area(P n Q).  Orientations are exact: coordinate differences
// below 2^26 make each FP64 product exact (128-bit integers beyond that).
//
// General form (below): one wavefront per candidate pair, lanes take the edges
// of one polygon while the other's vertices are read 64 at a time.
#include <algorithm>

#include "internal.hpp"
#include "refine_keys.hpp"

namespace polymh {

namespace {

template <bool WIDE>
struct Geo;

// Exact FP64 orientation (differences < 2^26).
template <>
struct Geo<false> {
    using C = double;
    __device__ static __forceinline__ double orient(double ax, double ay, double bx, double by,
                                                    double cx, double cy)
    {
        const double t = (by - ay) * (cx - ax);
        return __fma_rn(bx - ax, cy - ay, -t);
    }
    __device__ static __forceinline__ double conv(int64_t v) { return (double)v; }
    __device__ static __forceinline__ int sgn(double o) { return (o > 0) - (o < 0); }
    __device__ static __forceinline__ double val(double o) { return o; }
};

// Exact 128-bit orientation sign for wide pairs; the FP64 value (used only
// for crossing parameters) is rounded.
template <>
struct Geo<true> {
    using C = int64_t;
    struct O {
        __int128 v;
        double d;
    };
    __device__ static __forceinline__ O orient(int64_t ax, int64_t ay, int64_t bx, int64_t by,
                                               int64_t cx, int64_t cy)
    {
        O o;
        o.v = (__int128)(bx - ax) * (cy - ay) - (__int128)(by - ay) * (cx - ax);
        o.d = (double)(bx - ax) * (double)(cy - ay) - (double)(by - ay) * (double)(cx - ax);
        return o;
    }
    __device__ static __forceinline__ int64_t conv(int64_t v) { return v; }
    __device__ static __forceinline__ int sgn(O o) { return (o.v > 0) - (o.v < 0); }
    __device__ static __forceinline__ double val(O o) { return o.d; }
};

__device__ __forceinline__ double i128_to_double(__int128 v)
{
    const bool neg = v < 0;
    const unsigned __int128 u = neg ? (unsigned __int128)(-v) : (unsigned __int128)v;
    const double r = (double)(uint64_t)(u >> 64) * 18446744073709551616.0 + (double)(uint64_t)u;
    return neg ? -r : r;
}

// Sign of orient(a, b, X + delta) when orient(a, b, X) = 0: -sign(dy), else sign(dx).
__device__ __forceinline__ int tb_shift_point(int64_t dx, int64_t dy)
{
    return dy != 0 ? (dy > 0 ? -1 : 1) : (dx > 0 ? 1 : -1);
}
// Sign of orient(c + delta, d + delta, X) when orient(c, d, X) = 0: sign(dy'), else -sign(dx').
__device__ __forceinline__ int tb_shift_edge(int64_t dx, int64_t dy)
{
    return dy != 0 ? (dy > 0 ? 1 : -1) : (dx > 0 ? -1 : 1);
}

// 1/d: the hardware reciprocal (relative error about 2^-24 on gfx950) and
// one Newton step (error about 2^-48, measured), ample for crossing
// parameters summed into areas checked to 1e-9.
__device__ __forceinline__ double rcp_refined(double d)
{
    const double r = __builtin_amdgcn_rcp(d);
    return __fma_rn(r, __fma_rn(-d, r, 1.0), r);
}

__device__ __forceinline__ double wave_sum(double v) { return wave_sum_f64(v); }
__device__ __forceinline__ int32_t wmin(int32_t v) { return wave_min32(v); }
__device__ __forceinline__ int32_t wmax(int32_t v) { return wave_max32(v); }

struct PairIn {
    const int32_t *P;   // data polygon vertices
    int32_t n;
    const int32_t *Q;   // query polygon vertices (uniform)
    int32_t m;
    int64_t ox, oy;     // local origin
    int32_t qmbr[4];
    int sq;             // orientation of Q (+1 counter-clockwise, -1 clockwise)
    int sp;             // orientation of P
};

// The other ring's vertices are read 64 at a time, one per lane, by a
// wavefront whose lanes are all active, and handed to the edge loop by
// readlane: one coalesced load per 64 iterations instead of a dependent load
// in each.  Vertex (jb + lane + 1) mod m of an m-vertex ring.
__device__ __forceinline__ int2 next_vertex_block(const int32_t *V, int m, int jb, int lane)
{
    const int j = jb + lane + 1;
    const int jn = j < m ? j : (j == m ? 0 : 0);
    return *reinterpret_cast<const int2 *>(V + 2 * jn);
}

// Sum over P's edges of cross(a, b) * (fraction of the edge inside Q + delta),
// plus the exact doubled area of P (shoelace about the origin).
// Only the 64-edge blocks b0, b0 + bstride, ... of P (a split pair); (0, 1)
// takes them all.
template <bool WIDE>
__device__ void edges_in_other_P(const PairIn &in, int lane, double &sum, int64_t &area2, int b0 = 0,
                                 int bstride = 1)
{
    using G = Geo<WIDE>;
    sum = 0.0;
    area2 = 0;
    for (int eb = 64 * b0; eb < in.n; eb += 64 * bstride) {
        // every lane stays in the loop (the vertex blocks need all of them)
        const int e = eb + lane;
        const bool live = e < in.n;
        const int ei = live ? e : 0;
        const int f = (ei + 1 == in.n) ? 0 : ei + 1;
        const int64_t ax = (int64_t)in.P[2 * ei] - in.ox, ay = (int64_t)in.P[2 * ei + 1] - in.oy;
        const int64_t bx = (int64_t)in.P[2 * f] - in.ox, by = (int64_t)in.P[2 * f + 1] - in.oy;
        const __int128 cr = (__int128)ax * by - (__int128)bx * ay;
        if (live) area2 += (int64_t)cr;
        const int64_t ex0 = min(ax, bx) + in.ox, ex1 = max(ax, bx) + in.ox;
        const int64_t ey0 = min(ay, by) + in.oy, ey1 = max(ay, by) + in.oy;
        const bool act = live && !(ax == bx && ay == by) &&
                         !(ex1 < in.qmbr[0] || ex0 > in.qmbr[2] || ey1 < in.qmbr[1] || ey0 > in.qmbr[3]);
        if (__ballot(act) == 0) continue;
        const int tbe = tb_shift_point(bx - ax, by - ay);
        const auto Ax = G::conv(ax), Ay = G::conv(ay), Bx = G::conv(bx), By = G::conv(by);
        int64_t cx = (int64_t)in.Q[0] - in.ox, cy = (int64_t)in.Q[1] - in.oy;
        auto oc = G::orient(Ax, Ay, Bx, By, G::conv(cx), G::conv(cy));
        int sc = G::sgn(oc);
        sc = sc ? sc : tbe;
        int w = 0;
        double acc = 0.0;
        for (int jb = 0; jb < in.m; jb += 64) {
          const int2 blk = next_vertex_block(in.Q, in.m, jb, lane);
          const int cnt = min(64, in.m - jb);
          for (int t = 0; t < cnt; t++) {
            const int64_t dx = (int64_t)__builtin_amdgcn_readlane(blk.x, t) - in.ox;
            const int64_t dy = (int64_t)__builtin_amdgcn_readlane(blk.y, t) - in.oy;
            if (!act) {
                cx = dx; cy = dy;
                continue;
            }
            const auto Dx = G::conv(dx), Dy = G::conv(dy), Cx = G::conv(cx), Cy = G::conv(cy);
            auto od = G::orient(Ax, Ay, Bx, By, Dx, Dy);
            int sd = G::sgn(od);
            sd = sd ? sd : tbe;
            if (cx != dx || cy != dy) {
                const int tbf = tb_shift_edge(dx - cx, dy - cy);
                const auto oa = G::orient(Cx, Cy, Dx, Dy, Ax, Ay);
                const auto ob = G::orient(Cx, Cy, Dx, Dy, Bx, By);
                int sa = G::sgn(oa), sb = G::sgn(ob);
                sa = sa ? sa : tbf;
                sb = sb ? sb : tbf;
                // membership of a in Q + delta: half-open crossing rule
                w ^= ((cy >= ay) != (dy >= ay)) & (sa == (dy > cy ? 1 : -1));
                if ((sc != sd) & (sa != sb)) {
                    const double va = G::val(oa), vb = G::val(ob);
                    acc += (double)sb * (-vb) * rcp_refined(va - vb);
                }
            }
            cx = dx; cy = dy; sc = sd;
          }
        }
        // crossings change Q's winding number by sb; membership = sq * winding
        if (act) sum += i128_to_double(cr) * ((double)w + (double)in.sq * acc);
    }
}

// Sum over Q's edges (shifted by delta) of cross(c, d) * (fraction inside P),
// plus the exact doubled area of Q.
template <bool WIDE>
__device__ void edges_in_other_Q(const PairIn &in, const int32_t *pmbr, int lane, double &sum,
                                 int64_t &area2, int b0 = 0, int bstride = 1)
{
    using G = Geo<WIDE>;
    sum = 0.0;
    area2 = 0;
    for (int fb = 64 * b0; fb < in.m; fb += 64 * bstride) {
        // every lane stays in the loop (the vertex blocks need all of them)
        const int f = fb + lane;
        const bool live = f < in.m;
        const int fi = live ? f : 0;
        const int g = (fi + 1 == in.m) ? 0 : fi + 1;
        const int64_t cx = (int64_t)in.Q[2 * fi] - in.ox, cy = (int64_t)in.Q[2 * fi + 1] - in.oy;
        const int64_t dx = (int64_t)in.Q[2 * g] - in.ox, dy = (int64_t)in.Q[2 * g + 1] - in.oy;
        const __int128 cr = (__int128)cx * dy - (__int128)dx * cy;
        if (live) area2 += (int64_t)cr;
        const int64_t fx0 = min(cx, dx) + in.ox, fx1 = max(cx, dx) + in.ox;
        const int64_t fy0 = min(cy, dy) + in.oy, fy1 = max(cy, dy) + in.oy;
        const bool act = live && !(cx == dx && cy == dy) &&
                         !(fx1 < pmbr[0] || fx0 > pmbr[2] || fy1 < pmbr[1] || fy0 > pmbr[3]);
        if (__ballot(act) == 0) continue;
        const int tbf = tb_shift_edge(dx - cx, dy - cy);
        const auto Cx = G::conv(cx), Cy = G::conv(cy), Dx = G::conv(dx), Dy = G::conv(dy);
        int64_t ax = (int64_t)in.P[0] - in.ox, ay = (int64_t)in.P[1] - in.oy;
        auto oa = G::orient(Cx, Cy, Dx, Dy, G::conv(ax), G::conv(ay));
        int sa = G::sgn(oa);
        sa = sa ? sa : tbf;
        int w = 0;
        double acc = 0.0;
        for (int ib = 0; ib < in.n; ib += 64) {
          const int2 blk = next_vertex_block(in.P, in.n, ib, lane);
          const int cnt = min(64, in.n - ib);
          for (int t = 0; t < cnt; t++) {
            const int64_t bx = (int64_t)__builtin_amdgcn_readlane(blk.x, t) - in.ox;
            const int64_t by = (int64_t)__builtin_amdgcn_readlane(blk.y, t) - in.oy;
            if (!act) {
                ax = bx; ay = by;
                continue;
            }
            const auto Ax = G::conv(ax), Ay = G::conv(ay), Bx = G::conv(bx), By = G::conv(by);
            auto ob = G::orient(Cx, Cy, Dx, Dy, Bx, By);
            int sb = G::sgn(ob);
            sb = sb ? sb : tbf;
            if (ax != bx || ay != by) {
                const int tbe = tb_shift_point(bx - ax, by - ay);
                const auto oc = G::orient(Ax, Ay, Bx, By, Cx, Cy);
                const auto od = G::orient(Ax, Ay, Bx, By, Dx, Dy);
                int sc = G::sgn(oc), sd = G::sgn(od);
                sc = sc ? sc : tbe;
                sd = sd ? sd : tbe;
                // membership of c + delta in P: half-open crossing rule
                w ^= ((ay > cy) != (by > cy)) & (sc == (by > ay ? 1 : -1));
                if ((sa != sb) & (sc != sd)) {
                    const double vc = G::val(oc), vd = G::val(od);
                    acc += (double)sd * (-vd) * rcp_refined(vc - vd);
                }
            }
            ax = bx; ay = by; sa = sb;
          }
        }
        if (act) sum += i128_to_double(cr) * ((double)w + (double)in.sp * acc);
    }
}

__device__ __forceinline__ int64_t poly_area2(const int32_t *v, int32_t n, int64_t ox, int64_t oy,
                                             int lane)
{
    int64_t a = 0;
    for (int i = lane; i < n; i += 64) {
        const int j = (i + 1 == n) ? 0 : i + 1;
        const int64_t ax = (int64_t)v[2 * i] - ox, ay = (int64_t)v[2 * i + 1] - oy;
        const int64_t bx = (int64_t)v[2 * j] - ox, by = (int64_t)v[2 * j + 1] - oy;
        a += (int64_t)((__int128)ax * by - (__int128)bx * ay);
    }
    return wave_sum_i64(a);
}

__device__ __forceinline__ void poly_mbr(const int32_t *v, int32_t n, int lane, int32_t *out)
{
    int32_t mnx = INT32_MAX, mny = INT32_MAX, mxx = INT32_MIN, mxy = INT32_MIN;
    for (int i = lane; i < n; i += 64) {
        mnx = min(mnx, v[2 * i]); mxx = max(mxx, v[2 * i]);
        mny = min(mny, v[2 * i + 1]); mxy = max(mxy, v[2 * i + 1]);
    }
    out[0] = wmin(mnx); out[1] = wmin(mny); out[2] = wmax(mxx); out[3] = wmax(mxy);
}

// ---------------------------------------------------------------------------
// Tiled form.  The two boundaries are cut into chunks of 8 edges; only chunk
// pairs whose boxes overlap (tiles of 8 x 8 edge pairs) are tested.  Each
// crossing is found once and credited to both polygons.  The membership of
// each edge's start is not tested directly: it is the membership of the
// ring's first vertex plus the running sum of the crossing signs met along
// the ring, so with S_e the net sign of edge e's crossings,
//   sum_e cr_e * I(e) = sum_e cr_e * (w_0 + s * sum_{e' < e} S_e')
//                       + s * sum_{crossings} cr_e * sign * (1 - t).
// Q (the query) is staged once per workgroup; each wavefront stages groups of
// data polygons (k_refine) or windows (k_refine_wide).  Pairs with a polygon beyond kTileCap edges, or coordinate spans of
// 2^26 and more, take the general per-edge form above.
//
// Work layout: overlapping tiles are compacted into a per-wavefront list and
// taken 8 at a time; lane (slot, j) keeps edge j of its tile's Q chunk in
// registers and sweeps the 8 edges of the tile's P chunk.  With e = b - a,
// f = d - c, r = c - a and X = cross(e, f) the four orientations are
//   orient(a,b,c) = cross(e, r),  orient(a,b,d) = orient(a,b,c) + X,
//   orient(c,d,a) = cross(r, f),  orient(c,d,b) = orient(c,d,a) - X,
// all exact integers in FP64 (differences < 2^26).  The symbolic tie-break is
// folded into one compare: against a threshold of -1/2 or +1/2 for P's
// edges, and for Q's edges a floating-point class test whose "positive" set
// is {+denormal, +normal, +inf}, plus both zeros when the tie resolves to +1.
// Rings are padded with copies of vertex 0, so edges past the end are
// zero-length and can never cross: no per-lane bounds checks in the sweep.

constexpr int kTileCap = 512;
constexpr int kRingLds = kTileCap + 16;   // ring vertices incl. padding
constexpr int kWavesPerBlock = 4;
constexpr int kListCap = 256;             // per-wavefront ring of tile entries (< 16 pending + 128 new)
constexpr int kUnitCap = 256;             // per-wavefront ring of sweep units (< 64 pending + 128 new)
constexpr int kClassPos = (1 << 7) | (1 << 8) | (1 << 9);
constexpr int kClassPosZ = kClassPos | (1 << 5) | (1 << 6);

struct RingLds {
    int2 *v;            // vertices relative to the origin; v[n..] repeat v[0]
    int4 *box;          // per 8-edge chunk: xmin, ymin, xmax, ymax
    int64_t *suf;       // Q only: suffix sums of the edges' cross products (see below)
};

// Tie-break class set of a shifted Q edge (c + delta, d + delta), f = d - c,
// for orientations of points of P: a zero counts as positive when fy > 0, or
// fy = 0 and fx < 0 (zero-length edges never cross either way).
__device__ __forceinline__ int q_edge_class(int fx, int fy)
{
    return (fy > 0 || (fy == 0 && fx < 0)) ? kClassPosZ : kClassPos;
}

// Tie-break threshold of a P edge (e = b - a) for orientations of points of
// Q + delta: a zero counts as positive when the edge points down, or is
// horizontal and points right.  Orientations are integers, so o > -1/2 is
// o >= 0 and o > +1/2 is o > 0.  fma(ey, 2^32, -ex) carries the sign of ey,
// or of -ex when ey = 0 (|ex| < 2^26), and the threshold takes that sign.
__device__ __forceinline__ double p_edge_threshold(double ex, double ey)
{
    return copysign(0.5, __fma_rn(ey, 4294967296.0, -ex));
}

__device__ __forceinline__ double orient_d(int2 a, int2 b, int2 c)
{
    const double t = (double)(b.y - a.y) * (double)(c.x - a.x);
    return __fma_rn((double)(b.x - a.x), (double)(c.y - a.y), -t);
}

__device__ __forceinline__ int sgn_tb(double o, int tb) { return o > 0 ? 1 : (o < 0 ? -1 : tb); }

__device__ __forceinline__ int lanes_below(uint64_t mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
}

// Stage a ring relative to the origin into entries [0, pad_to), entries from
// n on repeating vertex 0.
__device__ void stage_ring(const int32_t *src, int n, int pad_to, int64_t ox, int64_t oy, RingLds R,
                           int t0, int nt)
{
    for (int i = t0; i < pad_to; i += nt) {
        const int k = i < n ? i : 0;
        R.v[i] = make_int2((int)((int64_t)src[2 * k] - ox), (int)((int64_t)src[2 * k + 1] - oy));
    }
}

__device__ void chunk_boxes(RingLds R, int n, int t0, int nt)
{
    const int nc = (n + 7) >> 3;
    for (int c = t0; c < nc; c += nt) {
        int x0 = INT32_MAX, y0 = INT32_MAX, x1 = INT32_MIN, y1 = INT32_MIN;
        const int e1 = min(n, 8 * c + 8);
        for (int v = 8 * c; v <= e1; v++) {
            const int2 p = R.v[v];
            x0 = min(x0, p.x); y0 = min(y0, p.y); x1 = max(x1, p.x); y1 = max(y1, p.y);
        }
        R.box[c] = make_int4(x0, y0, x1, y1);
    }
}

// Wavefront form for P (lane = chunk, up to MAXC chunks): the chunk boxes.
// The 9 vertices of a chunk are read at once (indices clamped to the ring's
// end, which only repeats a vertex) so their LDS latencies overlap.
template <int MAXC>
__device__ void chunk_boxes_p(RingLds R, int n, int lane)
{
    const int nc = (n + 7) >> 3;
#pragma unroll
    for (int c0 = 0; c0 < MAXC; c0 += 64) {
        int c = c0 + lane;
        // recomputed here rather than hoisted out of a caller's loop over
        // pairs, where the compiler would keep 8 c + 1 and 8 c + 8 live in
        // registers (or spill them) across the whole pair
        asm volatile("" : "+v"(c));
        if (c < nc) {
            const int e1 = min(n, 8 * c + 8);
            int2 p[9];
#pragma unroll
            for (int j = 0; j < 9; j++) p[j] = R.v[min(8 * c + j, e1)];
            int x0 = p[0].x, y0 = p[0].y, x1 = p[0].x, y1 = p[0].y;
#pragma unroll
            for (int j = 1; j < 9; j++) {
                x0 = min(x0, p[j].x); y0 = min(y0, p[j].y); x1 = max(x1, p[j].x); y1 = max(y1, p[j].y);
            }
            R.box[c] = make_int4(x0, y0, x1, y1);
        }
    }
}

// Edge (c, d)'s parity term in the membership of point a + sh*delta in a
// ring (half-open crossing rule with the perturbation): sh = -1 tests
// a - delta (a vertex of P against Q + delta), sh = +1 tests a + delta (a
// vertex of Q + delta against P).  A straddling edge is never horizontal.
__device__ __forceinline__ bool flips_parity(int2 c, int2 d, int2 a, int sh)
{
    const bool st = sh < 0 ? ((c.y >= a.y) != (d.y >= a.y)) : ((c.y > a.y) != (d.y > a.y));
    const int up = d.y > c.y ? 1 : -1;
    const int tb = sh < 0 ? up : -up;   // sign of orient(c, d, a + sh*delta) when orient(c, d, a) = 0
    const double o = orient_d(c, d, a);
    const int so = o > 0 ? 1 : (o < 0 ? -1 : tb);
    return st & (so == up);
}

// The same for edge e of a ring in LDS.
__device__ __forceinline__ bool member_edge(const int2 *v, int e, int2 a, int sh)
{
    return flips_parity(v[e], v[e + 1], a, sh);
}

// Indices of a leftmost, a rightmost, a lowest and a highest vertex of Q
// (rb: Q's MBR relative to the origin), by one wavefront.  A pair whose P
// MBR leaves one of those sides of Q's MBR open anchors Q's memberships at
// that vertex (it lies outside P).
__device__ void q_extremes(RingLds Q, int m, int4 rb, int lane, int *ext)
{
    int k0 = -1, k1 = -1, k2 = -1, k3 = -1;
    for (int base = 0; base < m; base += 64) {
        const int i = base + lane;
        const bool live = i < m;
        const int2 p = Q.v[live ? i : 0];
        const uint64_t b0 = __ballot(live & (p.x == rb.x)), b1 = __ballot(live & (p.x == rb.z));
        const uint64_t b2 = __ballot(live & (p.y == rb.y)), b3 = __ballot(live & (p.y == rb.w));
        if (k0 < 0 && b0 != 0) k0 = base + __builtin_ctzll(b0);
        if (k1 < 0 && b1 != 0) k1 = base + __builtin_ctzll(b1);
        if (k2 < 0 && b2 != 0) k2 = base + __builtin_ctzll(b2);
        if (k3 < 0 && b3 != 0) k3 = base + __builtin_ctzll(b3);
    }
    if (lane == 0) { ext[0] = k0; ext[1] = k1; ext[2] = k2; ext[3] = k3; }
}

// Q's suffix sums Suf(f) = A2Q - sum_{f' <= f} cr_f' (exact in 64-bit
// integers), by one wavefront.  They spare a pass per pair: exchanging the
// order of summation,
//   sum_f cr_f * (w0 + s' * sum_{f' < f} S_f') = w0 * A2Q + s' * sum_{f'} S_f' * Suf(f'),
// every crossing on Q's edge f' adds its sign times Suf(f').
__device__ int64_t q_suffix_sums(RingLds Q, int m, int64_t a2q, int lane, int64_t *suf, int64_t carry = 0)
{
    for (int base = 0; base < m; base += 64) {
        const int e = base + lane;
        const bool live = e < m;
        const int ee = live ? e : 0;
        const int2 a = Q.v[ee], b = Q.v[ee + 1];
        const int64_t cr = live ? (int64_t)a.x * b.y - (int64_t)b.x * a.y : 0;
        const int64_t incl = carry + wave_incl_scan64(cr);
        if (live) suf[e] = a2q - incl;
        carry = (int64_t)dpp::readlane64((uint64_t)incl, 63);
    }
    return carry;
}

// Masks of several comparisons are combined as scalars: combined as lane
// values they cost the vector unit two to twelve instructions more.
__device__ __forceinline__ bool lane_in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// The lanes whose value is of the class set (a ballot of the builtin's result
// turns the mask into numbers and compares those again).
__device__ __forceinline__ uint64_t class_mask(double v, int mask)
{
    uint64_t lanes;
    asm("v_cmp_class_f64 %0, %1, %2" : "=s"(lanes) : "v"(v), "v"(mask));
    return lanes;
}

// One sweep unit per lane: Q edge f held in registers against the 8 edges of
// P chunk cp (entry = cp << USHIFT | f).  Returns the lane's crossings, edge
// i of the chunk as bit 7 - i: the steps have no branches, and the few
// crossings are appended to the buffer after them.
template <int USHIFT, int CSTEP>
__device__ __forceinline__ uint32_t sweep_units(RingLds P, RingLds Q, int entry)
{
    const int cp = entry >> USHIFT, f = entry & ((1 << USHIFT) - 1);
    const int2 c = Q.v[f], d = Q.v[f + 1];
    const double fx = (double)(d.x - c.x), fy = (double)(d.y - c.y);
    const int mf = q_edge_class(d.x - c.x, d.y - c.y);
    int2 pv[9];
#pragma unroll
    for (int i = 0; i < 9; i++) pv[i] = P.v[CSTEP * cp + i];
    double rx = (double)(c.x - pv[0].x), ry = (double)(c.y - pv[0].y);
    // orient(c, d, a) of the chunk's first vertex; each edge's end value is
    // the next edge's start value
    double oa = __fma_rn(fy, rx, -(fx * ry));
    uint64_t p3 = class_mask(oa, mf);
    int64_t ka = down_right_key(pv[0].x, pv[0].y);
    uint32_t hits = 0;
#pragma unroll
    for (int i = 0; i < 8; i++) {
        // with r = c - a and r' = c - b: e = r - r', so orient(a, b, c) =
        // cross(r, r'), orient(c, d, b) = cross(r', f) and X = their change
        // from a to b (all exact integers below 2^53)
        const int2 b = pv[i + 1];
        const double sx = (double)(c.x - b.x), sy = (double)(c.y - b.y);
        const int64_t kb = down_right_key(b.x, b.y);
        const double thr = kb < ka ? -0.5 : 0.5;
        const double oc = __fma_rn(rx, sy, -(ry * sx));
        const double ob = __fma_rn(fy, sx, -(fx * sy));
        const double od = oc + (oa - ob);
        const uint64_t p1 = __ballot(oc > thr), p2 = __ballot(od > thr), p4 = class_mask(ob, mf);
        const uint64_t cross = (p1 ^ p2) & (p3 ^ p4);
        // hits = 2 hits + cross
        asm("v_addc_co_u32 %0, vcc, %0, %0, %1" : "+v"(hits) : "s"(cross) : "vcc");
        rx = sx; ry = sy; ka = kb;
        oa = ob;
        p3 = p4;
    }
    return hits;
}

// Expand up to 16 listed tiles (lane = tile slot x Q edge j, two slots per
// lane) into sweep units, keeping the (P chunk, Q edge) pairs whose boxes
// touch: a crossing needs the Q edge's box to meet the box of the P edge it
// crosses, inside the chunk's.
template <typename UnitT, int USHIFT, bool CID>
__device__ __forceinline__ void expand_tiles(RingLds P, RingLds Q, int m, const uint8_t *cid, const uint16_t *tiles,
                                             int head, int count, int lane, UnitT *units, int &utail)
{
    uint64_t keep[2];
    int entry[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        // branch-free (see the batch loop); slots past `count` read entry 0
        const int slot = (lane >> 3) + 8 * h;
        const bool live = slot < count;
        const int t = (int)tiles[(head + (live ? slot : 0)) & (kListCap - 1)];
        const int cp = t >> 8, cq = t & 0xff;
        const int f = 8 * cq + (lane & 7);
        const int2 c = Q.v[f], d = Q.v[f + 1];
        const int4 bp = P.box[cp];
        keep[h] = __ballot(live) & __ballot(f < m) & __ballot(max(c.x, d.x) >= bp.x) & __ballot(bp.z >= min(c.x, d.x)) &
                  __ballot(max(c.y, d.y) >= bp.y) & __ballot(bp.w >= min(c.y, d.y));
        if constexpr (CID) entry[h] = ((int)cid[cp] << USHIFT) | f;
        else entry[h] = (cp << USHIFT) | f;
    }
    const int c0 = __popcll(keep[0]);
    const int r0 = lanes_below(keep[0]), r1 = lanes_below(keep[1]);
    if (lane_in(keep[0])) units[(utail + r0) & (kUnitCap - 1)] = (UnitT)entry[0];
    if (lane_in(keep[1])) units[(utail + c0 + r1) & (kUnitCap - 1)] = (UnitT)entry[1];
    utail = __builtin_amdgcn_readfirstlane(utail + c0 + __popcll(keep[1]));
}

// The crossings of the edges of ncp chunks of P with the m edges of Q staged
// in LDS (a whole ring, or a window of a longer one), handed to `flush` 64
// and more at a time.  Sweep units are (P chunk, Q edge) entries packed as
// cp << USHIFT | f in UnitT (16 bits up to 512 edges a side, 32 beyond).  P's
// chunks hold CSTEP vertices each; with CID, box c is that of chunk cid[c].
template <typename UnitT, int USHIFT, int CSTEP, bool CID, int XCAP, typename Flush>
__device__ __forceinline__ void tiled_accumulate(RingLds P, int ncp, RingLds Q, int m, int lane, const uint8_t *cid,
                                                 uint16_t *list, UnitT *units, uint32_t *xbuf,
                                                 unsigned long long *swept, Flush flush)
{
    const int ncq = (m + 7) >> 3;
    const int total = ncp * ncq;
    // chunk pair idx = (idx / ncq, idx % ncq), a lane's next one 128 on: the
    // float quotient of idx + 1/2 is at least 1/(2 ncq) >= 1/256 away from an
    // integer (ncq <= 128) while its rounding error is below 2^-15
    const float rq = 1.0f / (float)ncq;
    const int dp = (int)(128.5f * rq), dq = 128 - dp * ncq;
    int cp[2], cq[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        cp[h] = (int)(((float)(64 * h + lane) + 0.5f) * rq);
        cq[h] = 64 * h + lane - cp[h] * ncq;
    }
    int head = 0, tail = 0, uhead = 0, utail = 0, xcount = 0;
    // two batches of 64 chunk pairs per round trip through the tile list
    for (int base = 0; base < total; base += 128) {
        uint64_t ov[2];
        int en[2];
        // branch-free: whole boxes loaded at once (no short-circuit chains of
        // dependent LDS reads); pairs past the end read pair 0's
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const bool live = cp[h] < ncp;
            const int4 bp = P.box[live ? cp[h] : 0], bq = Q.box[cq[h]];
            ov[h] = __ballot(live) & __ballot(bp.z >= bq.x) & __ballot(bq.z >= bp.x) & __ballot(bp.w >= bq.y) &
                    __ballot(bq.w >= bp.y);
            en[h] = (cp[h] << 8) | cq[h];
            cp[h] += dp;
            cq[h] += dq;
            if (cq[h] >= ncq) { cq[h] -= ncq; cp[h]++; }
        }
        const int c0 = __popcll(ov[0]);
        const int r0 = lanes_below(ov[0]), r1 = lanes_below(ov[1]);
        if (lane_in(ov[0])) list[(tail + r0) & (kListCap - 1)] = (uint16_t)en[0];
        if (lane_in(ov[1])) list[(tail + c0 + r1) & (kListCap - 1)] = (uint16_t)en[1];
        tail = __builtin_amdgcn_readfirstlane(tail + c0 + __popcll(ov[1]));
        const bool last = base + 128 >= total;
        while (tail - head >= 16 || (last && (tail > head || utail > uhead))) {
            wave_lds_sync();
            if (tail > head) {
                const int cnt = min(16, tail - head);
                expand_tiles<UnitT, USHIFT, CID>(P, Q, m, cid, list, head, cnt, lane, units, utail);
                head += cnt;
            }
            wave_lds_sync();
            const bool rest = last && tail == head;
            while (utail - uhead >= 64 || (rest && utail > uhead)) {
                // in a partial sweep idle lanes take a padding edge of Q (zero length)
                const int k = min(64, utail - uhead);
                const int entry = lane < k ? (int)units[(uhead + lane) & (kUnitCap - 1)] : 8 * ncq;
                uint32_t hits = sweep_units<USHIFT, CSTEP>(P, Q, entry);
                uhead += k;
                // (e << 16 | f) of the lanes' crossings, one a lane and turn
                for (uint64_t cm = __ballot(hits != 0); cm != 0; cm = __ballot(hits != 0)) {
                    if (xcount + __popcll(cm) > XCAP) {
                        wave_lds_sync();
                        flush(xcount);
                        wave_lds_sync();
                        xcount = 0;
                    }
                    if (hits != 0) {
                        const int lead = __builtin_clz(hits);    // 24 + i
                        xbuf[xcount + lanes_below(cm)] =
                            ((uint32_t)(8 * (entry >> USHIFT) + lead - 24) << 16) | (uint32_t)(entry & ((1 << USHIFT) - 1));
                        hits &= ~(0x80000000u >> lead);
                    }
                    xcount = __builtin_amdgcn_readfirstlane(xcount + __popcll(cm));
                }
            }
        }
    }
    if (xcount > 0) {
        wave_lds_sync();
        flush(xcount);
    }
    *swept += 8ull * (unsigned long long)utail;   // edge pairs tested (idle lanes excluded)
}

// A vertex of Q strictly outside P's MBR among Q's extreme vertices, or -1.
__device__ __forceinline__ int anchor_q(const int32_t *qb, const int32_t *pb, const int *ext)
{
    if (qb[0] < pb[0]) return ext[0];
    if (qb[2] > pb[2]) return ext[1];
    if (qb[1] < pb[1]) return ext[2];
    if (qb[3] > pb[3]) return ext[3];
    return -1;
}

// One workgroup per query: Q staged once, wavefronts take its candidates.
// Heavy pairs: a pair on the general form with n m >= kHeavyMin edge pairs
// would keep one wavefront busy for a long serial run (milliseconds for a few
// thousand edges a side), so it is deferred: the wavefront records it, and a
// second launch splits each side's edges into kHeavySlices strided slices,
// one wavefront each; the one that finishes a pair's last slice adds the
// partial sums in a fixed order (a launch of its own for that, and for the
// split pairs' sums, cost a small call 5 us each even with nothing deferred:
// 120 pairs 24 us, with eight launches 35).  Up to kHeavyCap pairs per call are deferred; the rest run in place.
constexpr int kHeavySlices = 64;
constexpr int kHeavyCap = 8192;
constexpr int64_t kHeavyMin = 1 << 17;

struct HeavyPair {
    int64_t c;            // candidate slot of the result
    int64_t pa, qa;       // first vertex of P (data) and of Q (query)
    int64_t ox, oy;       // local origin of the pair
    int64_t a2p, a2q;     // exact doubled areas
    int32_t n, m;
    int32_t qmbr[4], pm[4];
    int32_t wide;
    int32_t done;         // slices finished
};

constexpr int kStatSlots = 64;   // work counters spread over slots, folded at the end

// Wide tiled pairs: a pair with a polygon beyond kTileCap edges but none
// beyond kWideCap (and coordinate spans below 2^26) would take the general
// form, which tests all n m edge pairs; it is deferred instead, and a second
// launch runs the tiled form on it with one wavefront staging both rings.
// Up to kWideListCap pairs per call are deferred; the rest run in place.
constexpr int kWideCap = 1024;
constexpr int kWideRing = kWideCap + 16;   // ring vertices incl. padding
constexpr int kWideListCap = 1 << 20;

// A pair that spans more than two window pairs (of kWideCap edges a side) is
// split into units of one wavefront each: P windows of plen edges (128 for a
// staged polygon of kSplitFineP edges or more, else the shortest of 256, 512
// and kWideCap that keeps the units within kMultiUnits), each walking Q's
// windows, or, when Q has more than two windows, each (P window, Q window)
// alone.  wide_meta finds the pair's own quantities once (areas, anchors, the
// windows' carries) and every unit adds its crossings' terms to the pair's
// sum, in the fixed point of k_refine's groups: whole numbers, in any order.
// Up to kMultiCap such pairs per call (the rest take all their windows on one
// wavefront).
constexpr int kMultiCap = 4096;
constexpr int kMultiUnits = 512;
constexpr int kSplitFineP = 4096;

struct SplitShape {
    int plen;             // P window length of the units
    int qs;               // units per P window (Q windows, or 1)
    int units;            // 1: the pair is not split
};

// The split of a pair whose staged polygon (P's role) has np edges and the
// other nq; deterministic, so wide_meta and k_refine_wide recompute it.
__device__ __forceinline__ int split_plen(int np, int qs)
{
    return (np >= kSplitFineP && ((np + 127) >> 7) * qs <= kMultiUnits) ? 128
         : ((np + 255) >> 8) * qs <= kMultiUnits ? 256
         : ((np + 511) >> 9) * qs <= kMultiUnits ? 512
         : ((np + 1023) >> 10) * qs <= kMultiUnits ? 1024 : 0;
}

__device__ __forceinline__ SplitShape split_shape(int np, int nq)
{
    const int npw = (np + kWideCap - 1) / kWideCap, nqw = (nq + kWideCap - 1) / kWideCap;
    if (npw * nqw <= 2) return {kWideCap, 1, 1};
    int qs = nqw > 2 ? nqw : 1;
    int plen = split_plen(np, qs);
    if (plen == 0 && qs > 1) plen = split_plen(np, qs = 1);
    if (plen == 0) return {kWideCap, 1, 1};
    return {plen, qs, (np + plen - 1) / plen * qs};
}

struct WidePair {
    int64_t c;            // candidate slot of the result (-1: an unused entry)
    int64_t pa;           // first vertex of the data polygon
    int32_t n;            // its vertex count
    int32_t q;            // query index
    int16_t pw;           // P window of a split pair, or -1 for all windows
    int16_t qw;           // Q window of a pair split on both sides, or -1 for all
    int32_t slot;         // the split pair's slot, or -1
};

struct MultiPair {
    int64_t c;            // candidate slot (-1: the pair was not deferred)
    int64_t pa;
    int32_t n, q;
    int32_t units;        // counted down as they are done
    int32_t fs;           // bits of the fixed point
    unsigned long long sum;   // the units' terms (modulo 2^64)
    int32_t first;        // its first unit's place from the list's back
    // the pair's own quantities, written by wide_meta for its units (P and
    // Q in k_refine_wide's roles)
    int64_t a2p, a2q;     // exact doubled areas
    int32_t kp, kq;       // anchors (0 where a membership pass stands in; kp first holds the list entry)
    int32_t wkp, wkq;     // memberships of P's vertex 0 in Q, of Q's vertex 0 in P (0 when anchored)
};

struct MultiUnit {
    int64_t ppre, qpre;   // P's and Q's cross-product sums before the unit's windows (wide_meta)
};

struct HeavyWs {
    int32_t *count;       // [0] heavy pairs, [1] wide list entries recorded, [2] split pairs, [4] their
                          // units, from the list's back (each may exceed its cap: the excess runs
                          // in place or whole), [3] wide entries taken, [5] entries of up to
                          // kWideCap edges a side, [6] entries looked at for those, [7] pairs of a
                          // group moved there
    HeavyPair *pairs;     // [kHeavyCap]
    double *partial;      // [kHeavyCap][2][kHeavySlices]
    unsigned long long *stat_slots;   // [kStatSlots][4]
    WidePair *wide;       // [kWideListCap]
    MultiPair *multi;     // [kMultiCap]
    MultiUnit *units;     // [kMultiCap][kMultiUnits]
};

// Records the lane's pair for the launches after k_refine as one list entry,
// from the list's front; a pair that split_shape splits also gets a split slot
// and places for its units, counted from the list's back (wide_meta writes the
// units there and takes the entry back, or leaves the pair whole where they do
// not fit).  False when the list is full.  The lanes of a wavefront come here
// together, so that the counters, which all wavefronts share, take one addition
// each for them (one a pair set the time of a call with many: 300,000 pairs of
// 600 edges 6.6 ms, so 3.8).
__device__ bool defer_wide(const HeavyWs &hw, int64_t c, int64_t pa, int n, int m, int32_t q)
{
    const int slot = atomicAdd(hw.count + 1, 1);
    if (slot >= kWideListCap) return false;
    WidePair &w = hw.wide[slot];
    w.c = c; w.pa = pa; w.n = n; w.q = q; w.pw = -1; w.qw = -1; w.slot = -1;
    const bool swap = n > kWideCap && n > m;
    const SplitShape sh = split_shape(swap ? m : n, swap ? n : m);
    if (max(n, m) <= kWideCap) atomicAdd(hw.count + 5, 1);
    if (sh.units > 1) {
        const int ms = atomicAdd(hw.count + 2, 1);
        if (ms < kMultiCap) {
            MultiPair &mp = hw.multi[ms];
            mp.c = c; mp.pa = pa; mp.n = n; mp.q = q; mp.units = sh.units;
            mp.first = atomicAdd(hw.count + 4, sh.units);
            mp.kp = slot;
        }
    }
    return true;
}

// Are the pairs of up to kWideCap edges a side taken by workgroups (mid_pairs,
// before k_refine_wide), or by k_refine_wide with the larger ones?  Many of
// them beside larger pairs fill the time of those pairs' long units (4.5
// million pairs of workload 5's polygons 2.03 ms, first by workgroups 2.29;
// 900,000 pairs 0.75 and 0.80); a few are faster by workgroups, and so are any
// number without larger ones (20,000 pairs 99 us, one wavefront each 195;
// 400,000 pairs 882 and 922).
__device__ __forceinline__ bool mids_by_workgroup(const HeavyWs &hw)
{
    return hw.count[5] <= 512 || hw.count[5] == hw.count[1];
}

__device__ __forceinline__ double jaccard_of(double inter2, int64_t a2p, int64_t a2q)
{
    const double inter = 0.5 * inter2;
    const double ap = 0.5 * fabs((double)a2p), aq = 0.5 * fabs((double)a2q);
    const double u = ap + aq - inter;
    return u > 0 ? inter / u : 0.0;
}

// Groups of pairs.  A wavefront takes its candidates 64 at a time, a lane
// each, and packs consecutive tiled ones into groups of up to kGroup data
// polygons and 64 chunks: the pass over the vertices (a chunk a lane), the
// tile list, the sweep and the crossing buffer then serve the group together,
// where a pair of average size (78 by 76 edges, 58 sweep units) fills a third
// of each.  A chunk is staged with its 9 vertices (the shared ones twice), so
// polygons follow each other without padding and the sweep's strided reads
// fall on different banks.
//
// With T exchanged like Q's sum, sum_e cr_e * sum_{e' < e} S_e' =
// sum_{e'} S_e' Suf_P(e'), every term of 2 A(P n Q) but the anchors' is a sum
// over crossings, and the anchors' K are too: for a crossing of edges e and f
// with signs s4 (along P) and s2 (along Q), parameters t and t',
//   s4 (cr_e (1 - t) + Suf_P(e) - [e < kp] A2P) + s2 (cr_f (1 - t') + Suf_Q(f) - [f < kq] A2Q).
// Suf_P comes from the chunks' exclusive prefix of cross products and the
// cross products inside the crossing's chunk.  All but the parameters' terms
// are whole numbers; those are rounded to a fixed point of the pair (sums
// wrap, the result does not: 2 A(P n Q) is at most twice the box that the MBRs
// share, and 6 bits are spare), so a pair's sum is taken by 64-bit integer
// additions in any order and does not depend on the pairs beside it.  (By the
// query's own box, small polygons against a large query lost the bits that
// their areas need; whole numbers and fractions in sums of their own, two
// additions a crossing, took 7.43 ms for 6.5 million pairs instead of 7.27.)
//
// Bound by the vector units: 477 instructions a pair at 6.5 million pairs of
// 78 by 76 edges on average (a third of them the sweep's, 463 edge pairs and
// 24 crossings a pair), 7.2 ms with the units issuing 71% of the time, 12.4 ms
// a pair at a time (949 instructions).  Four wavefronts a SIMD by registers
// and LDS.  Not better: 16 pairs a group (LDS for three workgroups), a test
// of a chunk's box against the line of Q's edge (few units fall out).
constexpr int kGroup = 8;
constexpr int kGroupCross = 64;    // a crossing a lane

struct GroupLds {
    int2 *v;               // 9 vertices a chunk
    int64_t *pre;          // cross products before chunk c of the group
    uint8_t *pair_of;      // pair of chunk c
    int4 *con;             // per pair: first chunk, end chunk, P's anchor (edge of the group), Q's anchor
                           // and, from bit 16, the bits of the fixed point
    unsigned long long *acc;   // per pair: its sum, in fixed point
};

// The fixed point of a pair's sums, 2^-s with 2 <= s <= 52 (MBRs within 2^26).
__device__ __forceinline__ int fixed_point_bits(int4 pb, int4 qb)
{
    const double box2 = 2.0 * ((double)min(pb.z, qb.z) - max(pb.x, qb.x) + 1) *
                        ((double)min(pb.w, qb.w) - max(pb.y, qb.y) + 1);
    const int bits = (int)((__double_as_longlong(box2) >> 52) & 0x7ff) - 1022;   // box2 < 2^bits
    return max(1, min(52, 56 - bits));
}

// v << s, 0 < s < 64, in 32-bit shifts.  A 64-bit shift by an amount in the
// kernel's last register gave wrong values (s differed from the one read).
__device__ __forceinline__ uint64_t shift_left(uint64_t v, int s)
{
    const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32), l = lo << (s & 31);
    const uint32_t h = s & 32 ? l : __builtin_amdgcn_alignbit(hi, lo, (uint32_t)(32 - s));
    return ((uint64_t)h << 32) | (s & 32 ? 0u : l);
}

__device__ __forceinline__ double power_of_two(int s) { return __longlong_as_double((long long)(uint32_t)(1023 + s) << 52); }

// 2 A = sp sq sum + sp w(kp) A2P + sq w(kq) A2Q, then J.
__device__ __forceinline__ double group_jaccard(uint64_t sum, int wkp, int wkq, int64_t a2p, int64_t a2q, int s)
{
    const int64_t ends = (wkp ? (a2p < 0 ? -a2p : a2p) : 0) + (wkq ? (a2q < 0 ? -a2q : a2q) : 0);
    const int64_t fixed = (int64_t)(((a2p ^ a2q) < 0 ? 0 - sum : sum) + shift_left((uint64_t)ends, s));
    return jaccard_of((double)fixed * power_of_two(-s), a2p, a2q);
}

// A crossing's term in fixed point: of edge i of the chunk of P at v (9
// vertices) and the edge (c, d) of Q.  past: P's cross products before the
// chunk, taken from those of the whole ring, or from 0 before P's anchor;
// sq: Q's suffix sum at the edge, less A2Q before Q's anchor.
__device__ __forceinline__ uint64_t crossing_term(const int2 *v, int i, int64_t past, int2 c, int2 d, int64_t sq, int s)
{
    const int2 a = v[i], b = v[i + 1];
    int2 u = v[0];
    int64_t before = 0;    // cross products of the chunk's edges up to e
#pragma unroll
    for (int j = 0; j < 8; j++) {
        const int2 w = v[j + 1];
        const int keep = j <= i ? -1 : 0;
        before += (int64_t)(u.x & keep) * w.y - (int64_t)(w.x & keep) * u.y;
        u = w;
    }
    const int64_t sp = past - before;
    const double ax = (double)a.x, ay = (double)a.y, bx = (double)b.x, by = (double)b.y;
    const double cx = (double)c.x, cy = (double)c.y;
    const double ex = bx - ax, ey = by - ay;
    const double fx = (double)(d.x - c.x), fy = (double)(d.y - c.y);
    const double rx = cx - ax, ry = cy - ay;
    const double oc = __fma_rn(ex, ry, -(ey * rx));
    const double oa = __fma_rn(fy, rx, -(fx * ry));
    const double X = __fma_rn(ex, fy, -(ey * fx));
    const double od = oc + X, ob = oa - X;
    const bool p2 = od > p_edge_threshold(ex, ey);
    const bool p4 = __builtin_amdgcn_class(ob, q_edge_class(d.x - c.x, d.y - c.y));
    const double cre = __fma_rn(ax, by, -(bx * ay));
    const double crf = __fma_rn(cx, fy, -(fx * cy));
    const double t = cre * (p4 ? 1.0 : -1.0) * (-ob) * rcp_refined(oa - ob) +
                     crf * (p2 ? 1.0 : -1.0) * (-od) * rcp_refined(oc - od);
    // |t| is below 2^54
    const double down = floor(t);
    const int64_t whole = (p4 ? sp : -sp) + (p2 ? sq : -sq) + (int64_t)down;
    // the fraction rounded: added to 2^52, it is the low bits of the sum
    const double frac = __fma_rn(t - down, power_of_two(s), 4503599627370496.0);
    return shift_left((uint64_t)whole, s) + ((uint64_t)__double_as_longlong(frac) - 0x4330000000000000ull);
}

__device__ void flush_group(const GroupLds &G, RingLds Q, const int64_t *suf, int64_t a2q, const uint32_t *buf,
                            int count, int lane)
{
    if (lane < count) {
        const uint32_t ef = buf[lane];
        const int e = (int)(ef >> 16), f = (int)(ef & 0xffffu);
        const int cc = e >> 3;
        const int g = G.pair_of[cc];
        const int4 con = G.con[g];
        const uint64_t t = crossing_term(G.v + 9 * cc, e & 7, G.pre[e < con.z ? con.x : con.y] - G.pre[cc], Q.v[f],
                                         Q.v[f + 1], suf[f] - (f < (con.w & 0xffff) ? a2q : 0), con.w >> 16);
        atomicAdd(&G.acc[g], (unsigned long long)t);
    }
}

// Ring-start memberships of a pair in one pass: w0p for P's vertex 0 against
// Q + delta, w0q for Q's vertex 0 + delta against P (chunks of 9 vertices).
__device__ void member_starts(const int2 *P, int n, const int2 *Q, int m, int lane, bool need_p, bool need_q, int &w0p,
                              int &w0q)
{
    const int2 p0 = P[0], q0 = Q[0];
    bool oddp = false, oddq = false;
    const int top = max(need_p ? m : 0, need_q ? n : 0);
    for (int e = lane; e < top; e += 64) {
        const bool lq = need_p & (e < m), lp = need_q & (e < n);
        oddp ^= lq & member_edge(Q, lq ? e : 0, p0, -1);
        oddq ^= lp & member_edge(P, lp ? e + (e >> 3) : 0, q0, +1);
    }
    w0p = __popcll(__ballot(oddp)) & 1;
    w0q = __popcll(__ballot(oddq)) & 1;
}

// In a small call the few largest pairs of a group, of kMidMin edge pairs and
// more, go to mid_pairs, a workgroup each: one wavefront each set the time of
// k_refine (20,000 pairs of workload 3 139 us, so 120; 257,000 of workload 2
// 840 and 735; from half the edge pairs on small calls lose up to 3 us, from a
// quarter on all lose).  A large call has others to run beside them, and loses:
// 6.5 million pairs 7.2 ms, with 2^16 edge pairs and more moved 8.3.  So does a
// call that is made of them, where they are no tail: 30,000 pairs of 500 by 500
// edges 141 us, with all of them moved 661.  So at most one candidate in
// kMidShare is moved (such pairs are one in 500 to 1,000 of the workloads'), and
// none of a wavefront whose candidates are all of them (139 us then).
constexpr int kMidMin = 1 << 17;
constexpr int64_t kMidCand = 1 << 18, kMidShare = 256;

__global__ __launch_bounds__(256, 4) void k_refine(const int32_t *__restrict__ dxy,
                                                const int64_t *__restrict__ doff,
                                                const int32_t *__restrict__ qxy,
                                                const int64_t *__restrict__ qoff,
                                                const int64_t *__restrict__ cand_off,
                                                const int32_t *__restrict__ cand_ids,
                                                double *__restrict__ cand_j,
                                                unsigned long long *__restrict__ stats,
                                                int slices, int mid_taken, HeavyWs hw)
{
    __shared__ int2 sQv[kRingLds];
    __shared__ int4 sQbox[kTileCap / 8];
    __shared__ int64_t sQsuf[kTileCap];
    __shared__ int2 sPv[kWavesPerBlock][64 * 9];
    __shared__ int4 sPbox[kWavesPerBlock][64];
    __shared__ int64_t sPre[kWavesPerBlock][64 + 1];
    __shared__ int4 sCon[kWavesPerBlock][kGroup];
    __shared__ unsigned long long sAcc[kWavesPerBlock][kGroup];
    __shared__ uint8_t sPairOf[kWavesPerBlock][64];
    __shared__ uint8_t sCid[kWavesPerBlock][64];
    __shared__ uint16_t sList[kWavesPerBlock][kListCap];
    __shared__ uint16_t sUnits[kWavesPerBlock][kUnitCap];
    // the crossing buffer; before the sweep, the pairs' MBRs and P's anchors
    __shared__ __align__(16) uint32_t sCross[kWavesPerBlock][kGroupCross];
    static_assert(kGroupCross >= 5 * kGroup, "MBRs and anchors fit the crossing buffer");
    __shared__ int32_t sQmbr[4];
    __shared__ long long sQa2;
    __shared__ int sQext[4];

    // `slices` workgroups share a query, and their wavefronts its candidates
    // in equal runs
    const int64_t q = blockIdx.x / slices;
    const int slice = (int)(blockIdx.x % slices);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t qa = qoff[q];
    const int m = (int)(qoff[q + 1] - qa);
    const int32_t *Qg = qxy + 2 * qa;
    const int64_t c0 = cand_off[q], c1 = cand_off[q + 1];
    if (c0 == c1) return;
    if (m < 3) {
        for (int64_t c = c0 + (int64_t)slice * blockDim.x + tid; c < c1; c += (int64_t)slices * blockDim.x)
            cand_j[c] = 0.0;
        return;
    }
    const int nwaves = (int)(blockDim.x >> 6) * slices;   // wavefronts on this query
    const int64_t w = (int64_t)slice * (blockDim.x >> 6) + wave;
    const int64_t cs = c0 + (c1 - c0) * w / nwaves, ce = c0 + (c1 - c0) * (w + 1) / nwaves;
    // the first candidates' vertex ranges are fetched behind Q's staging
    int64_t pa_next = 0, pe_next = 0;
    if (cs < ce) {
        const int32_t id = cand_ids[cs + lane < ce ? cs + lane : cs];
        pa_next = doff[id];
        pe_next = doff[id + 1];
    }
    const int64_t ox = Qg[0], oy = Qg[1];
    const bool q_tiled = m <= kTileCap;
    if (wave == 0) {
        int32_t qm[4];
        poly_mbr(Qg, m, lane, qm);
        const int64_t a2 = poly_area2(Qg, m, ox, oy, lane);
        if (lane == 0) {
            sQmbr[0] = qm[0]; sQmbr[1] = qm[1]; sQmbr[2] = qm[2]; sQmbr[3] = qm[3];
            sQa2 = a2;
        }
    }
    const RingLds Qs{sQv, sQbox, nullptr};
    if (q_tiled) {
        // Q padded by one extra chunk: the all-padding chunk ncq fills empty
        // slots of a partial tile group
        const int qpad = 8 * ((m + 7) >> 3) + 8;
        stage_ring(Qg, m, qpad + 1, ox, oy, Qs, tid, blockDim.x);
        __syncthreads();
        chunk_boxes(Qs, m, tid, blockDim.x);
        __syncthreads();
        if (wave == 0) {
            q_suffix_sums(Qs, m, sQa2, lane, sQsuf);
            const int4 rb = make_int4((int)((int64_t)sQmbr[0] - ox), (int)((int64_t)sQmbr[1] - oy),
                                      (int)((int64_t)sQmbr[2] - ox), (int)((int64_t)sQmbr[3] - oy));
            q_extremes(Qs, m, rb, lane, sQext);
        }
    }
    __syncthreads();
    int32_t qmbr[4], qext[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        qmbr[i] = __builtin_amdgcn_readfirstlane(sQmbr[i]);
        qext[i] = __builtin_amdgcn_readfirstlane(sQext[i]);
    }
    const int64_t a2q = sQa2;
    const GroupLds G{sPv[wave], sPre[wave], sPairOf[wave], sCon[wave], sAcc[wave]};
    const RingLds Ps{sPv[wave], sPbox[wave], nullptr};
    int32_t *const box_of = reinterpret_cast<int32_t *>(sCross[wave]), *const anchor_of = box_of + 4 * kGroup;
    unsigned long long st_tiled = 0, st_swept = 0, st_general = 0, st_disjoint = 0;
    for (int64_t cb = cs; cb < ce; cb += 64) {
        const int64_t c = cb + lane;
        const bool live = c < ce;
        const int64_t pa = pa_next;
        const int n = (int)(pe_next - pa_next);
        if (cb + 64 < ce) {
            const int32_t id = cand_ids[c + 64 < ce ? c + 64 : cb + 64];
            pa_next = doff[id];
            pe_next = doff[id + 1];
        }
        const bool valid = live & (n >= 3) & (a2q != 0);
        bool small = valid & q_tiled & (n <= kTileCap);
        // a small call's few largest go to the launch after this one
        if (mid_taken > 0) {
            const bool largest = small & (edge_pairs(n, m) >= kMidMin);
            const uint64_t lm = __ballot(largest);
            if ((__popcll(lm) < 3 || lm != __ballot(valid)) && largest &&
                __hip_atomic_load(hw.count + 7, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < mid_taken)
                small = atomicAdd(hw.count + 7, 1) >= mid_taken;
        }
        if (live & !valid) cand_j[c] = 0.0;
        uint64_t big = __ballot(valid & !small), todo = __ballot(small);
        const int nch = small ? (n + 7) >> 3 : 0;
        const int before = wave_incl_scan32(nch) - nch, rank = lanes_below(todo);
        while (todo) {
            // the group: lanes `gm`, pair g's chunks from first_chunk
            const int first = __builtin_ctzll(todo);
            const int first_chunk = before - __builtin_amdgcn_readlane(before, first);
            const int g = rank - __builtin_amdgcn_readlane(rank, first);
            const bool mem = small & (lane >= first) & (first_chunk + nch <= 64) & (g < kGroup);
            const uint64_t gm = __ballot(mem);
            todo &= ~gm;
            const int total = __builtin_amdgcn_readlane(first_chunk + nch, 63 - __builtin_clzll(gm));
            // lane = chunk from here on: its pair's lane, polygon and place
            int src = first;
            for (uint64_t mm = gm & (gm - 1); mm; mm &= mm - 1) {
                const int sl = __builtin_ctzll(mm);
                src = lane >= __builtin_amdgcn_readlane(first_chunk, sl) ? sl : src;
            }
            const int pn = __shfl(n, src), pg = __shfl(g, src), v0 = 8 * (lane - __shfl(first_chunk, src));
            const int2 *V = reinterpret_cast<const int2 *>(dxy) + __shfl(pa, src);
            int2 p[9];
#pragma unroll
            for (int j = 0; j < 9; j++) p[j] = V[v0 + j < pn ? v0 + j : 0];
            // the wavefront is done with the group before
            wave_lds_sync();
            if (lane < 4 * kGroup) box_of[lane] = (lane & 3) < 2 ? INT32_MAX : INT32_MIN;
            if (lane < kGroup) { anchor_of[lane] = -1; G.acc[lane] = 0; }
            wave_lds_sync();
            int4 box = make_int4(p[0].x, p[0].y, p[0].x, p[0].y);
            int out = -1;
            int64_t cross = 0;
            int2 r0 = make_int2((int)((uint32_t)p[0].x - (uint32_t)ox), (int)((uint32_t)p[0].y - (uint32_t)oy));
            G.v[9 * lane] = r0;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                // relative coordinates in 32 bits (wrapping): exact unless the
                // pair spans 2^26 or more, which is found from the MBRs
                const int2 r1 = make_int2((int)((uint32_t)p[j + 1].x - (uint32_t)ox),
                                          (int)((uint32_t)p[j + 1].y - (uint32_t)oy));
                G.v[9 * lane + j + 1] = r1;
                cross += (int64_t)r0.x * r1.y - (int64_t)r1.x * r0.y;
                r0 = r1;
                box.x = min(box.x, p[j + 1].x); box.z = max(box.z, p[j + 1].x);
                box.y = min(box.y, p[j + 1].y); box.w = max(box.w, p[j + 1].y);
                const bool o = ((uint32_t)p[j].x - (uint32_t)qmbr[0] > (uint32_t)qmbr[2] - (uint32_t)qmbr[0]) |
                               ((uint32_t)p[j].y - (uint32_t)qmbr[1] > (uint32_t)qmbr[3] - (uint32_t)qmbr[1]);
                out = o ? (v0 + j < pn ? v0 + j : 0) : out;
            }
            const int64_t upto = wave_incl_scan64(cross);
            G.pre[lane + 1] = upto;
            if (lane == 0) G.pre[0] = 0;
            G.pair_of[lane] = (uint8_t)pg;
            if (lane < total) {
                atomicMin(&box_of[4 * pg], box.x); atomicMin(&box_of[4 * pg + 1], box.y);
                atomicMax(&box_of[4 * pg + 2], box.z); atomicMax(&box_of[4 * pg + 3], box.w);
                // any vertex outside Q's MBR will do
                if (out >= 0) atomicMax(&anchor_of[pg], out);
            }
            wave_lds_sync();
            // lane = pair: what it is, and its anchors
            const int gi = mem ? g : 0, ca = mem ? first_chunk : 0, cz = mem ? first_chunk + nch : 0;
            const int4 pb = *reinterpret_cast<const int4 *>(box_of + 4 * gi);
            int kp = anchor_of[gi];
            const int64_t a2p = G.pre[cz] - G.pre[ca];
            const bool apart = (pb.z <= qmbr[0]) | (qmbr[2] <= pb.x) | (pb.w <= qmbr[1]) | (qmbr[3] <= pb.y);
            const bool wide = ((uint32_t)max(pb.z, qmbr[2]) - (uint32_t)min(pb.x, qmbr[0]) >= 1u << 26) |
                              ((uint32_t)max(pb.w, qmbr[3]) - (uint32_t)min(pb.y, qmbr[1]) >= 1u << 26);
            const uint64_t wm = __ballot(mem & !apart & wide);
            st_disjoint += (unsigned long long)__popcll(__ballot(mem & apart));
            st_tiled += (unsigned long long)__popcll(__ballot(mem & !apart & !wide));
            big |= wm;
            const bool act = mem & !apart & !wide & (a2p != 0);
            const uint64_t am = __ballot(act);
            int kq = qmbr[0] < pb.x ? qext[0] : qmbr[2] > pb.z ? qext[1] : qmbr[1] < pb.y ? qext[2]
                   : qmbr[3] > pb.w ? qext[3] : -1;
            int wkp = 0, wkq = 0;
            for (uint64_t mm = __ballot(act & ((kp < 0) | (kq < 0))); mm; mm &= mm - 1) {
                const int sl = __builtin_ctzll(mm);
                int w0p, w0q;
                member_starts(G.v + 9 * __builtin_amdgcn_readlane(first_chunk, sl), __builtin_amdgcn_readlane(n, sl), sQv,
                              m, lane, __builtin_amdgcn_readlane(kp, sl) < 0, __builtin_amdgcn_readlane(kq, sl) < 0,
                              w0p, w0q);
                wkp = lane == sl ? w0p : wkp;
                wkq = lane == sl ? w0q : wkq;
            }
            kp = max(kp, 0);
            kq = max(kq, 0);
            const int fs = fixed_point_bits(pb, make_int4(qmbr[0], qmbr[1], qmbr[2], qmbr[3]));
            if (mem) G.con[g] = make_int4(first_chunk, first_chunk + nch, 8 * first_chunk + kp, kq | fs << 16);
            // lane = chunk: those that meet Q's MBR are listed
            const bool keep = (lane < total) & (((am >> src) & 1) != 0) & !((box.z < qmbr[0]) | (qmbr[2] < box.x) |
                              (box.w < qmbr[1]) | (qmbr[3] < box.y));
            const uint64_t km = __ballot(keep);
            const int at = lanes_below(km);
            if (keep) {
                sPbox[wave][at] = make_int4((int)((uint32_t)box.x - (uint32_t)ox), (int)((uint32_t)box.y - (uint32_t)oy),
                                            (int)((uint32_t)box.z - (uint32_t)ox), (int)((uint32_t)box.w - (uint32_t)oy));
                sCid[wave][at] = (uint8_t)lane;
            }
            wave_lds_sync();
            tiled_accumulate<uint16_t, 10, 9, true, kGroupCross>(
                Ps, __popcll(km), Qs, m, lane, sCid[wave], sList[wave], sUnits[wave], sCross[wave], &st_swept,
                [&](int count) { flush_group(G, Qs, sQsuf, a2q, sCross[wave], count, lane); });
            wave_lds_sync();
            // lane = pair
            const double J = act ? group_jaccard(G.acc[gi], wkp, wkq, a2p, a2q, G.con[gi].w >> 16) : 0.0;
            if (mem & !(!apart & wide)) cand_j[c] = J;
        }
        // pairs beyond the tiled form: their MBRs, one at a time
        int4 box = make_int4(0, 0, 0, 0);
        for (uint64_t mm = big; mm; mm &= mm - 1) {
            const int sl = __builtin_ctzll(mm);
            int32_t pm[4];
            poly_mbr(dxy + 2 * (int64_t)dpp::readlane64((uint64_t)pa, sl), __builtin_amdgcn_readlane(n, sl), lane, pm);
            box = lane == sl ? make_int4(pm[0], pm[1], pm[2], pm[3]) : box;
        }
        const bool apart = (box.z <= qmbr[0]) | (qmbr[2] <= box.x) | (box.w <= qmbr[1]) | (qmbr[3] <= box.y);
        const bool wide = ((uint32_t)max(box.z, qmbr[2]) - (uint32_t)min(box.x, qmbr[0]) >= 1u << 26) |
                          ((uint32_t)max(box.w, qmbr[3]) - (uint32_t)min(box.y, qmbr[1]) >= 1u << 26);
        bool here = lane_in(big) & !apart;     // of those that fit a group only wide ones
        st_disjoint += (unsigned long long)__popcll(__ballot(lane_in(big) & apart));
        if (lane_in(big) & apart) cand_j[c] = 0.0;
        // tiled form on the wavefronts of the next launches
        if (hw.count && here && !wide && !small) here = !defer_wide(hw, c, pa, n, m, (int32_t)q);
        for (uint64_t mm = __ballot(here); mm; mm &= mm - 1) {
            const int sl = __builtin_ctzll(mm);
            const int64_t cl = cb + sl;
            const int64_t pal = (int64_t)dpp::readlane64((uint64_t)pa, sl);
            const int nl = __builtin_amdgcn_readlane(n, sl);
            const int32_t *Pg = dxy + 2 * pal;
            const int32_t pm[4] = {__builtin_amdgcn_readlane(box.x, sl), __builtin_amdgcn_readlane(box.y, sl),
                                   __builtin_amdgcn_readlane(box.z, sl), __builtin_amdgcn_readlane(box.w, sl)};
            const bool wide_pair = __builtin_amdgcn_readlane((int)wide, sl) != 0;
            double J = 0.0;
            bool deferred = false;
            int slot = 0;
            double inter2 = 0.0;
            int64_t a2p = 0;
            st_general += 2ull * (unsigned long long)nl * (unsigned long long)m;
            if (hw.count && edge_pairs(nl, m) >= kHeavyMin && (a2p = poly_area2(Pg, nl, ox, oy, lane)) != 0 &&
                (slot = __builtin_amdgcn_readfirstlane(lane == 0 ? atomicAdd(hw.count, 1) : 0)) < kHeavyCap) {
                // split over many wavefronts by the next launches
                if (lane == 0) {
                    HeavyPair &h = hw.pairs[slot];
                    h.c = cl; h.pa = pal; h.qa = qa; h.ox = ox; h.oy = oy; h.a2p = a2p; h.a2q = a2q;
                    h.n = nl; h.m = m; h.wide = wide_pair; h.done = 0;
                    for (int i = 0; i < 4; i++) { h.qmbr[i] = qmbr[i]; h.pm[i] = pm[i]; }
                }
                deferred = true;
            } else {
                PairIn in;
                in.P = Pg; in.n = nl; in.Q = Qg; in.m = m; in.ox = ox; in.oy = oy;
                in.qmbr[0] = qmbr[0]; in.qmbr[1] = qmbr[1]; in.qmbr[2] = qmbr[2]; in.qmbr[3] = qmbr[3];
                in.sq = a2q > 0 ? 1 : -1;
                double sa, sb;
                if (!wide_pair) edges_in_other_P<false>(in, lane, sa, a2p);
                else edges_in_other_P<true>(in, lane, sa, a2p);
                a2p = wave_sum_i64(a2p);
                in.sp = a2p > 0 ? 1 : -1;
                if (a2p != 0) {
                    int64_t unused;
                    if (!wide_pair) edges_in_other_Q<false>(in, pm, lane, sb, unused);
                    else edges_in_other_Q<true>(in, pm, lane, sb, unused);
                    inter2 = wave_sum(in.sp * sa) + wave_sum(in.sq * sb);
                }
            }
            if (a2p != 0) J = jaccard_of(inter2, a2p, a2q);
            if (lane == 0 && !deferred) cand_j[cl] = J;
        }
    }
    if (stats) {
        // one sum per workgroup, added to one of kStatSlots slots when the
        // workspace has them (atomics of every wavefront on four words
        // serialise at the cache), nonzero counts only
        if (lane == 0) {
            sAcc[wave][0] = st_tiled; sAcc[wave][1] = st_swept;
            sAcc[wave][2] = st_general; sAcc[wave][3] = st_disjoint;
        }
        __syncthreads();
        if (tid < 4) {
            unsigned long long v = 0;
            for (int w = 0; w < (int)(blockDim.x >> 6); w++) v += sAcc[w][tid];
            if (v) {
                if (hw.stat_slots) atomicAdd(hw.stat_slots + (blockIdx.x % kStatSlots) * 4 + tid, v);
                else atomicAdd(stats + tid, v);
            }
        }
    }
}

// Vertex i of an m-vertex ring in global memory, relative to the origin.
__device__ __forceinline__ int2 ring_vertex(const int32_t *V, int m, int i, int64_t ox, int64_t oy)
{
    const int k = i < m ? i : i - m;
    return make_int2((int)((int64_t)V[2 * k] - ox), (int)((int64_t)V[2 * k + 1] - oy));
}

// The passes below read a ring in global memory with one wavefront and
// kPassU vertices a lane in flight: a long ring costs a few round trips to
// memory rather than one per 64 vertices.
constexpr int kPassU = 8;

// One pass: the ring's MBR (absolute coordinates) and twice its signed area
// about the origin (as poly_area2, exact in 64-bit integers).
__device__ void ring_sums_global(const int32_t *V, int m, int64_t ox, int64_t oy, int lane,
                                 int32_t *mbr, int64_t &a2)
{
    const int2 *W = reinterpret_cast<const int2 *>(V);
    int32_t mnx = INT32_MAX, mny = INT32_MAX, mxx = INT32_MIN, mxy = INT32_MIN;
    int64_t a = 0;
    for (int base = 0; base < m; base += 64 * kPassU) {
        int2 v[kPassU], w[kPassU];
#pragma unroll
        for (int k = 0; k < kPassU; k++) {
            const int i = min(base + 64 * k + lane, m - 1);
            v[k] = W[i];
            w[k] = W[i + 1 == m ? 0 : i + 1];
        }
#pragma unroll
        for (int k = 0; k < kPassU; k++) {
            const int i = base + 64 * k + lane;
            if (i < m) {
                mnx = min(mnx, v[k].x); mxx = max(mxx, v[k].x);
                mny = min(mny, v[k].y); mxy = max(mxy, v[k].y);
                const int64_t ax = (int64_t)v[k].x - ox, ay = (int64_t)v[k].y - oy;
                const int64_t bx = (int64_t)w[k].x - ox, by = (int64_t)w[k].y - oy;
                a += (int64_t)((__int128)ax * by - (__int128)bx * ay);
            }
        }
    }
    mbr[0] = wmin(mnx); mbr[1] = wmin(mny); mbr[2] = wmax(mxx); mbr[3] = wmax(mxy);
    a2 = wave_sum_i64(a);
}

// Membership of point a + sh*delta (relative coordinates) in a ring read from
// global memory: the half-open crossing rule of member_edge over every edge.
__device__ int member_point_global(const int32_t *V, int m, int64_t ox, int64_t oy, int2 a, int sh, int lane)
{
    bool odd = false;
    for (int base = 0; base < m; base += 64 * kPassU) {
        int2 cv[kPassU], dv[kPassU];
#pragma unroll
        for (int k = 0; k < kPassU; k++) {
            const int e = min(base + 64 * k + lane, m - 1);
            cv[k] = ring_vertex(V, m, e, ox, oy);
            dv[k] = ring_vertex(V, m, e + 1, ox, oy);
        }
#pragma unroll
        for (int k = 0; k < kPassU; k++) odd ^= (base + 64 * k + lane < m) & flips_parity(cv[k], dv[k], a, sh);
    }
    return __popcll(__ballot(odd)) & 1;
}

// Indices of a leftmost, a rightmost, a lowest and a highest vertex of a ring
// in global memory (mbr: its absolute MBR), as q_extremes.
__device__ void extremes_global(const int32_t *V, int m, const int32_t *mbr, int lane, int *ext)
{
    const int2 *W = reinterpret_cast<const int2 *>(V);
    int k0 = -1, k1 = -1, k2 = -1, k3 = -1;
    for (int base = 0; base < m; base += 64 * kPassU) {
        int2 v[kPassU];
#pragma unroll
        for (int k = 0; k < kPassU; k++) v[k] = W[min(base + 64 * k + lane, m - 1)];
#pragma unroll
        for (int k = 0; k < kPassU; k++) {
            const int b = base + 64 * k;
            const bool live = b + lane < m;
            const uint64_t b0 = __ballot(live & (v[k].x == mbr[0])), b1 = __ballot(live & (v[k].x == mbr[2]));
            const uint64_t b2 = __ballot(live & (v[k].y == mbr[1])), b3 = __ballot(live & (v[k].y == mbr[3]));
            if (k0 < 0 && b0 != 0) k0 = b + __builtin_ctzll(b0);
            if (k1 < 0 && b1 != 0) k1 = b + __builtin_ctzll(b1);
            if (k2 < 0 && b2 != 0) k2 = b + __builtin_ctzll(b2);
            if (k3 < 0 && b3 != 0) k3 = b + __builtin_ctzll(b3);
        }
    }
    ext[0] = k0; ext[1] = k1; ext[2] = k2; ext[3] = k3;
}

// Edges [w0, w0 + len) of an m-vertex ring staged as a chain: entry i holds
// vertex w0 + i for i <= len (vertex m is vertex 0), entries beyond len repeat
// vertex w0 + len, so edges from len on have zero length and never cross.
__device__ void stage_window(const int32_t *V, int m, int w0, int len, int pad_to, int64_t ox, int64_t oy,
                             RingLds R, int lane)
{
    for (int base = 0; base < pad_to; base += 64 * kPassU) {
        int2 v[kPassU];
#pragma unroll
        for (int k = 0; k < kPassU; k++) v[k] = ring_vertex(V, m, w0 + min(base + 64 * k + lane, len), ox, oy);
#pragma unroll
        for (int k = 0; k < kPassU; k++)
            if (base + 64 * k + lane < pad_to) R.v[base + 64 * k + lane] = v[k];
    }
}

// First vertex of a ring in global memory strictly outside the box b, or -1.
__device__ int first_outside_global(const int32_t *V, int n, const int32_t *b, int lane)
{
    const int2 *W = reinterpret_cast<const int2 *>(V);
    for (int base = 0; base < n; base += 64 * kPassU) {
        int2 v[kPassU];
#pragma unroll
        for (int k = 0; k < kPassU; k++) v[k] = W[min(base + 64 * k + lane, n - 1)];
#pragma unroll
        for (int k = 0; k < kPassU; k++) {
            const int x = v[k].x, y = v[k].y;
            const bool live = base + 64 * k + lane < n;
            const uint64_t mk = __ballot(live & ((x < b[0]) | (x > b[2]) | (y < b[1]) | (y > b[3])));
            if (mk != 0) return base + 64 * k + __builtin_ctzll(mk);
        }
    }
    return -1;
}

// The quantities of a split pair that all its units share, found once per
// pair by one workgroup (a unit used to find them itself, in four passes over
// both whole rings read from memory): both rings' MBRs and exact doubled
// areas, the anchors (P's first vertex strictly outside Q's MBR, Q's extreme
// vertex outside P's MBR), the memberships of the ring starts where there is
// no anchor, and the rings' cross-product sums before each window, written
// into the units' slots.  All are exact integers.  Rings of up to
// kMetaThreads x kMetaU vertices take one round trip to memory a pass.  The
// workgroup also writes the pair's unit entries at their places in the list.
constexpr int kMetaThreads = 1024;
constexpr int kMetaU = 8;

struct MetaLds {
    unsigned long long qwin[kMultiUnits];   // Q's cross products per window of kWideCap edges
    unsigned long long pwin[kMultiUnits];   // P's, per window of a unit
    unsigned long long a[2];                // doubled areas of Q and P
    int32_t box[8];                         // MBRs of Q and P: min x, min y, max x, max y
    int32_t idx[5];                         // Q's extreme vertices, P's first vertex outside
    int32_t odd[2];                         // crossings of the two membership passes
};

__device__ void wide_meta(MetaLds &L, const int32_t *__restrict__ dxy, const int32_t *__restrict__ qxy,
                          const int64_t *__restrict__ qoff, const HeavyWs &hw, int block, int blocks)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t count = min((int64_t)hw.count[2], (int64_t)kMultiCap);
    const int64_t room = kWideListCap - min((int64_t)hw.count[1], (int64_t)kWideListCap);
    for (int64_t s = block; s < count; s += blocks) {
        const MultiPair mp = hw.multi[s];
        if (mp.first + mp.units > room) {
            // its units do not fit the list: the pair stays whole, the places
            // that it claimed are unused
            for (int64_t j = mp.first + tid; j < room && j < mp.first + mp.units; j += kMetaThreads)
                hw.wide[kWideListCap - 1 - j].c = -1;
            continue;
        }
        // the roles of k_refine_wide
        const int64_t qa = qoff[mp.q];
        const int mq = (int)(qoff[mp.q + 1] - qa);
        const bool swap = mp.n > kWideCap && mp.n > mq;
        const int2 *PW = reinterpret_cast<const int2 *>(swap ? qxy + 2 * qa : dxy + 2 * mp.pa);
        const int2 *QW = reinterpret_cast<const int2 *>(swap ? dxy + 2 * mp.pa : qxy + 2 * qa);
        const int n = swap ? mq : mp.n, m = swap ? mp.n : mq;
        const int2 o = QW[0];
        const SplitShape sh = split_shape(n, m);
        const int len = max(n, m);
        for (int i = tid; i < kMultiUnits; i += kMetaThreads) L.qwin[i] = L.pwin[i] = 0;
        if (tid < 2) { L.a[tid] = 0; L.odd[tid] = 0; }
        if (tid < 8) L.box[tid] = (tid & 3) < 2 ? INT32_MAX : INT32_MIN;
        if (tid < 5) L.idx[tid] = INT32_MAX;
        __syncthreads();
        // MBRs, areas and the windows' sums (a wavefront's 64 edges lie in one window)
        {
            int32_t b[8] = {INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN, INT32_MAX, INT32_MAX, INT32_MIN, INT32_MIN};
            int64_t aq = 0, ap = 0;
            for (int base = 0; base < len; base += kMetaThreads * kMetaU) {
                int2 qv[kMetaU], qw[kMetaU], pv[kMetaU], pw[kMetaU];
#pragma unroll
                for (int k = 0; k < kMetaU; k++) {
                    const int i = base + k * kMetaThreads + tid;
                    const int iq = min(i, m - 1), ip = min(i, n - 1);
                    qv[k] = QW[iq]; qw[k] = QW[iq + 1 == m ? 0 : iq + 1];
                    pv[k] = PW[ip]; pw[k] = PW[ip + 1 == n ? 0 : ip + 1];
                }
#pragma unroll
                for (int k = 0; k < kMetaU; k++) {
                    const int i = base + k * kMetaThreads + tid;
                    int64_t cq = 0, cp = 0;
                    if (i < m) {
                        b[0] = min(b[0], qv[k].x); b[1] = min(b[1], qv[k].y);
                        b[2] = max(b[2], qv[k].x); b[3] = max(b[3], qv[k].y);
                        cq = (int64_t)(qv[k].x - o.x) * (qw[k].y - o.y) - (int64_t)(qw[k].x - o.x) * (qv[k].y - o.y);
                    }
                    if (i < n) {
                        b[4] = min(b[4], pv[k].x); b[5] = min(b[5], pv[k].y);
                        b[6] = max(b[6], pv[k].x); b[7] = max(b[7], pv[k].y);
                        cp = (int64_t)(pv[k].x - o.x) * (pw[k].y - o.y) - (int64_t)(pw[k].x - o.x) * (pv[k].y - o.y);
                    }
                    aq += cq;
                    ap += cp;
                    const int w0 = base + k * kMetaThreads + (tid & ~63);   // the wavefront's first edge
                    if (sh.qs > 1 && w0 < m) {
                        const int64_t ws = wave_sum_i64(cq);
                        if (lane == 0) atomicAdd(&L.qwin[w0 / kWideCap], (unsigned long long)ws);
                    }
                    if (w0 < n) {
                        const int64_t ws = wave_sum_i64(cp);
                        if (lane == 0) atomicAdd(&L.pwin[w0 / sh.plen], (unsigned long long)ws);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 8; j++) b[j] = (j & 3) < 2 ? wmin(b[j]) : wmax(b[j]);
            aq = wave_sum_i64(aq);
            ap = wave_sum_i64(ap);
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    if ((j & 3) < 2) atomicMin(&L.box[j], b[j]);
                    else atomicMax(&L.box[j], b[j]);
                }
                atomicAdd(&L.a[0], (unsigned long long)aq);
                atomicAdd(&L.a[1], (unsigned long long)ap);
            }
        }
        __syncthreads();
        const int32_t qm[4] = {L.box[0], L.box[1], L.box[2], L.box[3]}, pm[4] = {L.box[4], L.box[5], L.box[6], L.box[7]};
        const int64_t a2q = (int64_t)L.a[0], a2p = (int64_t)L.a[1];
        int kp = 0, kq = 0, wkp = 0, wkq = 0;
        if (a2p != 0 && a2q != 0) {
            // Q's extreme vertices (the first of each side) and P's first
            // vertex strictly outside Q's MBR
            int32_t e[5] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
            for (int base = 0; base < len; base += kMetaThreads * kMetaU) {
                int2 qv[kMetaU], pv[kMetaU];
#pragma unroll
                for (int k = 0; k < kMetaU; k++) {
                    const int i = base + k * kMetaThreads + tid;
                    qv[k] = QW[min(i, m - 1)];
                    pv[k] = PW[min(i, n - 1)];
                }
#pragma unroll
                for (int k = 0; k < kMetaU; k++) {
                    const int i = base + k * kMetaThreads + tid;
                    if (i < m) {
                        if (qv[k].x == qm[0]) e[0] = min(e[0], i);
                        if (qv[k].x == qm[2]) e[1] = min(e[1], i);
                        if (qv[k].y == qm[1]) e[2] = min(e[2], i);
                        if (qv[k].y == qm[3]) e[3] = min(e[3], i);
                    }
                    const bool out = (pv[k].x < qm[0]) | (pv[k].x > qm[2]) | (pv[k].y < qm[1]) | (pv[k].y > qm[3]);
                    if (i < n && out) e[4] = min(e[4], i);
                }
            }
#pragma unroll
            for (int j = 0; j < 5; j++) e[j] = wmin(e[j]);
            if (lane == 0) {
#pragma unroll
                for (int j = 0; j < 5; j++) atomicMin(&L.idx[j], e[j]);
            }
            __syncthreads();
            const int ext[4] = {L.idx[0], L.idx[1], L.idx[2], L.idx[3]};
            kq = anchor_q(qm, pm, ext);
            kp = L.idx[4] == INT32_MAX ? -1 : L.idx[4];
            if (kp < 0 || kq < 0) {
                // without an anchor: P's vertex 0 (against Q + delta) and Q's
                // vertex 0, the origin (plus delta, against P), by the
                // crossing rule over the other ring's edges
                const int2 p0 = make_int2(PW[0].x - o.x, PW[0].y - o.y), q0 = make_int2(0, 0);
                bool op = false, oq = false;
                for (int base = 0; base < len; base += kMetaThreads * kMetaU) {
                    int2 qv[kMetaU], qw[kMetaU], pv[kMetaU], pw[kMetaU];
#pragma unroll
                    for (int k = 0; k < kMetaU; k++) {
                        const int i = base + k * kMetaThreads + tid;
                        const int iq = min(i, m - 1), ip = min(i, n - 1);
                        qv[k] = QW[iq]; qw[k] = QW[iq + 1 == m ? 0 : iq + 1];
                        pv[k] = PW[ip]; pw[k] = PW[ip + 1 == n ? 0 : ip + 1];
                    }
#pragma unroll
                    for (int k = 0; k < kMetaU; k++) {
                        const int i = base + k * kMetaThreads + tid;
                        const int2 c = make_int2(qv[k].x - o.x, qv[k].y - o.y), d = make_int2(qw[k].x - o.x, qw[k].y - o.y);
                        const int2 f = make_int2(pv[k].x - o.x, pv[k].y - o.y), g = make_int2(pw[k].x - o.x, pw[k].y - o.y);
                        op ^= kp < 0 && i < m && flips_parity(c, d, p0, -1);
                        oq ^= kq < 0 && i < n && flips_parity(f, g, q0, +1);
                    }
                }
                const int cp = __popcll(__ballot(op)), cq = __popcll(__ballot(oq));
                if (lane == 0) { atomicAdd(&L.odd[0], cp); atomicAdd(&L.odd[1], cq); }
                __syncthreads();
                if (kp < 0) { wkp = L.odd[0] & 1; kp = 0; }
                if (kq < 0) { wkq = L.odd[1] & 1; kq = 0; }
            }
        }
        if (tid == 0) {
            MultiPair &out = hw.multi[s];
            out.a2p = a2p; out.a2q = a2q; out.kp = kp; out.kq = kq; out.wkp = wkp; out.wkq = wkq;
            out.fs = fixed_point_bits(make_int4(pm[0], pm[1], pm[2], pm[3]), make_int4(qm[0], qm[1], qm[2], qm[3]));
            out.sum = 0;
            hw.wide[mp.kp].c = -1;
        }
        for (int u = tid; u < mp.units; u += kMetaThreads) {
            const int pw = u / sh.qs, qw = u % sh.qs;
            MultiUnit pre{0, 0};
            for (int j = 0; j < pw; j++) pre.ppre += (int64_t)L.pwin[j];
            for (int j = 0; j < qw; j++) pre.qpre += (int64_t)L.qwin[j];
            hw.units[s * kMultiUnits + u] = pre;
            WidePair e;
            e.c = mp.c; e.pa = mp.pa; e.n = mp.n; e.q = mp.q;
            e.pw = (int16_t)pw;
            e.qw = (int16_t)(sh.qs == 1 ? -1 : qw);
            e.slot = (int32_t)s;
            hw.wide[kWideListCap - 1 - (mp.first + u)] = e;
        }
        // every thread is done with the LDS before the next pair clears it
        __syncthreads();
    }
}

// Cross products of P's window before each of its ncp chunks (lane = chunk),
// from those before the window; returns those up to its end.  One wavefront.
__device__ int64_t chunk_sums(RingLds P, int ncp, int64_t carry, int lane, int64_t *pre)
{
    for (int c0 = 0; c0 < ncp; c0 += 64) {
        const int c = c0 + lane;
        int64_t own = 0;
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const int e = c < ncp ? 8 * c + j : 0;
            const int2 a = P.v[e], b = P.v[e + 1];
            own += (int64_t)a.x * b.y - (int64_t)b.x * a.y;
        }
        own = c < ncp ? own : 0;
        const int64_t upto = carry + wave_incl_scan64(own);
        if (c < ncp) pre[c] = upto - own;
        carry = (int64_t)dpp::readlane64((uint64_t)upto, 63);
    }
    return carry;
}

// One wavefront per deferred pair (workgroups of one wavefront, so five fit a
// CU's LDS), any sizes: both rings pass through LDS in windows of up to
// kWideCap edges, P's windows in the outer loop and Q's in the inner one.
// A crossing's term needs no more of the rings than its own windows and the
// cross products before them, which are carried from window to window.  The
// terms and the sums are those of k_refine's groups and of mid_pairs: whole
// numbers, so that a pair's value is the same bit for bit, whichever of them
// takes it.  P is the data polygon, or the query when the data polygon has more
// than kWideCap edges and more than the query (so a polygon of at most kWideCap
// edges is staged once); exchanging the roles translates the data polygon by
// delta instead of the query: another consistent perturbation with the same
// limit area.
__global__ __launch_bounds__(64) void k_refine_wide(const int32_t *__restrict__ dxy,
                                                    const int32_t *__restrict__ qxy,
                                                    const int64_t *__restrict__ qoff,
                                                    double *__restrict__ cand_j, HeavyWs hw, int want_stats)
{
    __shared__ int2 sQv[kWideRing];
    __shared__ int4 sQbox[kWideCap / 8];
    __shared__ int64_t sQsuf[kWideCap];
    __shared__ int2 sPv[kWideRing];
    __shared__ int4 sPbox[kWideCap / 8];
    __shared__ int64_t sPre[kWideCap / 8 + 1];
    __shared__ uint16_t sList[kListCap];
    __shared__ uint32_t sUnits[kUnitCap];
    __shared__ uint32_t sCross[kGroupCross];

    const int lane = threadIdx.x;
    const int64_t norig = min((int64_t)hw.count[1], (int64_t)kWideListCap);
    const int64_t nunits = max((int64_t)0, min((int64_t)hw.count[4], (int64_t)kWideListCap - norig));
    // nothing deferred, or nothing of more than kWideCap edges (the usual
    // cases): no atomics on the counter
    const bool mids = mids_by_workgroup(hw);     // taken by mid_pairs
    if (norig + nunits <= (mids ? hw.count[5] : 0)) return;
    unsigned long long st_pairs = 0, st_swept = 0;
    // entries are taken from a counter as wavefronts come free, the split
    // pairs' units first: costs range from one window to many
    for (;;) {
        const int64_t t = __builtin_amdgcn_readfirstlane(lane == 0 ? atomicAdd(hw.count + 3, 1) : 0);
        if (t >= norig + nunits) break;
        const WidePair w = hw.wide[t < nunits ? kWideListCap - 1 - t : t - nunits];
        if (w.c < 0) continue;
        const int64_t qa = qoff[w.q];
        const int mq = (int)(qoff[w.q + 1] - qa);
        const bool swap = w.n > kWideCap && w.n > mq;
        const int32_t *Pg = swap ? qxy + 2 * qa : dxy + 2 * w.pa;
        const int32_t *Qg = swap ? dxy + 2 * w.pa : qxy + 2 * qa;
        const int n = swap ? mq : w.n, m = swap ? w.n : mq;
        if (mids && max(n, m) <= kWideCap) continue;
        const int64_t ox = Qg[0], oy = Qg[1];
        // windows of this entry: all, or one P window (and one Q window) of
        // a split pair
        const SplitShape sh = split_shape(n, m);
        const int pfirst = w.pw < 0 ? 0 : w.pw * sh.plen;
        const int pend = w.pw < 0 ? n : min(n, pfirst + sh.plen);
        const int qfirst = w.qw < 0 ? 0 : w.qw * kWideCap;
        const int qend = w.qw < 0 ? m : min(m, qfirst + kWideCap);
        const int u = w.qw < 0 ? w.pw : w.pw * sh.qs + w.qw;   // a split pair's unit slot
        int64_t a2q, a2p, ppre = 0, qpre = 0;
        int kp = 0, kq = 0, wkp = 0, wkq = 0, fs = 0;
        if (w.pw >= 0) {
            // a split pair's unit: the pair's own quantities from wide_meta
            const MultiPair &mp = hw.multi[w.slot];
            a2p = mp.a2p; a2q = mp.a2q; kp = mp.kp; kq = mp.kq; wkp = mp.wkp; wkq = mp.wkq; fs = mp.fs;
            const MultiUnit pre = hw.units[(int64_t)w.slot * kMultiUnits + u];
            ppre = pre.ppre;
            qpre = pre.qpre;
        } else {
            int32_t qm[4], pm[4];
            ring_sums_global(Qg, m, ox, oy, lane, qm, a2q);
            ring_sums_global(Pg, n, ox, oy, lane, pm, a2p);
            fs = fixed_point_bits(make_int4(pm[0], pm[1], pm[2], pm[3]), make_int4(qm[0], qm[1], qm[2], qm[3]));
            if (a2p != 0 && a2q != 0) {
                // anchors: a vertex outside the other polygon's MBR has
                // membership 0; without one, a crossing-number pass
                int qext[4];
                extremes_global(Qg, m, qm, lane, qext);
                kq = anchor_q(qm, pm, qext);
                kp = first_outside_global(Pg, n, qm, lane);
                if (kp < 0) {
                    const int2 p0 = make_int2((int)((int64_t)Pg[0] - ox), (int)((int64_t)Pg[1] - oy));
                    wkp = member_point_global(Qg, m, ox, oy, p0, -1, lane);
                    kp = 0;
                }
                if (kq < 0) {
                    // Q's vertex 0 is the origin
                    wkq = member_point_global(Pg, n, ox, oy, make_int2(0, 0), +1, lane);
                    kq = 0;
                }
            }
        }
        uint64_t acc = 0;
        if (a2p != 0 && a2q != 0) {
            const RingLds Qs{sQv, sQbox, sQsuf}, Ps{sPv, sPbox, nullptr};
            const int pstep = w.pw < 0 ? kWideCap : sh.plen;
            int64_t pcarry = ppre;
            for (int p0 = pfirst; p0 < pend; p0 += pstep) {
                const int plen = min(pstep, pend - p0);
                stage_window(Pg, n, p0, plen, 8 * ((plen + 7) >> 3) + 1, ox, oy, Ps, lane);
                wave_lds_sync();
                chunk_boxes_p<kWideCap / 8>(Ps, plen, lane);
                pcarry = chunk_sums(Ps, (plen + 7) >> 3, pcarry, lane, sPre);
                int64_t qcarry = qpre;
                for (int w0 = qfirst; w0 < qend; w0 += kWideCap) {
                    const int len = min(kWideCap, m - w0);
                    // one all-padding chunk past the window, as for whole rings
                    stage_window(Qg, m, w0, len, 8 * ((len + 7) >> 3) + 9, ox, oy, Qs, lane);
                    wave_lds_sync();
                    chunk_boxes(Qs, len, lane, 64);
                    qcarry = q_suffix_sums(Qs, len, a2q, lane, sQsuf, qcarry);
                    wave_lds_sync();
                    tiled_accumulate<uint32_t, 16, 8, false, kGroupCross>(
                        Ps, (plen + 7) >> 3, Qs, len, lane, nullptr, sList, sUnits, sCross, &st_swept, [&](int count) {
                            if (lane < count) {
                                const uint32_t ef = sCross[lane];
                                const int e = (int)(ef >> 16), f = (int)(ef & 0xffffu);
                                acc += crossing_term(sPv + (e & ~7), e & 7, (p0 + e < kp ? 0 : a2p) - sPre[e >> 3], sQv[f],
                                                     sQv[f + 1], sQsuf[f] - (w0 + f < kq ? a2q : 0), fs);
                            }
                        });
                    // every lane is done with the window before the next one
                    wave_lds_sync();
                }
            }
        }
        acc = (uint64_t)wave_sum_i64((int64_t)acc);
        st_pairs += (w.pw <= 0) & (w.qw <= 0);
        if (lane == 0) {
            bool whole = true;
            if (w.pw >= 0) {
                // A unit adds its terms, then counts itself; whoever counts the
                // last one finds the sum complete.  Both are additions at the
                // device's own scope, and the count waits for the sum's
                // returned value, so no caches are written back in between (a
                // fence a unit cost 5 us: 15,000 pairs of 3,000 edges 9.9 ms).
                unsigned long long before = __hip_atomic_fetch_add(&hw.multi[w.slot].sum, (unsigned long long)acc,
                                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                int32_t one = 1;
                asm volatile("; %1 has returned" : "+v"(one) : "v"(before) : "memory");
                whole = __hip_atomic_fetch_sub(&hw.multi[w.slot].units, one, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) == 1;
                if (whole) acc = __hip_atomic_fetch_add(&hw.multi[w.slot].sum, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            if (whole)
                cand_j[w.c] = a2p != 0 && a2q != 0 ? group_jaccard(acc, wkp, wkq, a2p, a2q, fs) : 0.0;
        }
        // every lane is done with both rings before the next pair restages them
        wave_lds_sync();
    }
    if (want_stats && lane == 0) {
        unsigned long long *slot = hw.stat_slots + (blockIdx.x % kStatSlots) * 4;
        if (st_pairs) atomicAdd(slot + 0, st_pairs);
        if (st_swept) atomicAdd(slot + 1, st_swept);
    }
}

// One wavefront per (heavy pair, side, slice): the slice's share of that
// side's edge sums; slices past the side's last block add nothing.  The one
// that finishes a pair's last slice adds them in a fixed order, then J.
__device__ void heavy_slices(const int32_t *__restrict__ dxy, const int32_t *__restrict__ qxy,
                             double *__restrict__ cand_j, const HeavyWs &hw, int64_t wave, int64_t nw, int lane)
{
    const int64_t count = min(hw.count[0], kHeavyCap);
    for (int64_t t = wave; t < count * 2 * kHeavySlices; t += nw) {
        const int64_t h = t / (2 * kHeavySlices);
        const int side = (int)((t / kHeavySlices) & 1), slice = (int)(t % kHeavySlices);
        const HeavyPair &e = hw.pairs[h];
        PairIn in;
        in.P = dxy + 2 * e.pa; in.n = e.n; in.Q = qxy + 2 * e.qa; in.m = e.m; in.ox = e.ox; in.oy = e.oy;
        for (int i = 0; i < 4; i++) in.qmbr[i] = e.qmbr[i];
        in.sq = e.a2q > 0 ? 1 : -1;
        in.sp = e.a2p > 0 ? 1 : -1;
        int32_t pm[4] = {e.pm[0], e.pm[1], e.pm[2], e.pm[3]};
        double s = 0.0;
        int64_t unused;
        if (side == 0) {
            if (e.wide) edges_in_other_P<true>(in, lane, s, unused, slice, kHeavySlices);
            else edges_in_other_P<false>(in, lane, s, unused, slice, kHeavySlices);
        } else {
            if (e.wide) edges_in_other_Q<true>(in, pm, lane, s, unused, slice, kHeavySlices);
            else edges_in_other_Q<false>(in, pm, lane, s, unused, slice, kHeavySlices);
        }
        s = wave_sum(s);
        if (lane == 0) hw.partial[(h * 2 + side) * kHeavySlices + slice] = s;
        __threadfence();
        // every lane takes part (all but lane 0 with nothing), so that the
        // result is not read across a divergent branch
        const int done = atomicAdd(&hw.pairs[h].done, lane == 0 ? 1 : 0);
        if (__builtin_amdgcn_readfirstlane(done) == 2 * kHeavySlices - 1) {
            __threadfence();
            static_assert(kHeavySlices == 64, "a slice a lane");
            const double vp = hw.partial[(h * 2 + 0) * kHeavySlices + lane];
            const double vq = hw.partial[(h * 2 + 1) * kHeavySlices + lane];
            const double inter2 = wave_sum((double)in.sp * vp) + wave_sum((double)in.sq * vq);
            if (lane == 0) cand_j[e.c] = jaccard_of(inter2, e.a2p, e.a2q);
        }
    }
}

// Pairs of up to kWideCap edges a side, a workgroup each: its first lanes take
// a chunk of P or of Q each (vertices, box, prefix of cross products), its 16
// wavefronts share P's chunks, and the crossings' terms are added as in
// k_refine's groups.  A wavefront a pair, 33 KB of LDS each, left a SIMD with
// one wavefront and the launch with the time of its longest pair (20,000
// pairs of which 595 of 513 to 1,024 edges: 258 us, so 137).
constexpr int kMidWaves = kMetaThreads / 64;

struct MidLds {
    int2 qv[kWideRing];
    int4 qbox[kWideCap / 8];
    int64_t suf[kWideCap];
    int2 pv[kWideCap / 8 * 9];
    int4 pbox[kWideCap / 8];
    int64_t pre[kWideCap / 8 + 1];
    uint8_t pair_of[kWideCap / 8], cid[kWideCap / 8];
    uint16_t list[kMidWaves][kListCap];
    uint32_t units[kMidWaves][kUnitCap];
    uint32_t cross[kMidWaves][kGroupCross];
    int64_t sum[4];              // cross products of P's chunks 0-63, 64-127, Q's
    int4 con;
    unsigned long long acc;
    int32_t mbr[8];              // P's, Q's
    int32_t anchor[2], odd[2], kept[2];
    int32_t taken;
};

__device__ void mid_pairs(MidLds &L, const int32_t *__restrict__ dxy, const int32_t *__restrict__ qxy,
                          const int64_t *__restrict__ qoff, double *__restrict__ cand_j, const HeavyWs &hw, int slot)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t count = min((int64_t)hw.count[1], (int64_t)kWideListCap);
    if (hw.count[5] == 0 || !mids_by_workgroup(hw)) return;
    unsigned long long st_swept = 0, st_pairs = 0;
    if (tid < kWideCap / 8) L.pair_of[tid] = 0;
    for (;;) {
        __syncthreads();
        if (tid == 0) L.taken = atomicAdd(hw.count + 6, 1);
        __syncthreads();
        const int64_t t = __builtin_amdgcn_readfirstlane(L.taken);
        if (t >= count) break;
        const WidePair w = hw.wide[t];
        const int64_t qa = qoff[w.q];
        const int n = __builtin_amdgcn_readfirstlane(w.n), m = __builtin_amdgcn_readfirstlane((int)(qoff[w.q + 1] - qa));
        if (max(n, m) > kWideCap) continue;      // k_refine_wide's
        const int ncp = (n + 7) >> 3, ncq = (m + 7) >> 3;
        // this lane's chunk: of P, of Q (and one of padding), or none
        const bool isq = tid >= kWideCap / 8;
        const int c = isq ? tid - kWideCap / 8 : tid, nv = isq ? m : n;
        const bool mine = isq ? c <= ncq : c < ncp, real = isq ? c < ncq : c < ncp;
        const int2 *V = reinterpret_cast<const int2 *>(isq ? qxy + 2 * qa : dxy + 2 * w.pa);
        const int2 org = *reinterpret_cast<const int2 *>(qxy + 2 * qa);
        int2 v[9];
        int4 box{};
        int64_t cross[8];
        if (tid < 8) L.mbr[tid] = (tid & 3) < 2 ? INT32_MAX : INT32_MIN;
        if (tid < 2) { L.anchor[tid] = -1; L.odd[tid] = 0; }
        if (tid == 0) L.acc = 0;
        __syncthreads();
        int64_t upto = 0, own = 0;
        if (wave <= 4) {
            int2 p[9];
#pragma unroll
            for (int j = 0; j < 9; j++) {
                const int i = mine && 8 * c + j < nv ? 8 * c + j : 0;
                p[j] = V[i];
                v[j] = make_int2(p[j].x - org.x, p[j].y - org.y);
            }
            box = make_int4(p[0].x, p[0].y, p[0].x, p[0].y);
#pragma unroll
            for (int j = 0; j < 8; j++) {
                cross[j] = mine ? (int64_t)v[j].x * v[j + 1].y - (int64_t)v[j + 1].x * v[j].y : 0;
                own += cross[j];
                box.x = min(box.x, p[j + 1].x); box.z = max(box.z, p[j + 1].x);
                box.y = min(box.y, p[j + 1].y); box.w = max(box.w, p[j + 1].y);
            }
            if (mine) {
#pragma unroll
                for (int j = 0; j < 9; j++) {
                    if (!isq) L.pv[9 * c + j] = v[j];
                    else if (j < 8 || c == ncq) L.qv[8 * c + j] = v[j];
                }
            }
            if (real) {
                int32_t *b = L.mbr + (isq ? 4 : 0);
                atomicMin(b, box.x); atomicMin(b + 1, box.y);
                atomicMax(b + 2, box.z); atomicMax(b + 3, box.w);
            }
            upto = wave_incl_scan64(own);
            if (lane == 63 && wave < 4) L.sum[wave] = upto;
        }
        __syncthreads();
        const int64_t a2p = L.sum[0] + L.sum[1], a2q = L.sum[2] + L.sum[3];
        const int32_t *pm = L.mbr, *qm = L.mbr + 4;
        const int fs = fixed_point_bits(make_int4(pm[0], pm[1], pm[2], pm[3]), make_int4(qm[0], qm[1], qm[2], qm[3]));
        bool keep = false;
        uint64_t km = 0;
        if (wave <= 4) {
            upto += (wave == 1 || wave == 3) ? L.sum[wave - 1] : 0;
            const int32_t *o = isq ? pm : qm;
            int out = -1;
            int64_t run = upto - own;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const int x = v[j].x + org.x, y = v[j].y + org.y, i = 8 * c + j;
                if (real && i < nv && ((x < o[0]) | (x > o[2]) | (y < o[1]) | (y > o[3]))) out = i;
                run += cross[j];
                if (isq && real) L.suf[i] = a2q - run;
            }
            if (out >= 0) atomicMax(&L.anchor[isq ? 1 : 0], out);
            const int4 rel = make_int4(box.x - org.x, box.y - org.y, box.z - org.x, box.w - org.y);
            if (isq) {
                if (real) L.qbox[c] = rel;
            } else {
                if (real) L.pre[c] = upto - own;
                if (c == ncp - 1) L.pre[ncp] = upto;
                keep = real & !((box.z < o[0]) | (o[2] < box.x) | (box.w < o[1]) | (o[3] < box.y));
            }
            km = __ballot(keep);
            if (lane == 0 && wave < 2) L.kept[wave] = __popcll(km);
            box = rel;
        }
        __syncthreads();
        if (keep) {
            const int at = lanes_below(km) + (wave == 1 ? L.kept[0] : 0);
            L.pbox[at] = box;
            L.cid[at] = (uint8_t)c;
        }
        int kp = L.anchor[0], kq = L.anchor[1];
        if (kp < 0 || kq < 0) {
            // no anchor: the ring starts' memberships, an edge a thread
            const int e = tid;
            const bool op = kp < 0 && e < m && member_edge(L.qv, e < m ? e : 0, L.pv[0], -1);
            const bool oq = kq < 0 && e < n && member_edge(L.pv, e < n ? e + (e >> 3) : 0, L.qv[0], +1);
            const int cp = __popcll(__ballot(op)), cq = __popcll(__ballot(oq));
            if (lane == 0) { atomicAdd(&L.odd[0], cp); atomicAdd(&L.odd[1], cq); }
        }
        if (tid == 0) L.con = make_int4(0, ncp, max(kp, 0), max(kq, 0) | fs << 16);
        __syncthreads();
        if (a2p != 0 && a2q != 0) {
            const int kept = L.kept[0] + L.kept[1];
            const int b0 = kept * wave / kMidWaves, b1 = kept * (wave + 1) / kMidWaves;
            const RingLds Q{L.qv, L.qbox, nullptr}, P{L.pv, L.pbox + b0, nullptr};
            const GroupLds G{L.pv, L.pre, L.pair_of, &L.con, &L.acc};
            tiled_accumulate<uint32_t, 16, 9, true, kGroupCross>(
                P, b1 - b0, Q, m, lane, L.cid + b0, L.list[wave], L.units[wave], L.cross[wave], &st_swept,
                [&](int got) { flush_group(G, Q, L.suf, a2q, L.cross[wave], got, lane); });
        }
        __syncthreads();
        if (tid == 0) {
            double J = 0.0;
            if (a2p != 0 && a2q != 0) J = group_jaccard(L.acc, L.odd[0] & 1, L.odd[1] & 1, a2p, a2q, L.con.w >> 16);
            cand_j[w.c] = J;
            st_pairs++;
        }
    }
    if (hw.stat_slots && lane == 0) {
        unsigned long long *out = hw.stat_slots + (slot % kStatSlots) * 4;
        if (st_pairs) atomicAdd(out + 0, st_pairs);
        if (st_swept) atomicAdd(out + 1, st_swept);
    }
}

// What k_refine deferred, but for the pairs of more than kWideCap edges: the
// first workgroups prepare those that are split, the next take the heavy
// pairs' slices, the last the pairs of up to kWideCap edges.
constexpr int kMetaBlocks = 256;
__global__ __launch_bounds__(kMetaThreads) void k_deferred(const int32_t *__restrict__ dxy,
                                                         const int32_t *__restrict__ qxy,
                                                         const int64_t *__restrict__ qoff,
                                                         double *__restrict__ cand_j, HeavyWs hw)
{
    constexpr size_t kBytes = sizeof(MidLds) > sizeof(MetaLds) ? sizeof(MidLds) : sizeof(MetaLds);
    __shared__ __align__(16) unsigned char lds[kBytes];
    const int block = (int)blockIdx.x;
    if (block < kMetaBlocks) {
        wide_meta(*reinterpret_cast<MetaLds *>(lds), dxy, qxy, qoff, hw, block, kMetaBlocks);
    } else if (block < 2 * kMetaBlocks) {
        constexpr int kWaves = kMetaThreads / 64;
        const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        heavy_slices(dxy, qxy, cand_j, hw, (int64_t)(block - kMetaBlocks) * kWaves + wave,
                     (int64_t)kMetaBlocks * kWaves, threadIdx.x & 63);
    } else {
        mid_pairs(*reinterpret_cast<MidLds *>(lds), dxy, qxy, qoff, cand_j, hw, block);
    }
}

HeavyWs carve_heavy(Carve &cv)
{
    HeavyWs hw{};
    hw.count = cv.take<int32_t>(64);
    hw.pairs = cv.take<HeavyPair>(kHeavyCap);
    hw.partial = cv.take<double>((size_t)kHeavyCap * 2 * kHeavySlices);
    hw.stat_slots = cv.take<unsigned long long>(kStatSlots * 4);
    hw.wide = cv.take<WidePair>(kWideListCap);
    hw.multi = cv.take<MultiPair>(kMultiCap);
    hw.units = cv.take<MultiUnit>((size_t)kMultiCap * kMultiUnits);
    return hw;
}

// Clears the pair counts, the work counter and the counter slots (256 threads).
__global__ void k_zero_count(int32_t *p, unsigned long long *slots)
{
    if (threadIdx.x < 8) p[threadIdx.x] = 0;
    if (threadIdx.x < kStatSlots * 4) slots[threadIdx.x] = 0;
}

// Adds the counter slots to the caller's four counters (one wavefront).
__global__ void k_fold_stats(const unsigned long long *slots, unsigned long long *stats)
{
    const int i = threadIdx.x;
    if (i < 4) {
        unsigned long long v = 0;
        for (int s = 0; s < kStatSlots; s++) v += slots[s * 4 + i];
        if (v) atomicAdd(stats + i, v);
    }
}

}  // namespace

size_t refine_workspace_bytes()
{
    Carve cv{nullptr, 0};
    carve_heavy(cv);
    return align_up(cv.used, 256);
}

polymh_status launch_refine(const polymh_polys *data, const polymh_polys *queries,
                            const int64_t *cand_off, const int32_t *cand_ids, int64_t nq,
                            int64_t n_cand, double *cand_j, hipStream_t s,
                            unsigned long long *stats, void *ws, size_t ws_bytes)
{
    if (n_cand == 0 || nq == 0) return POLYMH_OK;
    HeavyWs hw{};
    if (ws) {
        Carve cv{static_cast<char *>(ws), ws_bytes};
        hw = carve_heavy(cv);
        if (!cv.ok) return set_error(POLYMH_ECAPACITY, "refine: workspace of %zu bytes, need %zu", ws_bytes, cv.used);
        hipLaunchKernelGGL(k_zero_count, dim3(1), dim3(kStatSlots * 4), 0, s, hw.count, hw.stat_slots);
    }
    if (nq > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "refine: too many queries");
    // a query's candidates are spread over several workgroups (each stages
    // the query once) when the batch is small or its lists are long: at
    // least 2048 workgroups, at most about 128 candidates per workgroup on
    // average (32 per wavefront, a few groups: at 650 candidates a query
    // 7.99 ms, with 64 8.20, with 256 8.09; without a workspace 64, as a pair
    // beyond the tiled form then runs in its wavefront: 300,000 pairs of
    // workload 3 7.2 ms, with 128 8.7), at least 4 (one per wavefront: 35
    // queries of 121 candidates 45 us, with 2 a workgroup 51), at most 64
    // workgroups per query
    const int64_t most = ws ? 128 : 64;
    const int64_t by_batch = std::min((2048 + nq - 1) / nq, (n_cand + nq * 4 - 1) / (nq * 4));
    const int64_t by_length = (n_cand + nq * most - 1) / (nq * most);
    int64_t sl = std::max<int64_t>(1, std::min<int64_t>(64, std::max(by_batch, by_length)));
    if (nq * sl > 0x7fffffffLL) sl = 1;
    const int slices = (int)sl;
    const int mid_taken = ws && n_cand < kMidCand ? (int)(n_cand / kMidShare) : 0;
    hipLaunchKernelGGL(k_refine, dim3((unsigned)(nq * slices)), dim3(64 * kWavesPerBlock), 0, s, data->xy,
                       data->offsets, queries->xy, queries->offsets, cand_off, cand_ids, cand_j, stats,
                       slices, mid_taken, hw);
    polymh_status st = check_launch("refine");
    if (st || !ws) return st;
    hipLaunchKernelGGL(k_deferred, dim3(3 * kMetaBlocks), dim3(kMetaThreads), 0, s, data->xy, queries->xy,
                       queries->offsets, cand_j, hw);
    if ((st = check_launch("refine: deferred pairs"))) return st;
    // deferred wide tiled pairs: the five one-wavefront workgroups a CU's LDS
    // holds (15,000 pairs of 3,000 edges 6.6 ms, with four 8.0)
    hipLaunchKernelGGL(k_refine_wide, dim3((unsigned)(5 * cu_count())), dim3(64), 0, s, data->xy, queries->xy, queries->offsets, cand_j,
                       hw, stats ? 1 : 0);
    if ((st = check_launch("refine: wide pairs"))) return st;
    if (!stats) return POLYMH_OK;
    hipLaunchKernelGGL(k_fold_stats, dim3(1), dim3(64), 0, s, hw.stat_slots, stats);
    return check_launch("refine: counters");
}

}  // namespace polymh
