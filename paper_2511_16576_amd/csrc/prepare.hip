// Polygon staging (Sec. 3.1 global MBR, Alg. 1 local MBR), the sampling box
// of a polygon set, and the longest-expected-first order used by the
// persistent signing launch (expected walk length from Thm. 2).
#include "internal.hpp"

#include <cmath>

namespace polymh {

namespace {

__device__ __forceinline__ int32_t wave_min(int32_t v)
{
    for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ int32_t wave_max(int32_t v)
{
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}
// Over one 16-lane DPP row (quads, then rotations by 4 and 8 within the row):
// every lane of the row receives the row's result.
template <class Op>
__device__ __forceinline__ int32_t row_reduce32(int32_t x, Op op)
{
    x = op(x, dpp::mov<dpp::kQuad1032>(x, x));
    x = op(x, dpp::mov<dpp::kQuad2301>(x, x));
    x = op(x, dpp::mov<dpp::kRowRor4>(x, x));
    x = op(x, dpp::mov<dpp::kRowRor8>(x, x));
    return x;
}
__device__ __forceinline__ uint64_t row_sum_u64(uint64_t v)
{
    v += dpp::mov64<dpp::kQuad1032>(v, v);
    v += dpp::mov64<dpp::kQuad2301>(v, v);
    v += dpp::mov64<dpp::kRowRor4>(v, v);
    v += dpp::mov64<dpp::kRowRor8>(v, v);
    return v;
}

// A lane's share of a polygon's staging: its vertices' box and the sum modulo
// 2^64 of its fan terms (v - v0) x (v' - v0), and whether one is not zero,
// which 64 bits decide while the differences stay below 2^31 (else 128).
struct Staged {
    int32_t mnx = INT32_MAX, mny = INT32_MAX, mxx = INT32_MIN, mxy = INT32_MIN;
    int32_t nz = 0;
    uint64_t acc = 0;

    // lane `l` of kLanes takes every kLanes-th vertex, kU in flight
    template <int kLanes, int kU>
    __device__ __forceinline__ void take(const int32_t *__restrict__ xy, int64_t a, int64_t b, int l)
    {
        const int64_t x0 = xy[2 * a], y0 = xy[2 * a + 1];
        for (int64_t v0 = a; v0 < b; v0 += kLanes * kU) {
            int32_t x[kU], y[kU], xn[kU], yn[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                // past the end: the first vertex, whose fan term is zero
                const int64_t v = v0 + kLanes * u + l < b ? v0 + kLanes * u + l : a, w = v + 1 < b ? v + 1 : a;
                x[u] = xy[2 * v];
                y[u] = xy[2 * v + 1];
                xn[u] = xy[2 * w];
                yn[u] = xy[2 * w + 1];
            }
#pragma unroll
            for (int u = 0; u < kU; u++) {
                mnx = min(mnx, x[u]); mxx = max(mxx, x[u]);
                mny = min(mny, y[u]); mxy = max(mxy, y[u]);
                const int64_t dx = x[u] - x0, dy = y[u] - y0, ex = xn[u] - x0, ey = yn[u] - y0;
                const uint64_t t = (uint64_t)dx * (uint64_t)ey - (uint64_t)ex * (uint64_t)dy;
                acc += t;
                bool any = t != 0;
                if (((dx + (1ll << 31)) | (dy + (1ll << 31)) | (ex + (1ll << 31)) | (ey + (1ll << 31))) >> 32)
                    any = (__int128)dx * ey != (__int128)ex * dy;
                nz |= any ? 1 : 0;
            }
        }
    }
    __device__ __forceinline__ void reduce_row()
    {
        mnx = row_reduce32(mnx, [](int32_t u, int32_t v) { return min(u, v); });
        mny = row_reduce32(mny, [](int32_t u, int32_t v) { return min(u, v); });
        mxx = row_reduce32(mxx, [](int32_t u, int32_t v) { return max(u, v); });
        mxy = row_reduce32(mxy, [](int32_t u, int32_t v) { return max(u, v); });
        nz = row_reduce32(nz, [](int32_t u, int32_t v) { return u | v; });
        acc = row_sum_u64(acc);
    }
    __device__ __forceinline__ void reduce_wave()
    {
        mnx = wave_min32(mnx); mny = wave_min32(mny);
        mxx = wave_max32(mxx); mxy = wave_max32(mxy);
        nz = __ballot(nz != 0) != 0;
        acc = (uint64_t)wave_sum_i64((int64_t)acc);
    }
    __device__ __forceinline__ void write(int64_t p, int64_t m, int32_t *__restrict__ mbr, int64_t *__restrict__ area2,
                                          uint32_t *__restrict__ flags) const
    {
        mbr[4 * p + 0] = m > 0 ? mnx : 0; mbr[4 * p + 1] = m > 0 ? mny : 0;
        mbr[4 * p + 2] = m > 0 ? mxx : 0; mbr[4 * p + 3] = m > 0 ? mxy : 0;
        if (area2) area2[p] = (int64_t)acc;
        if (!flags) return;
        uint32_t f = 0;
        if (m < 3) f |= kFlagFew;
        if (!nz) f |= kFlagCollinear;
        if (m > 0 && ((int64_t)mxx - mnx >= (1ll << 26) || (int64_t)mxy - mny >= (1ll << 26))) f |= kFlagWide;
        flags[p] = f;
    }
};

// MBR, twice the signed area (exact whenever |area2| < 2^63) and flags of
// every polygon.  Bound: the latency of the chain offsets -> vertices ->
// reductions, so `per` = 4 polygons share a wavefront, a 16-lane row each; one
// of more than kRowMost vertices is taken by the whole wavefront afterwards (a
// row alone would need 256 round trips for 8,192 vertices).  2 M polygons of
// 22 vertices 358 us against 878 with a wavefront each.  As long as the CUs
// hold a wavefront for every polygon, each has its own (per = 1): four of
// 300,000 vertices 1.07 ms, 3.92 one after another; 64 of 20,000 69 us, 225.
constexpr int kRowMost = 128;
__global__ __launch_bounds__(256) void k_prepare(const int32_t *__restrict__ xy,
                                                 const int64_t *__restrict__ off, int64_t n,
                                                 int32_t *__restrict__ mbr,
                                                 int64_t *__restrict__ area2,
                                                 uint32_t *__restrict__ flags, int per)
{
    const int lane = threadIdx.x & 63, rl = lane & 15;
    const int64_t step = (((int64_t)gridDim.x * blockDim.x) >> 6) * per;
    for (int64_t p0 = (((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6) * per; p0 < n; p0 += step) {
        const int64_t p = p0 + (lane >> 4);
        const bool in = (lane >> 4) < per && p < n;
        const int64_t a = in ? off[p] : 0, b = in ? off[p + 1] : 0;
        const bool big = b - a > kRowMost;
        Staged s;
        if (b > a && !big) s.take<16, 2>(xy, a, b, rl);
        s.reduce_row();
        if (in && !big && rl == 0) s.write(p, b - a, mbr, area2, flags);
        uint64_t todo = __ballot(big && rl == 0);
        while (todo) {
            const int r = __ffsll((unsigned long long)todo) - 1;
            todo &= todo - 1;
            const int64_t ra = (int64_t)dpp::readlane64((uint64_t)a, r), rb = (int64_t)dpp::readlane64((uint64_t)b, r);
            Staged w;
            w.take<64, 4>(xy, ra, rb, lane);
            w.reduce_wave();
            if (lane == 0) w.write(p0 + (r >> 4), rb - ra, mbr, area2, flags);
        }
    }
}

__global__ void k_box_init(int32_t *acc)
{
    if (threadIdx.x == 0) {
        acc[0] = INT32_MAX; acc[1] = INT32_MAX; acc[2] = INT32_MIN; acc[3] = INT32_MIN;
    }
}

// Bound: HBM once the atomics are few: one set a 1,024-thread workgroup and a
// workgroup a CU (one set a wavefront from 4,096 workgroups, 65,536 atomics on
// one line, took 750 us where the 8.6 M vertices' bytes take 15).
constexpr int kBoxThreads = 1024;
__global__ __launch_bounds__(kBoxThreads) void k_box_of(const int32_t *__restrict__ xy, int64_t nv,
                                                        int32_t *__restrict__ acc)
{
    __shared__ int32_t s_r[4][kBoxThreads / 64];
    int32_t mnx = INT32_MAX, mny = INT32_MAX, mxx = INT32_MIN, mxy = INT32_MIN;
    constexpr int kU = 4;
    const int64_t step = (int64_t)gridDim.x * kBoxThreads;
    for (int64_t v0 = (int64_t)blockIdx.x * kBoxThreads + threadIdx.x; v0 < nv; v0 += step * kU) {
        int32_t x[kU], y[kU];
#pragma unroll
        for (int u = 0; u < kU; u++) {
            const int64_t v = v0 + u * step < nv ? v0 + u * step : v0;
            x[u] = xy[2 * v];
            y[u] = xy[2 * v + 1];
        }
#pragma unroll
        for (int u = 0; u < kU; u++) {
            mnx = min(mnx, x[u]); mxx = max(mxx, x[u]);
            mny = min(mny, y[u]); mxy = max(mxy, y[u]);
        }
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    mnx = wave_min(mnx); mny = wave_min(mny);
    mxx = wave_max(mxx); mxy = wave_max(mxy);
    if (lane == 0) {
        s_r[0][wave] = mnx; s_r[1][wave] = mny;
        s_r[2][wave] = mxx; s_r[3][wave] = mxy;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int c = threadIdx.x;
        int32_t r = s_r[c][0];
        for (int w = 1; w < kBoxThreads / 64; w++) r = c < 2 ? min(r, s_r[c][w]) : max(r, s_r[c][w]);
        if (c < 2) atomicMin(acc + c, r);
        else atomicMax(acc + c, r);
    }
}

constexpr int kBuckets = 64;

// Expected work of a polygon's k walks, in draw units: Thm. 2 gives
// E[draws] = 1/S_p = N_B / N_P (capped), plus the MBR-passing draws that run a
// point-in-polygon test, about (A_mbr / A_P) edges-worth each.  Bucketed by
// log2, longest first.
__device__ __forceinline__ int cost_bucket(const int64_t *off, const int32_t *mbr,
                                           const int64_t *area2, const uint32_t *flags,
                                           int64_t p, double nb, int32_t k, double cap)
{
    if (flags[p] & (kFlagFew | kFlagCollinear)) return kBuckets - 1;
    const double ap = fmax(0.5 * fabs((double)area2[p]), 0.5);
    const double amb = ((double)mbr[4 * p + 2] - mbr[4 * p] + 1) * ((double)mbr[4 * p + 3] - mbr[4 * p + 1] + 1);
    const double n = (double)(off[p + 1] - off[p]);
    const double draws = fmin(nb / ap, cap);
    const double cost = (double)k * (draws + 0.25 * n * fmin(amb / ap, draws));
    int lg = (int)floor(log2(cost + 1.0));
    lg = lg < 0 ? 0 : (lg > kBuckets - 2 ? kBuckets - 2 : lg);
    return (kBuckets - 2) - lg;  // ascending bucket = descending cost
}

// The whole order of a small set (kSmallOrder polygons at most) in one
// workgroup: one launch of 3.4 us at 1,000 polygons instead of four and the
// gaps between them (some 12 us).
constexpr int kSmallOrder = 8192;

__global__ __launch_bounds__(1024) void k_order_small(const int64_t *off, const int32_t *mbr, const int64_t *area2,
                                                      const uint32_t *flags, int32_t n, double nb, int32_t k,
                                                      double cap, int32_t *order)
{
    constexpr int kPer = kSmallOrder / 1024;
    __shared__ int32_t h[kBuckets];
    const int tid = threadIdx.x;
    if (tid < kBuckets) h[tid] = 0;
    __syncthreads();
    int b[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const int p = tid + 1024 * u;
        b[u] = 0;
        rank[u] = 0;
        if (p < n) {
            b[u] = cost_bucket(off, mbr, area2, flags, p, nb, k, cap);
            rank[u] = atomicAdd(&h[b[u]], 1);
        }
    }
    __syncthreads();
    if (tid < kBuckets) {
        const int c = h[tid];
        h[tid] = wave_incl_scan32(c) - c;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const int p = tid + 1024 * u;
        if (p < n) order[h[b[u]] + rank[u]] = p;
    }
}

__global__ void k_order_init(int32_t *counts)
{
    if (threadIdx.x < 2 * kBuckets) counts[threadIdx.x] = 0;
}

__global__ __launch_bounds__(256) void k_order_hist(const int64_t *off, const int32_t *mbr,
                                                    const int64_t *area2, const uint32_t *flags,
                                                    int64_t n, double nb, int32_t k, double cap,
                                                    int32_t *counts)
{
    __shared__ int32_t h[kBuckets];
    if (threadIdx.x < kBuckets) h[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
         p += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(&h[cost_bucket(off, mbr, area2, flags, p, nb, k, cap)], 1);
    __syncthreads();
    if (threadIdx.x < kBuckets && h[threadIdx.x]) atomicAdd(&counts[threadIdx.x], h[threadIdx.x]);
}

__global__ void k_order_scan(int32_t *counts)
{
    // counts[0..63] histogram -> counts[64..127] exclusive prefix (cursors)
    if (threadIdx.x == 0) {
        int32_t s = 0;
        for (int b = 0; b < kBuckets; b++) {
            counts[kBuckets + b] = s;
            s += counts[b];
        }
    }
}

// Each block reserves, per bucket, one contiguous range of the order with a
// single global atomic, then places its polygons inside it through LDS
// atomics (one block-stride slice of polygons per pass).
__global__ __launch_bounds__(256) void k_order_scatter(const int64_t *off, const int32_t *mbr,
                                                       const int64_t *area2, const uint32_t *flags,
                                                       int64_t n, double nb, int32_t k, double cap,
                                                       int32_t *counts, int32_t *order)
{
    __shared__ int32_t h[kBuckets];
    __shared__ int32_t base[kBuckets];
    for (int64_t p0 = (int64_t)blockIdx.x * blockDim.x; p0 < n; p0 += (int64_t)gridDim.x * blockDim.x) {
        if (threadIdx.x < kBuckets) h[threadIdx.x] = 0;
        __syncthreads();
        const int64_t p = p0 + threadIdx.x;
        int b = -1, rank = 0;
        if (p < n) {
            b = cost_bucket(off, mbr, area2, flags, p, nb, k, cap);
            rank = atomicAdd(&h[b], 1);
        }
        __syncthreads();
        if (threadIdx.x < kBuckets && h[threadIdx.x])
            base[threadIdx.x] = atomicAdd(&counts[kBuckets + threadIdx.x], h[threadIdx.x]);
        __syncthreads();
        if (b >= 0) order[base[b] + rank] = (int32_t)p;
        __syncthreads();
    }
}

__global__ __launch_bounds__(256) void k_fill_u64(unsigned long long *p, int64_t count,
                                                  unsigned long long v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

int grid_for(int64_t items, int per_block, int max_blocks)
{
    int64_t g = (items + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > max_blocks) g = max_blocks;
    return (int)g;
}

}  // namespace

polymh_status launch_prepare(const int32_t *xy, const int64_t *off, int64_t n, int32_t *mbr,
                             int64_t *area2, uint32_t *flags, hipStream_t s)
{
    if (n == 0) return POLYMH_OK;
    const int per = n <= 16 * (int64_t)cu_count() ? 1 : 4;
    hipLaunchKernelGGL(k_prepare, dim3(grid_for(n, 4 * per, 1 << 16)), dim3(256), 0, s, xy, off, n, mbr,
                       area2, flags, per);
    return check_launch("prepare");
}

polymh_status launch_box_of(const int32_t *xy, int64_t nv, int32_t *acc4, hipStream_t s)
{
    hipLaunchKernelGGL(k_box_init, dim3(1), dim3(64), 0, s, acc4);
    if (nv > 0)
        hipLaunchKernelGGL(k_box_of, dim3(grid_for(nv, kBoxThreads, cu_count())), dim3(kBoxThreads), 0, s, xy, nv,
                           acc4);
    return check_launch("box_of");
}

polymh_status launch_sign_order(const int64_t *off, const int32_t *mbr, const int64_t *area2,
                                const uint32_t *flags, int64_t n, polymh_box box, int32_t k,
                                uint32_t cap, int32_t *counts, int32_t *order, hipStream_t s)
{
    const double nb = ((double)box.xmax - box.xmin + 1) * ((double)box.ymax - box.ymin + 1);
    if (n <= kSmallOrder) {
        hipLaunchKernelGGL(k_order_small, dim3(1), dim3(1024), 0, s, off, mbr, area2, flags, (int32_t)n, nb, k,
                           (double)cap, order);
        return check_launch("sign_order");
    }
    hipLaunchKernelGGL(k_order_init, dim3(1), dim3(2 * kBuckets), 0, s, counts);
    const int g = grid_for(n, 256, 2048);
    hipLaunchKernelGGL(k_order_hist, dim3(g), dim3(256), 0, s, off, mbr, area2, flags, n, nb, k,
                       (double)cap, counts);
    hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(64), 0, s, counts);
    hipLaunchKernelGGL(k_order_scatter, dim3(g), dim3(256), 0, s, off, mbr, area2, flags, n, nb,
                       k, (double)cap, counts, order);
    return check_launch("sign_order");
}

polymh_status launch_fill_u64(unsigned long long *p, int64_t count, unsigned long long v,
                              hipStream_t s)
{
    if (count <= 0) return POLYMH_OK;
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(count, 256, 4096)), dim3(256), 0, s, p, count, v);
    return check_launch("fill");
}

}  // namespace polymh
