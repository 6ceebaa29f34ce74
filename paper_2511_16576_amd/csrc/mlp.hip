// Learned candidate scorer: a 288 -> 256 -> 256 -> 1 MLP (GELU, GELU,
// sigmoid) with BF16 weights and activations on the MFMA units, FP32
// accumulation, MSE loss and Adam on FP32 master weights.
//
// Products run on v_mfma_f32_32x32x16_bf16: one wavefront owns 32 x 32 tiles
// of the output and walks K in steps of 16.  Operand fragments: lane l holds
// row (l % 32) of A and column (l % 32) of B, for the 8 consecutive k values
// 8*(l / 32) .. 8*(l / 32) + 7 of the step; result element r of lane l is
// row 8*(r / 4) + 4*(l / 32) + r % 4, column l % 32.
//
// The layers of a 32-row tile of the batch never leave the chip between their
// products: k_mlp_forward runs both hidden layers and the output of a tile
// (each wavefront keeps its 32 hidden units' weights in registers, as the
// fused inference does) and k_mlp_back the way back to the first layer's
// pre-activations; k_wgrad then reduces the weight gradients over the batch.
#include "internal.hpp"
#include "scorer_common.hpp"

#include <algorithm>
#include <cmath>

namespace polymh {

namespace {

constexpr int kIn = kScorerIn, kHid = kScorerHid;

__device__ __forceinline__ __bf16 to_bf16(float x) { return (__bf16)x; }

struct Operand {
    const __bf16 *p;
    int64_t si;  // stride of the row (A) / column (B) index
    int64_t sk;  // stride of the reduction index
};

template <bool KC>
__device__ __forceinline__ bf16x8 frag(const Operand &o, int64_t row, int64_t k)
{
    const __bf16 *q = o.p + row * o.si + k * o.sk;
    if constexpr (KC) {
        return *reinterpret_cast<const bf16x8 *>(q);
    } else {
        bf16x8 v;
#pragma unroll
        for (int t = 0; t < 8; t++) v[t] = q[t * o.sk];
        return v;
    }
}

struct GemmArgs {
    Operand A, B;
    int64_t M, N, K;   // M, N multiples of 32; K multiple of 16
    float *out;
};

// C = A B with arbitrary strides (the exported product): one wavefront a
// 32 x 32 tile, operands from memory.
template <bool AKC, bool BKC>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g)
{
    const int lane = threadIdx.x & 63;
    const int64_t tiles_n = g.N / 32;
    const int64_t tile = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (tile >= (g.M / 32) * tiles_n) return;
    const int64_t i0 = (tile / tiles_n) * 32, j0 = (tile % tiles_n) * 32;
    const int64_t row = i0 + (lane & 31), col = j0 + (lane & 31);
    const int64_t kl = 8 * (lane >> 5);
    f32x16 acc = {};
    for (int64_t k0 = 0; k0 < g.K; k0 += 16) {
        const bf16x8 a = frag<AKC>(g.A, row, k0 + kl);
        const bf16x8 b = frag<BKC>(g.B, col, k0 + kl);
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int64_t i = i0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        g.out[i * g.N + col] = acc[r];
    }
}

// Parameter block (FP32 master): W1[256][288], b1[256], W2[256][256], b2[256], w3[256], b3.
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + (int64_t)kHid * kIn, kOffW2 = kOffB1 + kHid,
                  kOffB2 = kOffW2 + (int64_t)kHid * kHid, kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid,
                  kNParams = kOffB3 + 1;
// BF16 copies: W1 then W2.
constexpr int64_t kNBf16 = (int64_t)kHid * kIn + (int64_t)kHid * kHid;

constexpr int kTile = 32;                        // batch rows of a tile
constexpr int kTileThreads = 512, kTileWaves = kTileThreads / 64;
constexpr int kXStride = kIn + 8, kHStride = kHid + 8;   // LDS row strides (16-byte multiples)
constexpr int kK1 = kIn / 16, kK2 = kHid / 16;
constexpr int kXChunks = kTile * kIn / 8, kHChunks = kTile * kHid / 8;   // 16-byte pieces of a tile

// z += row tile [32][ld] (LDS) x w, a wavefront's 32 columns over K steps.
template <int K>
__device__ __forceinline__ f32x16 tile_product(const __bf16 *rows, int ld, const bf16x8 (&w)[K], int lane)
{
    f32x16 acc = {};
    const __bf16 *a = rows + (lane & 31) * ld + 8 * (lane >> 5);
#pragma unroll
    for (int ks = 0; ks < K; ks++)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(a + 16 * ks), w[ks], acc, 0, 0,
                                                      0);
    return acc;
}
// A 32 x 256 BF16 tile from LDS to rows r0 .. of out [.][256], 16 bytes a lane.
__device__ __forceinline__ void store_tile(const __bf16 *tile, __bf16 *__restrict__ out, int64_t r0)
{
    for (int c = threadIdx.x; c < kHChunks; c += kTileThreads) {
        const int r = c / (kHid / 8), k = c % (kHid / 8);
        *reinterpret_cast<uint4 *>(out + (r0 + r) * kHid + 8 * k) =
            *reinterpret_cast<const uint4 *>(tile + r * kHStride + 8 * k);
    }
}

// sum_j h[j] w3[j] over a row of 256 in LDS, one wavefront a row.
__device__ __forceinline__ float row_dot(const __bf16 *h, const float (&w3)[kHid / 64], int lane)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < kHid / 64; i++) s += (float)h[lane + 64 * i] * w3[i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    return s;
}

// Both hidden layers and the output of 32 rows at a time: z1 = X W1^T + b1,
// h1 = gelu(z1), z2 = h1 W2^T + b2, h2 = gelu(z2), y = sigmoid(h2 . w3 + b3),
// all kept for the backward pass.  One workgroup a CU; the next tile's rows
// are loaded while a tile runs.  Bound: the 512 GELUs a row (VALU) and the 3
// KB a row that the activations take.  8,192 rows 19 us, 200,000 rows 294 us;
// as two products and an output pass through memory 91 and 577 us.
__global__ __launch_bounds__(kTileThreads) void k_mlp_forward(const __bf16 *__restrict__ X, int64_t tiles,
                                                              const float *__restrict__ params,
                                                              const __bf16 *__restrict__ wbf16,
                                                              float *__restrict__ z1, __bf16 *__restrict__ h1,
                                                              float *__restrict__ z2, __bf16 *__restrict__ h2,
                                                              float *__restrict__ y)
{
    __shared__ __attribute__((aligned(16))) __bf16 s_x[kTile * kXStride];
    __shared__ __attribute__((aligned(16))) __bf16 s_h1[kTile * kHStride];
    __shared__ __attribute__((aligned(16))) __bf16 s_h2[kTile * kHStride];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = 32 * wave + (lane & 31), kl = 8 * (lane >> 5);
    constexpr int kPer = (kXChunks + kTileThreads - 1) / kTileThreads;
    uint4 xv[kPer];
    auto load_x = [&](int64_t t) {
        const uint4 *src = reinterpret_cast<const uint4 *>(X + t * kTile * kIn);
#pragma unroll
        for (int i = 0; i < kPer; i++)
            if (tid + i * kTileThreads < kXChunks) xv[i] = src[tid + i * kTileThreads];
    };
    int64_t t = blockIdx.x;
    if (t >= tiles) return;
    load_x(t);
    const __bf16 *W1 = wbf16, *W2 = wbf16 + (int64_t)kHid * kIn;
    bf16x8 w1[kK1], w2[kK2];
#pragma unroll
    for (int ks = 0; ks < kK1; ks++)
        w1[ks] = *reinterpret_cast<const bf16x8 *>(W1 + (int64_t)col * kIn + 16 * ks + kl);
#pragma unroll
    for (int ks = 0; ks < kK2; ks++)
        w2[ks] = *reinterpret_cast<const bf16x8 *>(W2 + (int64_t)col * kHid + 16 * ks + kl);
    const float b1c = params[kOffB1 + col], b2c = params[kOffB2 + col], b3 = params[kOffB3];
    float w3[kHid / 64];
#pragma unroll
    for (int i = 0; i < kHid / 64; i++) w3[i] = params[kOffW3 + lane + 64 * i];
    for (; t < tiles; t += gridDim.x) {
        const int64_t r0 = t * kTile;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int c = tid + i * kTileThreads;
            if (c < kXChunks) *reinterpret_cast<uint4 *>(s_x + (c / (kIn / 8)) * kXStride + 8 * (c % (kIn / 8))) = xv[i];
        }
        if (t + gridDim.x < tiles) load_x(t + gridDim.x);
        __syncthreads();
        f32x16 acc = tile_product(s_x, kXStride, w1, lane);
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int row = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const float z = acc[e] + b1c;
            z1[(r0 + row) * kHid + col] = z;
            s_h1[row * kHStride + col] = to_bf16(gelu(z));
        }
        __syncthreads();
        store_tile(s_h1, h1, r0);
        acc = tile_product(s_h1, kHStride, w2, lane);
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int row = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const float z = acc[e] + b2c;
            z2[(r0 + row) * kHid + col] = z;
            s_h2[row * kHStride + col] = to_bf16(gelu(z));
        }
        __syncthreads();
        store_tile(s_h2, h2, r0);
#pragma unroll
        for (int u = 0; u < kTile / kTileWaves; u++) {
            const int row = wave + kTileWaves * u;
            const float s = row_dot(s_h2 + row * kHStride, w3, lane);
            if (lane == 0) y[r0 + row] = 1.0f / (1.0f + expf(-(s + b3)));
        }
        // s_x is written next by threads past the first product; s_h2's
        // readers are past before its next writes, two barriers on
    }
}

// W2^T in BF16, the operand of the backward product.
__global__ __launch_bounds__(256) void k_transpose_w2(const __bf16 *__restrict__ w2, __bf16 *__restrict__ w2t)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < kHid * kHid; i += gridDim.x * blockDim.x)
        w2t[i] = w2[(i % kHid) * kHid + i / kHid];
}

// Partial sums of a workgroup of k_mlp_back over its rows: columns' db1, db2
// and dw3, then db3 and the loss.
constexpr int kBackItems = 3 * kHid + 2;

// From the loss back to the first layer's pre-activations, 32 rows at a time:
// y and dz3 = 2 (y - label) / B y (1 - y) from h2, dz2 = dz3 w3 gelu'(z2),
// dz1 = (dz2 W2) gelu'(z1); dz2 and dz1 in BF16 for the weight gradients, the
// column sums of the FP32 values and the loss as a workgroup's partials.
// 8,192 rows 19 us (a training step 75 us with all its launches; 286 with a
// launch for each product, derivative, column sum and copy).
__global__ __launch_bounds__(kTileThreads) void k_mlp_back(int64_t tiles, int64_t B, const float *__restrict__ params,
                                                           const __bf16 *__restrict__ w2t,
                                                           const float *__restrict__ z1, const float *__restrict__ z2,
                                                           const __bf16 *__restrict__ h2,
                                                           const float *__restrict__ label, float *__restrict__ y,
                                                           __bf16 *__restrict__ dz1, __bf16 *__restrict__ dz2,
                                                           float *__restrict__ part)
{
    __shared__ __attribute__((aligned(16))) __bf16 s_d2[kTile * kHStride];
    __shared__ __attribute__((aligned(16))) __bf16 s_d1[kTile * kHStride];
    __shared__ float s_dz3[kTile], s_loss[kTile];
    __shared__ float s_sum[3][2][kHid];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = 32 * wave + (lane & 31), kl = 8 * (lane >> 5);
    bf16x8 w[kK2];
#pragma unroll
    for (int ks = 0; ks < kK2; ks++)
        w[ks] = *reinterpret_cast<const bf16x8 *>(w2t + (int64_t)col * kHid + 16 * ks + kl);
    float w3[kHid / 64];
#pragma unroll
    for (int i = 0; i < kHid / 64; i++) w3[i] = params[kOffW3 + lane + 64 * i];
    const float b3 = params[kOffB3];
    const int vc = tid & (kHid - 1), half = tid / kHid;   // column phase: a column, 16 of the 32 rows
    const float w3c = params[kOffW3 + vc];
    float db1 = 0.f, db2 = 0.f, dw3 = 0.f, db3 = 0.f, loss = 0.f;
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t r0 = t * kTile;
        float zz1[16];
#pragma unroll
        for (int e = 0; e < 16; e++)
            zz1[e] = z1[(r0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * kHid + col];
#pragma unroll
        for (int u = 0; u < kTile / kTileWaves; u++) {
            const int row = wave + kTileWaves * u;
            const float s = row_dot(h2 + (r0 + row) * kHid, w3, lane);
            if (lane == 0) {
                const float yy = 1.0f / (1.0f + expf(-(s + b3)));
                const float e = yy - label[r0 + row];
                y[r0 + row] = yy;
                s_dz3[row] = 2.0f * e / (float)B * yy * (1.0f - yy);
                s_loss[row] = e * e / (float)B;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTile / 2; u++) {
            const int row = kTile / 2 * half + u;
            const int64_t i = (r0 + row) * kHid + vc;
            const float d = s_dz3[row] * w3c * gelu_grad(z2[i]);
            db2 += d;
            dw3 += s_dz3[row] * (float)h2[i];
            s_d2[row * kHStride + vc] = to_bf16(d);
        }
        if (tid == 0)
            for (int r = 0; r < kTile; r++) {
                db3 += s_dz3[r];
                loss += s_loss[r];
            }
        __syncthreads();
        store_tile(s_d2, dz2, r0);
        const f32x16 acc = tile_product(s_d2, kHStride, w, lane);
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int row = 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            const float d = acc[e] * gelu_grad(zz1[e]);
            db1 += d;
            s_d1[row * kHStride + col] = to_bf16(d);
        }
        __syncthreads();
        store_tile(s_d1, dz1, r0);
    }
    s_sum[0][lane >> 5][col] = db1;
    s_sum[1][half][vc] = db2;
    s_sum[2][half][vc] = dw3;
    __syncthreads();
    float *out = part + (int64_t)blockIdx.x * kBackItems;
    for (int i = tid; i < 3 * kHid; i += kTileThreads) out[i] = s_sum[i / kHid][0][i % kHid] + s_sum[i / kHid][1][i % kHid];
    if (tid == 0) {
        out[3 * kHid] = db3;
        out[3 * kHid + 1] = loss;
    }
}

// Weight gradients dW2 = dz2^T h1 and dW1 = dz1^T X, reductions over the
// whole batch with outputs of a few dozen tiles: split over the rows
// (blockIdx.x, kc rows each, partials added in order by k_grad_sum, so the
// gradient is deterministic), over 64 output rows (blockIdx.y) and over the
// two products (blockIdx.z), so that 8,192 rows occupy 256 workgroups.  Both
// operands have the batch as the reduction index, which is their slow one:
// 64 rows at a time are transposed into LDS (a thread takes two columns of
// eight rows), where a lane's eight k values are one 16-byte read.  Four
// wavefronts: 32 output rows by half the output columns each.  Bound: the
// transposition through LDS; 8,192 rows 18 us for both products, 31 with a
// tile a wavefront read from memory.
constexpr int kGradRows = 64;                       // batch rows a step
constexpr int kGradStride = kGradRows + 8;
constexpr int kMaxSplit = 64;
constexpr int64_t kW2Size = (int64_t)kHid * kHid, kW1Size = (int64_t)kHid * kIn;

template <int N>
__device__ __forceinline__ void wgrad(const __bf16 *__restrict__ dz, const __bf16 *__restrict__ in, int64_t B,
                                      int64_t kc, float *__restrict__ out, __bf16 *s_a, __bf16 *s_b)
{
    constexpr int kGroups = kGradRows / 8;
    constexpr int kItems = N / 2 * kGroups, kPer = (kItems + 255) / 256;
    constexpr int kMost = (N / 32 + 1) / 2;         // output tiles of a wavefront
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wo = wave & 1, t0 = (wave >> 1) * kMost, nt = min(kMost, N / 32 - t0);
    const int o0 = 64 * blockIdx.y;
    const int64_t lo = (int64_t)blockIdx.x * kc, hi = min(B, lo + kc);
    uint32_t av[8], bv[kPer][8];
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int64_t r = k0 + 8 * (tid >> 5) + u;
            av[u] = r < hi ? *reinterpret_cast<const uint32_t *>(dz + r * kHid + o0 + 2 * (tid & 31)) : 0u;
        }
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int w = tid + 256 * i, c = w % (N / 2), g = w / (N / 2);
#pragma unroll
            for (int u = 0; u < 8; u++) {
                const int64_t r = k0 + 8 * g + u;
                bv[i][u] = w < kItems && r < hi ? *reinterpret_cast<const uint32_t *>(in + r * N + 2 * c) : 0u;
            }
        }
    };
    // two columns of eight rows as two 16-byte rows of the transposed tile
    auto put = [](__bf16 *s, int c, int g, const uint32_t (&v)[8]) {
        uint4 e, o;
        e.x = (v[0] & 0xffffu) | v[1] << 16; o.x = v[0] >> 16 | (v[1] & 0xffff0000u);
        e.y = (v[2] & 0xffffu) | v[3] << 16; o.y = v[2] >> 16 | (v[3] & 0xffff0000u);
        e.z = (v[4] & 0xffffu) | v[5] << 16; o.z = v[4] >> 16 | (v[5] & 0xffff0000u);
        e.w = (v[6] & 0xffffu) | v[7] << 16; o.w = v[6] >> 16 | (v[7] & 0xffff0000u);
        *reinterpret_cast<uint4 *>(s + 2 * c * kGradStride + 8 * g) = e;
        *reinterpret_cast<uint4 *>(s + (2 * c + 1) * kGradStride + 8 * g) = o;
    };
    f32x16 acc[kMost] = {};
    load(lo);
    for (int64_t k0 = lo; k0 < hi; k0 += kGradRows) {
        put(s_a, tid & 31, tid >> 5, av);
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            const int w = tid + 256 * i;
            if (w < kItems) put(s_b, w % (N / 2), w / (N / 2), bv[i]);
        }
        __syncthreads();
        if (k0 + kGradRows < hi) load(k0 + kGradRows);
        const __bf16 *a = s_a + (32 * wo + (lane & 31)) * kGradStride + 8 * (lane >> 5);
        const __bf16 *b = s_b + (32 * t0 + (lane & 31)) * kGradStride + 8 * (lane >> 5);
#pragma unroll
        for (int ks = 0; ks < kGradRows / 16; ks++) {
            const bf16x8 fa = *reinterpret_cast<const bf16x8 *>(a + 16 * ks);
#pragma unroll
            for (int j = 0; j < kMost; j++)
                if (j < nt)
                    acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        fa, *reinterpret_cast<const bf16x8 *>(b + 32 * j * kGradStride + 16 * ks), acc[j], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kMost; j++)
        if (j < nt)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const int row = o0 + 32 * wo + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                out[(int64_t)row * N + 32 * (t0 + j) + (lane & 31)] = acc[j][e];
            }
}

__global__ __launch_bounds__(256, 2) void k_wgrad(const __bf16 *__restrict__ dz1, const __bf16 *__restrict__ dz2,
                                               const __bf16 *__restrict__ X, const __bf16 *__restrict__ h1, int64_t B,
                                               int64_t kc, float *__restrict__ part)
{
    __shared__ __attribute__((aligned(16))) __bf16 s_a[64 * kGradStride];
    __shared__ __attribute__((aligned(16))) __bf16 s_b[kIn * kGradStride];
    float *out = part + (int64_t)blockIdx.x * (kW1Size + kW2Size);
    if (blockIdx.z == 0) wgrad<kIn>(dz1, X, B, kc, out, s_a, s_b);
    else wgrad<kHid>(dz2, h1, B, kc, out + kW1Size, s_a, s_b);
}

// The partials' sums, each in the order of the splits: the weight gradients
// (one thread an entry), then the biases', w3's gradients and the loss (eight
// threads an item, each a run of the partials).
__global__ __launch_bounds__(256) void k_grad_sum(const float *__restrict__ wpart, int nsplit,
                                                  const float *__restrict__ bpart, int nback, int wblocks,
                                                  float *__restrict__ grad, float *__restrict__ loss)
{
    constexpr int64_t kSize = kW1Size + kW2Size;
    if ((int)blockIdx.x < wblocks) {
        const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
        if (e >= kSize) return;
        float v = 0.f;
#pragma unroll 8
        for (int s = 0; s < nsplit; s++) v += wpart[s * kSize + e];
        grad[e < kW1Size ? kOffW1 + e : kOffW2 + e - kW1Size] = v;
        return;
    }
    __shared__ float s_v[8][32];
    const int item = 32 * ((int)blockIdx.x - wblocks) + (threadIdx.x & 31), g = threadIdx.x >> 5;
    const int run = (nback + 7) / 8;
    float v = 0.f;
    if (item < kBackItems) {
#pragma unroll 8
        for (int s = g * run; s < min(nback, (g + 1) * run); s++) v += bpart[(int64_t)s * kBackItems + item];
    }
    s_v[g][threadIdx.x & 31] = v;
    __syncthreads();
    if (g != 0 || item >= kBackItems) return;
    for (int i = 1; i < 8; i++) v += s_v[i][threadIdx.x & 31];
    if (item < kHid) grad[kOffB1 + item] = v;
    else if (item < 2 * kHid) grad[kOffB2 + item - kHid] = v;
    else if (item < 3 * kHid) grad[kOffW3 + item - 2 * kHid] = v;
    else if (item == 3 * kHid) grad[kOffB3] = v;
    else *loss = v;
}

// One Adam step, and the BF16 copy of the weights it moved.
__global__ __launch_bounds__(256) void k_adam(float *__restrict__ p, const float *__restrict__ g,
                                              float *__restrict__ m, float *__restrict__ v, int64_t n,
                                              float lr, float b1, float b2, float eps, float c1, float c2,
                                              __bf16 *__restrict__ wbf16)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.0f - b1) * gi;
        const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
        p[i] = pi;
        if (i < kOffB1) wbf16[i] = to_bf16(pi);
        else if (i >= kOffW2 && i < kOffB2) wbf16[i - kOffW2 + kW1Size] = to_bf16(pi);
    }
}

__global__ __launch_bounds__(256) void k_to_bf16(const float *__restrict__ x, __bf16 *__restrict__ y, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = to_bf16(x[i]);
}

int grid_of(int64_t items, int per)
{
    int64_t g = (items + per - 1) / per;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return (int)g;
}

polymh_status gemm(const GemmArgs &g, hipStream_t s)
{
    const int64_t tiles = (g.M / 32) * (g.N / 32);
    if (tiles == 0) return POLYMH_OK;
    if (tiles > (int64_t)0x7fffffff / 4) return set_error(POLYMH_EINVAL, "mlp: product too large");
    const dim3 grid((unsigned)((tiles + 3) / 4)), block(256);
    const bool akc = g.A.sk == 1, bkc = g.B.sk == 1;
    if (akc && bkc) hipLaunchKernelGGL((k_gemm<true, true>), grid, block, 0, s, g);
    else if (akc) hipLaunchKernelGGL((k_gemm<true, false>), grid, block, 0, s, g);
    else if (bkc) hipLaunchKernelGGL((k_gemm<false, true>), grid, block, 0, s, g);
    else hipLaunchKernelGGL((k_gemm<false, false>), grid, block, 0, s, g);
    return check_launch("mlp gemm");
}

}  // namespace

int64_t mlp_param_count() { return kNParams; }
int64_t mlp_bf16_count() { return kNBf16; }

size_t mlp_acts_bytes(int64_t B)
{
    // z1, z2 (f32), h1, h2 (bf16), y (f32)
    return (size_t)B * kHid * (4 + 4 + 2 + 2) + (size_t)B * 4 + 1024;
}

struct Acts {
    float *z1, *z2, *y;
    __bf16 *h1, *h2;
};

static Acts carve_acts(void *p, int64_t B)
{
    char *c = static_cast<char *>(p);
    Acts a;
    a.z1 = reinterpret_cast<float *>(c);
    c += align_up((size_t)B * kHid * 4, 256);
    a.z2 = reinterpret_cast<float *>(c);
    c += align_up((size_t)B * kHid * 4, 256);
    a.h1 = reinterpret_cast<__bf16 *>(c);
    c += align_up((size_t)B * kHid * 2, 256);
    a.h2 = reinterpret_cast<__bf16 *>(c);
    c += align_up((size_t)B * kHid * 2, 256);
    a.y = reinterpret_cast<float *>(c);
    return a;
}

size_t mlp_acts_bytes_aligned(int64_t B)
{
    return 4 * align_up((size_t)B * kHid * 4, 256) + align_up((size_t)B * 4, 256) + 256;
}

polymh_status launch_mlp_sync_bf16(const float *params, uint16_t *wbf16, hipStream_t s)
{
    __bf16 *w = reinterpret_cast<__bf16 *>(wbf16);
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_of((int64_t)kHid * kIn, 256)), dim3(256), 0, s,
                       params + kOffW1, w, (int64_t)kHid * kIn);
    hipLaunchKernelGGL(k_to_bf16, dim3(grid_of((int64_t)kHid * kHid, 256)), dim3(256), 0, s,
                       params + kOffW2, w + (int64_t)kHid * kIn, (int64_t)kHid * kHid);
    return check_launch("mlp bf16 copy");
}

polymh_status launch_mlp_forward(const uint16_t *X, int64_t B, const float *params,
                                 const uint16_t *wbf16, float *y, void *acts, hipStream_t s)
{
    if (B == 0) return POLYMH_OK;
    Acts a = carve_acts(acts, B);
    const int64_t tiles = B / kTile;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)std::min<int64_t>(tiles, cu_count())), dim3(kTileThreads), 0, s,
                       reinterpret_cast<const __bf16 *>(X), tiles, params, reinterpret_cast<const __bf16 *>(wbf16),
                       a.z1, a.h1, a.z2, a.h2, y ? y : a.y);
    return check_launch("mlp forward");
}

// Loss and parameter gradient of one batch (the forward must have run on the
// same X and acts).  grad [kNParams] is overwritten; loss (device float) is
// overwritten with the batch MSE.  scratch: dz2 and dz1 in BF16, W2^T, and the
// partial sums of k_mlp_back and k_wgrad.
constexpr int kMaxBack = 512;                    // workgroups of k_mlp_back at most

// Steps of a split: at least two, and four rather than more than 32 splits
// (8,192 rows 256 workgroups), until there are kMaxSplit, so that a partial sum
// adds no more than 256 rows up to 16,384.
int64_t split_steps(int64_t B)
{
    const int64_t steps = (B + kGradRows - 1) / kGradRows;
    return std::max({(int64_t)2, std::min((int64_t)4, (steps + 31) / 32), (steps + kMaxSplit - 1) / kMaxSplit});
}
// The most splits of any batch up to B.
int64_t most_splits(int64_t B)
{
    return std::min<int64_t>(kMaxSplit, std::max<int64_t>(32, (B + 4 * kGradRows - 1) / (4 * kGradRows)));
}

size_t mlp_backward_scratch_bytes(int64_t B)
{
    return 2 * align_up((size_t)B * kHid * 2, 256) + align_up((size_t)kW2Size * 2, 256) +
           align_up((size_t)kMaxBack * kBackItems * 4, 256) +
           align_up((size_t)most_splits(B) * (kW1Size + kW2Size) * 4, 256) + 256;
}

polymh_status launch_mlp_backward(const uint16_t *X, int64_t B, const float *params,
                                  const uint16_t *wbf16, void *acts, const float *label,
                                  float *grad, float *loss, void *scratch, hipStream_t s)
{
    if (B == 0) return POLYMH_OK;
    Acts a = carve_acts(acts, B);
    char *c = static_cast<char *>(scratch);
    __bf16 *dz2 = reinterpret_cast<__bf16 *>(c); c += align_up((size_t)B * kHid * 2, 256);
    __bf16 *dz1 = reinterpret_cast<__bf16 *>(c); c += align_up((size_t)B * kHid * 2, 256);
    __bf16 *w2t = reinterpret_cast<__bf16 *>(c); c += align_up((size_t)kW2Size * 2, 256);
    float *bpart = reinterpret_cast<float *>(c); c += align_up((size_t)kMaxBack * kBackItems * 4, 256);
    float *wpart = reinterpret_cast<float *>(c);
    const __bf16 *w2 = reinterpret_cast<const __bf16 *>(wbf16) + kW1Size;
    const int64_t tiles = B / kTile;
    const int nback = (int)std::min<int64_t>(tiles, std::min(cu_count(), kMaxBack));
    hipLaunchKernelGGL(k_transpose_w2, dim3(64), dim3(256), 0, s, w2, w2t);
    hipLaunchKernelGGL(k_mlp_back, dim3(nback), dim3(kTileThreads), 0, s, tiles, B, params, w2t, a.z1, a.z2, a.h2,
                       label, a.y, dz1, dz2, bpart);
    const int64_t kc = split_steps(B) * kGradRows;
    const int nsplit = (int)((B + kc - 1) / kc);
    hipLaunchKernelGGL(k_wgrad, dim3(nsplit, kHid / 64, 2), dim3(256), 0, s, dz1, dz2,
                       reinterpret_cast<const __bf16 *>(X), a.h1, B, kc, wpart);
    const int wblocks = (int)((kW1Size + kW2Size + 255) / 256), bblocks = (kBackItems + 31) / 32;
    hipLaunchKernelGGL(k_grad_sum, dim3(wblocks + bblocks), dim3(256), 0, s, wpart, nsplit, bpart, nback, wblocks, grad,
                       loss);
    return check_launch("mlp backward");
}

polymh_status launch_mlp_adam(float *params, const float *grad, float *m, float *v, int64_t step,
                              float lr, float b1, float b2, float eps, uint16_t *wbf16, hipStream_t s)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(grid_of(kNParams, 256)), dim3(256), 0, s, params, grad, m, v,
                       kNParams, lr, b1, b2, eps, c1, c2, reinterpret_cast<__bf16 *>(wbf16));
    return check_launch("mlp adam");
}

polymh_status launch_gemm_bf16(const uint16_t *A, int64_t sai, int64_t sak, const uint16_t *B,
                               int64_t sbj, int64_t sbk, int64_t M, int64_t N, int64_t K, float *C,
                               hipStream_t s)
{
    GemmArgs g{};
    g.A = Operand{reinterpret_cast<const __bf16 *>(A), sai, sak};
    g.B = Operand{reinterpret_cast<const __bf16 *>(B), sbj, sbk};
    g.M = M; g.N = N; g.K = K; g.out = C;
    return gemm(g, s);
}

}  // namespace polymh
