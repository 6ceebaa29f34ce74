// LSH band keys over MinHash signatures (Sec. 3.2's hashmap of codes, in the
// banded form of the MMDS technique the paper cites).  One thread per
// (polygon, band): r chained SplitMix64 mixes of the band's rows.
#include "internal.hpp"

namespace polymh {

namespace {

// kVec: rows of four values are read 16 bytes at a time (r and k multiples of
// 4, sig 16-byte aligned: then every band's row is).  Bound: HBM: 4 M rows of
// 256 in 64 bands 1.15 ms, 5.3 TB/s (1.61 ms with 4-byte loads and 64-bit
// divisions).
template <bool kVec, class Index>
__global__ __launch_bounds__(256) void k_band(const uint32_t *__restrict__ sig, Index total, int32_t k,
                                              int32_t b, int32_t r, uint64_t band_seed,
                                              uint64_t *__restrict__ keys)
{
    for (Index id = (Index)blockIdx.x * blockDim.x + threadIdx.x; id < total; id += (Index)gridDim.x * blockDim.x) {
        const Index p = id / (Index)b;
        const int32_t t = (int32_t)(id - p * (Index)b);
        const uint32_t *row = sig + (int64_t)p * k + (int64_t)t * r;
        uint64_t f = mix64(band_seed + (uint64_t)(t + 1) * kGamma);
        if constexpr (kVec) {
            for (int32_t u = 0; u < r; u += 4) {
                const uint4 v = *reinterpret_cast<const uint4 *>(row + u);
                f = mix64(f ^ (uint64_t)v.x);
                f = mix64(f ^ (uint64_t)v.y);
                f = mix64(f ^ (uint64_t)v.z);
                f = mix64(f ^ (uint64_t)v.w);
            }
        } else {
            for (int32_t u = 0; u < r; u++) f = mix64(f ^ (uint64_t)row[u]);
        }
        keys[id] = f;
    }
}

}  // namespace

polymh_status launch_band(const uint32_t *sig, int64_t n, int32_t k, int32_t b, int32_t r,
                          uint64_t band_seed, uint64_t *keys, hipStream_t s)
{
    const int64_t total = n * b;
    if (total == 0) return POLYMH_OK;
    int64_t g = (total + 255) / 256;
    if (g > 65536) g = 65536;
    const bool vec = r % 4 == 0 && k % 4 == 0 && reinterpret_cast<uintptr_t>(sig) % 16 == 0;
    // 32-bit indices while the last stride past the end stays below 2^32
    if (total <= 0x7fffffffLL) {
        if (vec)
            hipLaunchKernelGGL((k_band<true, uint32_t>), dim3((unsigned)g), dim3(256), 0, s, sig, (uint32_t)total, k, b,
                               r, band_seed, keys);
        else
            hipLaunchKernelGGL((k_band<false, uint32_t>), dim3((unsigned)g), dim3(256), 0, s, sig, (uint32_t)total, k,
                               b, r, band_seed, keys);
    } else if (vec) {
        hipLaunchKernelGGL((k_band<true, int64_t>), dim3((unsigned)g), dim3(256), 0, s, sig, total, k, b, r, band_seed,
                           keys);
    } else {
        hipLaunchKernelGGL((k_band<false, int64_t>), dim3((unsigned)g), dim3(256), 0, s, sig, total, k, b, r, band_seed,
                           keys);
    }
    return check_launch("band");
}

}  // namespace polymh
