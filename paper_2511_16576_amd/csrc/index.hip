// Bucket table of Sec. 3.2's hashmap: a stable radix sort of the n*b
// (band key, entry index p*b + t) pairs by the 64-bit key.
//
// Band keys are SplitMix64 outputs, so a few of their eight 8-bit digits
// almost determine the order.  One read of the keys counts all eight digits
// (k_sort_hist); k_sort_plan then chooses, from the top digit down, as many
// as the counts say are needed to leave few equal prefixes, skips digits
// with a single value, and takes all eight when the keys are not spread (the
// sort is then complete, as a plain LSD sort).  The chosen digits are sorted
// low to high, one launch a digit (k_sort_pass), and k_sort_fix /
// k_sort_fix_long put right the runs of equal prefixes whose keys differ.
//
// k_sort_pass moves each entry once (12 B in, 12 B out): a tile's digit
// counts become global positions by looking back over the counts that the
// tiles before it have published, so no counting launch re-reads the keys.
// Bound: HBM.  4 M polygons in 64 bands (256 M entries, 12 B each) take four
// passes: 10.3 ms in all, against 36.4 for eight passes that counted, scanned
// and scattered in launches of their own; 70 K entries 62 us against 236
// (13 launches against 32).
#include "internal.hpp"

namespace polymh {

namespace {

constexpr int kRadix = 256;
constexpr int kDigits = 8;
constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kItemsBig = 16, kItemsSmall = 8;   // entries per thread per tile
// Below this many entries the smaller tile is used, so that enough
// workgroups share the sort: 0.5 M entries take 77 us in tiles of 4,096 and
// 84 in tiles of 8,192, 1 M 112 and 115, 2 M 165 and 143, 34 M 1,544 and 1,260.
constexpr int64_t kBigFrom = (int64_t)3 << 19;

struct SortPlan {
    uint32_t mask;        // digits sorted, bit d = bits 8d..8d+7
    uint32_t low;         // entries end up sorted by key >> 8*low
    uint8_t src[kDigits]; // buffer a digit's pass reads: 0 the caller's keys, 1 temporaries, 2 outputs
};

struct SortBufs {
    const uint64_t *keys;            // input; value = entry index
    uint64_t *tk, *ok;               // temporaries and outputs
    int32_t *ti, *oi;
    uint32_t *hist;                  // [kDigits][kRadix] counts, then exclusive offsets
    uint32_t *tickets;               // [kDigits] next tile of each pass
    uint32_t *n_long;                // runs left to k_sort_fix_long
    SortPlan *plan;
    unsigned long long *desc;        // [tiles][kRadix] published counts
    uint32_t *claim;                 // one bit per position: run start taken
    uint32_t *long_runs;
    int64_t m;
    uint32_t tiles;
};

// The lanes of `among` whose 8-bit digit equals this lane's.
__device__ __forceinline__ uint64_t same_digit(uint32_t d, uint64_t among)
{
    uint32_t lo = (uint32_t)among, hi = (uint32_t)(among >> 32);
#pragma unroll
    for (int bit = 0; bit < 8; bit++) {
        const uint32_t m = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);   // all ones where the bit is set
        const uint64_t bb = __ballot(m != 0);
        lo &= ~((uint32_t)bb ^ m);
        hi &= ~((uint32_t)(bb >> 32) ^ m);
    }
    return ((uint64_t)hi << 32) | lo;
}

__global__ __launch_bounds__(256) void k_sort_init(unsigned long long *p, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// All eight digit counts from one read of the keys.
__global__ __launch_bounds__(kThreads) void k_sort_hist(SortBufs B)
{
    __shared__ uint32_t h[kDigits * kRadix];
    for (int i = threadIdx.x; i < kDigits * kRadix; i += kThreads) h[i] = 0;
    __syncthreads();
    constexpr int kU = 4;
    for (int64_t e0 = (int64_t)blockIdx.x * (kThreads * kU); e0 < B.m; e0 += (int64_t)gridDim.x * (kThreads * kU)) {
        uint64_t k[kU];
#pragma unroll
        for (int u = 0; u < kU; u++) {
            const int64_t e = e0 + u * kThreads + threadIdx.x;
            k[u] = e < B.m ? B.keys[e] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; u++) {
            if (e0 + u * kThreads + threadIdx.x < B.m) {
#pragma unroll
                for (int d = 0; d < kDigits; d++)
                    atomicAdd(&h[d * kRadix + ((uint32_t)(k[u] >> (8 * d)) & 0xffu)], 1u);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kDigits * kRadix; i += kThreads)
        if (h[i]) atomicAdd(&B.hist[i], h[i]);
}

// One wavefront per digit: exclusive offsets of its counts and its effective
// bits, -log2 of the chance that two entries agree on it; then the digits to
// sort.  Digits are taken from the top until their bits reach log2(m) + 4:
// among spread keys at most about m / 32 pairs of neighbours are then out of
// order, which k_sort_fix mends in less than the pass that it saves (1.7
// against 1.95 ms at 256 M entries).
__global__ __launch_bounds__(kThreads) void k_sort_plan(SortBufs B, int in_place)
{
    __shared__ float s_bits[kDigits];
    const int lane = threadIdx.x & 63, d = threadIdx.x >> 6;
    uint32_t *h = B.hist + d * kRadix;
    uint32_t c[4], s = 0;
    double sq = 0.0;
    for (int i = 0; i < 4; i++) {
        c[i] = h[4 * lane + i];
        const double p = (double)c[i] / (double)B.m;
        sq += p * p;
        s += c[i];
    }
    uint32_t at = (uint32_t)wave_incl_scan32((int)s) - s;
    sq = wave_sum_f64(sq);
    bool single = false;
    for (int i = 0; i < 4; i++) {
        single |= (int64_t)c[i] == B.m;
        h[4 * lane + i] = at;
        at += c[i];
    }
    const bool one_value = __ballot(single) != 0;
    if (lane == 0) s_bits[d] = one_value ? 0.f : fmaxf((float)-log2(sq), 1e-6f);
    __syncthreads();
    if (threadIdx.x != 0) return;
    const float need = log2f((float)B.m) + 4.f;
    uint32_t mask = 0;
    int low = kDigits;
    float got = 0.f;
    while (low > 0 && got < need) {
        low--;
        if (s_bits[low] > 0.f) {
            mask |= 1u << low;
            got += s_bits[low];
        }
    }
    if (mask == 0) mask = 1u << (kDigits - 1);
    // keys that share memory with the outputs are read by the first pass
    // only, which must then write the temporaries: an even number of passes
    if (in_place && (__popc(mask) & 1)) {
        int d2 = low > 0 ? low - 1 : 0;
        while (mask >> d2 & 1u) d2++;
        mask |= 1u << d2;
    }
    SortPlan p{};
    p.mask = mask;
    p.low = (uint32_t)low;
    int left = __popc(mask), from = 0;
    for (int i = 0; i < kDigits; i++) {
        if (!(mask >> i & 1u)) continue;
        p.src[i] = (uint8_t)from;
        left--;
        from = (left & 1) ? 1 : 2;   // the last pass writes the outputs
    }
    *B.plan = p;
}

// One digit's stable scatter.  Workgroups take tiles by ticket, in order, and
// finish one before they start the next, so the first unfinished tile never
// waits and waiting for the published counts of earlier ones always ends.  A
// wavefront holds kItems x 64 consecutive entries; its lanes with equal
// digits find each other by ballots, and a count per (wavefront, digit) in
// LDS gives each entry its place in the tile.  The tile is reordered through
// LDS so that the stores of a digit are consecutive; the next tile's entries
// are loaded meanwhile.  desc: the count with, in the upper word, 2 * digit
// + 1 (the tile's own count) or 2 * digit + 2 (count of the tile and all
// before it); the digit in the tag keeps one pass's words apart from
// another's.  Measured at 256 M entries: 1.95 ms a pass (3.1 TB/s); with the
// same traffic written in input order 1.68, and without looking back 1.37.
// One 512-thread workgroup a CU (its registers allow no second) is faster
// than more of fewer registers or smaller tiles (10.6 ms in all before the
// prefetch, against 15.8 for two 1,024-thread workgroups and 12.3 for 256
// threads): more tiles in flight means looking back further.
template <int kItems>
__global__ __launch_bounds__(kThreads, 2) void k_sort_pass(SortBufs B, int digit)
{
    constexpr int kTile = kThreads * kItems;
    const uint32_t mask = B.plan->mask;
    if (!(mask >> digit & 1u)) return;
    const int from = B.plan->src[digit];
    // the number of passes left decides where this one writes
    const bool to_out = !(__popc(mask >> (digit + 1)) & 1);
    const uint64_t *__restrict__ in_k = from == 0 ? B.keys : from == 1 ? B.tk : B.ok;
    const int32_t *__restrict__ in_i = from == 0 ? nullptr : from == 1 ? B.ti : B.oi;
    uint64_t *__restrict__ out_k = to_out ? B.ok : B.tk;
    int32_t *__restrict__ out_i = to_out ? B.oi : B.ti;

    __shared__ uint64_t s_key[kTile];
    __shared__ uint16_t s_cnt[kWaves][kRadix];
    __shared__ uint32_t s_gbase[kRadix];
    __shared__ uint32_t s_wsum[kRadix / 64];
    __shared__ uint32_t s_tile;
    int32_t *s_id = reinterpret_cast<int32_t *>(s_key);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int shift = 8 * digit;
    const int w0 = wave * (64 * kItems) + lane;
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
    const unsigned long long tag_own = (unsigned long long)(2 * digit + 1) << 32,
                             tag_all = (unsigned long long)(2 * digit + 2) << 32;
    uint64_t key[kItems];
    int32_t id[kItems];
    auto load_keys = [&](uint32_t t) {
        const int64_t base = (int64_t)t * kTile + w0;
#pragma unroll
        for (int i = 0; i < kItems; i++) key[i] = base + 64 * i < B.m ? in_k[base + 64 * i] : ~0ull;
    };
    auto load_ids = [&](uint32_t t) {
        const int64_t base = (int64_t)t * kTile + w0;
#pragma unroll
        for (int i = 0; i < kItems; i++)
            id[i] = !in_i ? (int32_t)(base + 64 * i) : base + 64 * i < B.m ? in_i[base + 64 * i] : 0;
    };

    if (tid == 0) s_tile = atomicAdd(&B.tickets[digit], 1u);
    for (int i = tid; i < kWaves * kRadix; i += kThreads) (&s_cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t tile = s_tile;
    if (tile < B.tiles) {
        load_keys(tile);
        load_ids(tile);
    }
    while (tile < B.tiles) {
        const int cnt = (int)min((int64_t)kTile, B.m - (int64_t)tile * kTile);
        uint32_t pos[kItems];
        volatile uint16_t *wc = s_cnt[wave];
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const bool valid = w0 + 64 * i < cnt;
            const uint32_t d = (uint32_t)(key[i] >> shift) & 0xffu;
            const uint64_t eq = same_digit(d, __ballot(valid));
            const uint32_t before = (uint32_t)__popcll(eq & lt);
            const uint32_t pre = wc[d];
            pos[i] = pre + before;
            __builtin_amdgcn_wave_barrier();
            if (valid && before == 0) wc[d] = (uint16_t)(pre + (uint32_t)__popcll(eq));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        uint32_t tot = 0, incl = 0;
        if (tid < kRadix) {
            for (int w = 0; w < kWaves; w++) {
                const uint32_t c = s_cnt[w][tid];
                s_cnt[w][tid] = (uint16_t)tot;
                tot += c;
            }
            __hip_atomic_store(&B.desc[(int64_t)tile * kRadix + tid], (tile ? tag_own : tag_all) | tot,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            incl = (uint32_t)wave_incl_scan32((int)tot);
            if (lane == 63) s_wsum[wave] = incl;
        }
        __syncthreads();
        uint32_t start = 0;
        if (tid < kRadix) {
            start = incl - tot;
            for (int w = 0; w < wave; w++) start += s_wsum[w];
            for (int w = 0; w < kWaves; w++) s_cnt[w][tid] += (uint16_t)start;
        }
        if (tid == kThreads - 1) s_tile = atomicAdd(&B.tickets[digit], 1u);
        __syncthreads();
        const uint32_t next = s_tile;
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const uint32_t d = (uint32_t)(key[i] >> shift) & 0xffu;
            pos[i] += s_cnt[wave][d];
            if (w0 + 64 * i < cnt) s_key[pos[i]] = key[i];
        }
        if (next < B.tiles) load_keys(next);
        if (tid < kRadix) {
            uint32_t before = 0;
            if (tile) {
                constexpr int kBack = 4;   // published words in flight at once
                int64_t p = (int64_t)tile - 1;
                bool done = false;
                while (!done) {
                    unsigned long long v[kBack];
#pragma unroll
                    for (int u = 0; u < kBack; u++)
                        v[u] = p - u >= 0 ? __hip_atomic_load(&B.desc[(p - u) * kRadix + tid], __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)
                                          : 0ull;
                    int used = 0;
#pragma unroll
                    for (int u = 0; u < kBack; u++) {
                        if (done || used < u) continue;
                        const unsigned long long tag = v[u] & ~0xffffffffull;
                        if (tag == tag_all) {
                            before += (uint32_t)v[u];
                            done = true;
                        } else if (tag == tag_own) {
                            before += (uint32_t)v[u];
                            used = u + 1;
                        }
                    }
                    p -= used;
                    if (!done && used == 0) __builtin_amdgcn_s_sleep(1);
                }
                __hip_atomic_store(&B.desc[(int64_t)tile * kRadix + tid], tag_all | (before + tot),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s_gbase[tid] = B.hist[digit * kRadix + tid] + before - start;
        }
        __syncthreads();
        uint32_t dst[kItems];
#pragma unroll
        for (int i = 0; i < kItems; i++) {
            const int j = i * kThreads + tid;
            if (j < cnt) {
                const uint64_t k = s_key[j];
                dst[i] = s_gbase[(uint32_t)(k >> shift) & 0xffu] + (uint32_t)j;
                out_k[dst[i]] = k;
            }
        }
        for (int i = tid; i < kWaves * kRadix; i += kThreads) (&s_cnt[0][0])[i] = 0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; i++)
            if (w0 + 64 * i < cnt) s_id[pos[i]] = id[i];
        if (next < B.tiles) load_ids(next);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kItems; i++)
            if (i * kThreads + tid < cnt) out_i[dst[i]] = s_id[i * kThreads + tid];
        __syncthreads();
        tile = next;
    }
}

// Runs of equal prefixes whose keys are out of order.  Every position i with
// an equal prefix but a larger key than its neighbour i + 1 leads to its run.
// A run of up to kShortRun entries inside a tile is found in the tile's copy
// in LDS, by its first such position alone, and sorted by a group of 16
// lanes.  The others are sought in memory, where workgroups may meet: one
// claim (the bit of the run's start) decides who sorts a run.  Prefixes do
// not change while a run is sorted, so the search for its ends is safe beside
// another workgroup's sort, and what is read of the lower bits there only
// decides whether to try a claim.
constexpr int kFixThreads = 256, kFixItems = 8, kShortRun = 16;

__global__ __launch_bounds__(kFixThreads) void k_sort_fix(SortBufs B)
{
    const uint32_t low = B.plan->low;
    if (low == 0) return;
    const int shift = 8 * (int)low;
    constexpr int kSpan = kFixThreads * kFixItems;
    __shared__ uint64_t s_key[kSpan + 1];
    __shared__ uint16_t s_list[kSpan], s_run[kSpan];
    __shared__ uint64_t s_down[kSpan / 64];
    __shared__ uint32_t s_n, s_nrun, s_nmore;
    uint16_t *s_more = s_list;        // entries of s_list that are still needed move to its front
    uint64_t *key = B.ok;
    int32_t *id = B.oi;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t b0 = (int64_t)blockIdx.x * kSpan; b0 + 1 < B.m; b0 += (int64_t)gridDim.x * kSpan) {
        const int cnt = (int)min((int64_t)kSpan, B.m - b0);
        if (threadIdx.x == 0) {
            s_n = s_nrun = s_nmore = 0;
            s_key[cnt] = cnt == kSpan && b0 + cnt < B.m ? key[b0 + cnt] : ~0ull;
        }
#pragma unroll
        for (int u = 0; u < kFixItems; u++) {
            const int i = u * kFixThreads + threadIdx.x;
            if (i < cnt) s_key[i] = key[b0 + i];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kFixItems; u++) {
            const int i = u * kFixThreads + threadIdx.x;
            const bool down = i < cnt && s_key[i] > s_key[i + 1] && (s_key[i] ^ s_key[i + 1]) >> shift == 0;
            const uint64_t all = __ballot(down);
            if (lane == 0) s_down[i >> 6] = all;
            if (down) s_list[atomicAdd(&s_n, 1u)] = (uint16_t)i;
        }
        __syncthreads();
        const uint32_t n = s_n;
        for (uint32_t t0 = 0; t0 < n; t0 += kFixThreads) {
            const uint32_t t = t0 + threadIdx.x;
            int i = 0, kind = 0;           // 1: short run inside the tile, 2: another
            int s = 0, e = 0;
            if (t < n) {
                i = s_list[t];
                const uint64_t pre = s_key[i] >> shift;
                // an earlier such place of the run, if there is one, leads to
                // it (entries are in order of their prefixes, so one with the
                // same prefix is in the same run)
                int w = i >> 6;
                uint64_t bits = s_down[w] & ((1ull << (i & 63)) - 1);
                while (bits == 0 && w > 0 && s_key[w << 6] >> shift == pre) bits = s_down[--w];
                if (bits == 0 || s_key[(w << 6) + 63 - __clzll((long long)bits)] >> shift != pre) {
                    kind = 1;
                    s = i;
                    e = i + 2;
                    while (s > 0 && i - s < kShortRun && s_key[s - 1] >> shift == pre) s--;
                    while (e < cnt && e - s <= kShortRun && s_key[e] >> shift == pre) e++;
                    if (e - s > kShortRun || s == 0 || e >= cnt) kind = 2;
                }
            }
            __syncthreads();               // s_list[t0 ..] has been read
            if (kind == 1) s_run[atomicAdd(&s_nrun, 1u)] = (uint16_t)(s << 4 | (e - s - 1));
            if (kind == 2) s_more[atomicAdd(&s_nmore, 1u)] = (uint16_t)i;
        }
        __syncthreads();
        for (uint32_t t = threadIdx.x >> 4; t < s_nrun; t += kFixThreads / 16) {
            const int s = s_run[t] >> 4, len = (s_run[t] & 15) + 1, l = threadIdx.x & 15;
            const uint64_t k = s_key[s + (l < len ? l : 0)];
            const int32_t v = id[b0 + s + (l < len ? l : 0)];
            int rank = 0;
            for (int u = 0; u < len; u++) {
                const uint64_t ku = s_key[s + u];
                rank += (ku < k || (ku == k && u < l)) ? 1 : 0;
            }
            if (l < len) {
                key[b0 + s + rank] = k;
                id[b0 + s + rank] = v;
            }
        }
        // longer ones: one wavefront each; up to 64 entries are sorted in
        // registers, more are left to k_sort_fix_long
        for (uint32_t t = wave; t < s_nmore; t += kFixThreads / 64) {
            const int64_t i = b0 + s_more[t];
            const uint64_t pre = key[i] >> shift;
            int64_t s = i;
            bool skip = false;
            for (;;) {
                const int64_t j = s - 1 - lane;
                const uint64_t k = j >= 0 ? key[j] : 0;
                const bool in = j >= 0 && k >> shift == pre;
                const uint64_t kn = in ? key[j + 1] : 0;
                const uint64_t out = __ballot(!in), down = __ballot(in && k > kn);
                const int n_in = out ? __ffsll((unsigned long long)out) - 1 : 64;
                if (down & (n_in == 64 ? ~0ull : (1ull << n_in) - 1)) {
                    skip = true;
                    break;
                }
                s -= n_in;
                if (n_in < 64) break;
            }
            if (skip) continue;
            const int64_t j = s + lane;
            uint64_t k = j < B.m ? key[j] : 0;
            const bool in = j < B.m && k >> shift == pre;
            const uint64_t out = __ballot(!in);
            const bool more = out == 0 && s + 64 < B.m && key[s + 64] >> shift == pre;
            // every lane takes part in the claim (all but lane 0 with no bit),
            // so that its result is not read across a divergent branch
            const uint32_t bit = 1u << (s & 31);
            const uint32_t was = atomicOr(&B.claim[s >> 5], lane == 0 ? bit : 0u);
            const bool mine = (__builtin_amdgcn_readfirstlane((int)was) & (int)bit) == 0;
            const int len = !mine || more ? 0 : out ? __ffsll((unsigned long long)out) - 1 : 64;
            const int32_t v = lane < len ? id[j] : 0;
            int rank = 0;
            for (int u = 0; u < len; u++) {
                const uint64_t ku = dpp::readlane64(k, u);
                rank += (ku < k || (ku == k && u < lane)) ? 1 : 0;
            }
            if (lane < len) {
                key[s + rank] = k;
                id[s + rank] = v;
            }
            if (mine && more && lane == 0) B.long_runs[atomicAdd(B.n_long, 1u)] = (uint32_t)s;
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
    }
}

// A run of more than 64 equal prefixes: one workgroup sorts it by the digits
// below the prefix, back and forth between the outputs and the temporaries
// of the same positions (digits with one value are skipped).
__global__ __launch_bounds__(kThreads) void k_sort_fix_long(SortBufs B)
{
    __shared__ uint32_t s_base[kRadix];
    __shared__ uint32_t s_cnt[kWaves][kRadix];
    __shared__ uint32_t s_wsum[kRadix / 64];
    __shared__ unsigned long long s_end;
    const uint32_t low = B.plan->low, runs = *B.n_long;
    const int shift = 8 * (int)low;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = lane == 0 ? 0ull : ~0ull >> (64 - lane);
    for (uint32_t r = blockIdx.x; r < runs; r += gridDim.x) {
        const int64_t s = B.long_runs[r];
        const uint64_t pre = B.ok[s] >> shift;
        int64_t e = s;
        for (;;) {
            if (tid == 0) s_end = kThreads;
            __syncthreads();
            const int64_t j = e + tid;
            const bool in = j < B.m && B.ok[j] >> shift == pre;
            const uint64_t out = __ballot(!in);
            if (lane == 0 && out)
                atomicMin(&s_end, (unsigned long long)(wave * 64 + __ffsll((unsigned long long)out) - 1));
            __syncthreads();
            const int n_in = (int)s_end;
            __syncthreads();
            e += n_in;
            if (n_in < kThreads) break;
        }
        const int64_t len = e - s;
        bool in_tmp = false;
        for (uint32_t d = 0; d < low; d++) {
            const uint64_t *ik = in_tmp ? B.tk + s : B.ok + s;
            const int32_t *ii = in_tmp ? B.ti + s : B.oi + s;
            uint64_t *pk = in_tmp ? B.ok + s : B.tk + s;
            int32_t *pi = in_tmp ? B.oi + s : B.ti + s;
            if (tid < kRadix) s_base[tid] = 0;
            __syncthreads();
            for (int64_t j = tid; j < len; j += kThreads)
                atomicAdd(&s_base[(uint32_t)(ik[j] >> (8 * d)) & 0xffu], 1u);
            __syncthreads();
            uint32_t c = 0, incl = 0;
            bool single = false;
            if (tid < kRadix) {
                c = s_base[tid];
                single = (int64_t)c == len;
                incl = (uint32_t)wave_incl_scan32((int)c);
                if (lane == 63) s_wsum[wave] = incl;
            }
            if (__syncthreads_or(single)) continue;
            if (tid < kRadix) {
                uint32_t at = incl - c;
                for (int w = 0; w < wave; w++) at += s_wsum[w];
                s_base[tid] = at;
            }
            for (int i = tid; i < kWaves * kRadix; i += kThreads) (&s_cnt[0][0])[i] = 0;
            __syncthreads();
            for (int64_t j0 = 0; j0 < len; j0 += kThreads) {
                const int64_t j = j0 + tid;
                const bool valid = j < len;
                const uint64_t k = valid ? ik[j] : 0;
                const int32_t v = valid ? ii[j] : 0;
                const uint32_t dg = (uint32_t)(k >> (8 * d)) & 0xffu;
                const uint64_t eq = same_digit(dg, __ballot(valid));
                const uint32_t before = (uint32_t)__popcll(eq & lt);
                if (valid && before == 0) s_cnt[wave][dg] = (uint32_t)__popcll(eq);
                __syncthreads();
                if (valid) {
                    uint32_t at = s_base[dg] + before;
                    for (int w = 0; w < wave; w++) at += s_cnt[w][dg];
                    pk[at] = k;
                    pi[at] = v;
                }
                __syncthreads();
                if (tid < kRadix) {
                    uint32_t sum = 0;
                    for (int w = 0; w < kWaves; w++) {
                        sum += s_cnt[w][tid];
                        s_cnt[w][tid] = 0;
                    }
                    s_base[tid] += sum;
                }
                __syncthreads();
            }
            in_tmp = !in_tmp;
        }
        if (in_tmp) {
            for (int64_t j = tid; j < len; j += kThreads) {
                B.ok[s + j] = B.tk[s + j];
                B.oi[s + j] = B.ti[s + j];
            }
        }
        __syncthreads();
    }
}

int64_t tile_of(int64_t m) { return kThreads * (m >= kBigFrom ? kItemsBig : kItemsSmall); }

}  // namespace

size_t index_workspace_bytes(int64_t m)
{
    const int64_t tiles = (m + tile_of(m) - 1) / tile_of(m);
    size_t bytes = 0;
    // counts, tickets, number of long runs; published counts; claims
    bytes += align_up((kDigits * kRadix + 64) * sizeof(uint32_t), 256);
    bytes += align_up((size_t)tiles * kRadix * sizeof(unsigned long long), 256);
    bytes += align_up((size_t)(m / 32 + 1) * sizeof(uint32_t), 256);
    bytes += align_up(sizeof(SortPlan), 256);
    bytes += align_up((size_t)(m / 64 + 1) * sizeof(uint32_t), 256);
    bytes += align_up((size_t)m * sizeof(uint64_t), 256);
    bytes += align_up((size_t)m * sizeof(int32_t), 256);
    return bytes + 256;
}

polymh_status launch_index_build(const uint64_t *keys, int64_t n, int32_t b, void *ws,
                                 size_t ws_bytes, uint64_t *sorted_keys, int32_t *sorted_ids,
                                 hipStream_t s)
{
    const int64_t m = n * b;
    if (m == 0) return POLYMH_OK;
    if (m > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "index_build: more than 2^31-1 entries");
    const int64_t tile = tile_of(m), tiles = (m + tile - 1) / tile;
    Carve cv{static_cast<char *>(ws), ws_bytes};
    SortBufs B{};
    B.keys = keys;
    B.ok = sorted_keys;
    B.oi = sorted_ids;
    B.m = m;
    B.tiles = (uint32_t)tiles;
    // the first three are cleared together
    B.hist = cv.take<uint32_t>(kDigits * kRadix + 64);
    B.desc = cv.take<unsigned long long>((size_t)tiles * kRadix);
    B.claim = cv.take<uint32_t>((size_t)(m / 32 + 1));
    const size_t cleared = align_up(cv.used, 256);
    B.plan = cv.take<SortPlan>(1);
    B.long_runs = cv.take<uint32_t>((size_t)(m / 64 + 1));
    B.tk = cv.take<uint64_t>((size_t)m);
    B.ti = cv.take<int32_t>((size_t)m);
    if (!cv.ok)
        return set_error(POLYMH_ECAPACITY, "index_build: workspace of %zu bytes, need %zu", ws_bytes, cv.used);
    B.tickets = B.hist + kDigits * kRadix;
    B.n_long = B.tickets + kDigits;
    const auto meets = [&](const void *out, size_t bytes) {
        const char *k = reinterpret_cast<const char *>(keys), *o = static_cast<const char *>(out);
        return k < o + bytes && o < k + (size_t)m * sizeof(*keys);
    };
    const bool in_place = meets(sorted_keys, (size_t)m * sizeof(*sorted_keys)) ||
                          meets(sorted_ids, (size_t)m * sizeof(*sorted_ids));
    const int cus = cu_count();
    auto grid = [](int64_t items, int64_t per, int64_t most) {
        int64_t g = (items + per - 1) / per;
        return dim3((unsigned)(g < 1 ? 1 : g > most ? most : g));
    };
    const int64_t words = (int64_t)(cleared / sizeof(unsigned long long));
    hipLaunchKernelGGL(k_sort_init, grid(words, 1024, 8 * cus), dim3(256), 0, s,
                       reinterpret_cast<unsigned long long *>(B.hist), words);
    hipLaunchKernelGGL(k_sort_hist, grid(m, kThreads * 4, 4 * cus), dim3(kThreads), 0, s, B);
    hipLaunchKernelGGL(k_sort_plan, dim3(1), dim3(kThreads), 0, s, B, in_place ? 1 : 0);
    for (int d = 0; d < kDigits; d++) {
        if (m >= kBigFrom)
            hipLaunchKernelGGL(k_sort_pass<kItemsBig>, grid(tiles, 1, 2 * cus), dim3(kThreads), 0, s, B, d);
        else
            hipLaunchKernelGGL(k_sort_pass<kItemsSmall>, grid(tiles, 1, 2 * cus), dim3(kThreads), 0, s, B, d);
    }
    hipLaunchKernelGGL(k_sort_fix, grid(m, kFixThreads * kFixItems, 8 * cus), dim3(kFixThreads), 0, s, B);
    hipLaunchKernelGGL(k_sort_fix_long, dim3((unsigned)cus), dim3(kThreads), 0, s, B);
    return check_launch("index_build");
}

}  // namespace polymh
