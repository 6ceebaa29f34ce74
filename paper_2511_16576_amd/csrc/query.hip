// Candidate generation (Sec. 3.2: a query's candidates are the polygons in
// its buckets).  Each (query, band) key is looked up in the sorted bucket
// table; a query's candidate list is the ids of the bucket entries that
// belong to the same band, in ascending order without repeats.  Where a
// query's bitmap of the data set fits LDS and the queries run at once, its
// entries mark it there (k_mark_row).  Else a query's same-band bucket
// entries are gathered into its own bitmap row in memory (work in proportion
// to its entries), then sorted and kept without repeats on chip (one wavefront
// for up to kSparseCap entries, where rows do not fit LDS a block for up to
// kBigCap); a query with more entries marks its polygons in its row.  Every
// way gives the same list.
#include "internal.hpp"

#include <algorithm>
#include <mutex>

namespace polymh {

namespace {

constexpr int kSparseCap = 4096;

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
}

// First index in a[0, n) whose value is >= key.  Band keys are SplitMix64
// outputs, uniform over 64 bits, so a probe placed by linear interpolation
// between the bracket's end values lands near the answer (about log log n
// probes): the first five probes interpolate, then interpolation
// alternates with bisection, which bounds the probes by about 5 + 2 log2 n
// on any key set (long runs of equal keys included).  On 2^25 uniform keys
// the probes average 5.4, against 8.9 when alternating from the first.
__device__ __forceinline__ int64_t lower_bound_interp(const uint64_t *__restrict__ a, int64_t n, uint64_t key)
{
    int64_t lo = 0, hi = n;                 // answer in [lo, hi]
    uint64_t klo = 0, khi = ~0ull;          // a[lo - 1] < key <= a[hi] (or the ends of the key range)
    int step = 0;
    while (lo < hi) {
        int64_t p = (lo + hi) >> 1;
        const bool interp = step < 5 || (step & 1);
        if (interp && khi > klo) {
            const double f = (double)(key - klo) / (double)(khi - klo);
            const int64_t g = lo + (int64_t)(f * (double)(hi - lo));
            p = g < lo ? lo : (g >= hi ? hi - 1 : g);
        }
        step++;
        const uint64_t v = a[p];
        if (v < key) {
            lo = p + 1;
            klo = v;
        } else {
            hi = p;
            khi = v;
        }
    }
    return lo;
}

// One past the last entry of key's bucket, whose first one is at lo (lo if it
// has none), by a galloping search: probes 1, 2, 4, ... entries on, then a
// binary search between the last two.  (Eight probes at a time were slower:
// 284 against 253 us for 10,000 queries of 100,000 polygons, and 34 against
// 32 for ten.)
__device__ __forceinline__ int64_t bucket_end(const uint64_t *__restrict__ skeys, int64_t n_entries, uint64_t key,
                                              int64_t lo)
{
    if (lo >= n_entries || skeys[lo] != key) return lo;
    int64_t last = lo, step = 1;
    while (lo + step < n_entries && skeys[lo + step] == key) {
        last = lo + step;
        step <<= 1;
    }
    int64_t a = last + 1, c = lo + step < n_entries ? lo + step : n_entries;
    while (a < c) {
        const int64_t mid = (a + c) >> 1;
        if (skeys[mid] == key) a = mid + 1;
        else c = mid;
    }
    return a;
}

// A key's bucket by 16 lanes (a DPP row) that all have the key.  A round reads
// 16 keys about the interpolated place, the square root of the bracket's
// length apart up to a quarter (a uniform key lies within half of it, about),
// so that some 3 rounds of memory latency find the place instead of the 8
// probes the last of a wavefront's lanes needs; from the fifth round on the
// bracket is cut into 17 equal parts, which bounds them.  Lanes of other rows
// may be done.
struct Bucket {
    int64_t lo, hi;
};
__device__ __forceinline__ Bucket bucket_by_row(const uint64_t *__restrict__ a, int64_t n, uint64_t key, int l16,
                                                int row_shift)
{
    int64_t lo = 0, hi = n;                 // answer in [lo, hi]
    uint64_t klo = 0, khi = ~0ull;
    for (int round = 0; lo < hi; round++) {
        const int64_t len = hi - lo;
        const double f = khi > klo ? (double)(key - klo) / (double)(khi - klo) : 0.5;
        const int64_t d = max((int64_t)1, (int64_t)(0.25f * sqrtf((float)len)));
        const int64_t about = lo + (int64_t)(f * (double)len) + (l16 - 8) * d, part = lo + (l16 + 1) * len / 17;
        int64_t p = len <= 16 ? lo + l16 : round < 4 ? about : part;
        // lanes past the bracket count as at its last key
        p = p < lo ? lo : (p >= hi ? hi - 1 : p);
        const uint64_t v = a[p];
        const uint32_t below = (uint32_t)(__ballot(v < key) >> row_shift) & 0xffffu;
        const int c = __popc(below);        // the first c lanes' keys are below
        const int from = row_shift + (c > 0 ? c - 1 : 0), to = row_shift + (c < 16 ? c : 15);
        const int64_t pf = __shfl(p, from), pt = __shfl(p, to);
        const uint64_t vf = __shfl(v, from), vt = __shfl(v, to);
        if (c > 0) { lo = pf + 1; klo = vf; }
        if (c < 16) { hi = pt; khi = vt; }
    }
    Bucket r{lo, lo};
    for (;;) {
        const bool in = r.hi + l16 < n && a[r.hi + l16] == key;
        const uint32_t run = (uint32_t)(__ballot(in) >> row_shift) & 0xffffu;
        const int c = __builtin_ctz(~run);  // 16 if all are
        r.hi += c;
        if (c < 16) break;
        if (r.hi - r.lo >= 64) {            // a long bucket: gallop on from here
            r.hi = bucket_end(a, n, key, r.hi);
            break;
        }
    }
    return r;
}

// The candidates of a query as a bitmap row, a workgroup a query: a thread a
// band finds its bucket (kRowTeam: 16 lanes a band), the buckets' entries are
// spread over the threads and mark their polygons, the bits are counted.
// kLds: the row is built in LDS and written out for k_emit, else in place.
// Bound: the latency of the searches' dependent reads.  100,000 polygons, 32 bands, 1,000 queries 53
// us for the whole lookup and 10,000 253, against 85 and 573 with a wavefront a
// (query, band) and the rows cleared, marked and counted in memory.
constexpr int kRowThreads = 256, kRowTeam = 1024;
template <bool kLds, int kThreads>
__device__ __forceinline__ void mark_row(const uint64_t *__restrict__ skeys, const int32_t *__restrict__ sids,
                                         int64_t n_entries, const uint64_t *__restrict__ qkeys, int64_t q, int32_t b,
                                         uint32_t *bitmap, int64_t words, int64_t *__restrict__ counts)
{
    extern __shared__ uint32_t s_row[];
    __shared__ int64_t s_base[kThreads + 1], s_lo[kThreads], s_w[kThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t *row = bitmap + q * words;
    uint32_t *bits = kLds ? s_row : row;
    for (int64_t i = tid; i < words; i += kThreads) bits[i] = 0u;
    for (int32_t t0 = 0; t0 < b; t0 += kThreads) {
        const int32_t t = t0 + tid;
        int64_t lo = 0, hi = 0;
        if constexpr (kThreads == kRowTeam) {
            // few queries: the searches' latency is the launch's
            const int l16 = tid & 15, row_shift = lane & 48, count = min(kThreads, b - t0);
            for (int r = tid >> 4; r < count; r += kThreads / 16) {
                const Bucket k = bucket_by_row(skeys, n_entries, qkeys[q * b + t0 + r], l16, row_shift);
                if (l16 == 0) {
                    s_lo[r] = k.lo;
                    s_base[r] = k.hi - k.lo;
                }
            }
            __syncthreads();
            if (t < b) {
                lo = s_lo[tid];
                hi = lo + s_base[tid];
            }
        } else if (t < b) {
            const uint64_t key = qkeys[q * b + t];
            lo = lower_bound_interp(skeys, n_entries, key);
            hi = bucket_end(skeys, n_entries, key, lo);
        }
        const int64_t incl = wave_incl_scan64(hi - lo);
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int64_t at = incl - (hi - lo);
        for (int w = 0; w < wave; w++) at += s_w[w];
        s_base[tid] = at;
        s_lo[tid] = lo;
        if (tid == kThreads - 1) s_base[kThreads] = at + (hi - lo);
        __syncthreads();
        const int64_t total = s_base[kThreads];
        const int top = min(kThreads, b - t0) - 1;
        constexpr int kU = 4;                   // entries in flight a thread
        for (int64_t j0 = tid; j0 < total; j0 += kThreads * kU) {
            int32_t ent[kU];
            int band[kU];
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int64_t j = j0 + kThreads * u;
                ent[u] = -1;
                band[u] = 0;
                if (j < total) {
                    int l = 0, h = top;         // the last band with s_base[l] <= j
                    while (l < h) {
                        const int mid = (l + h + 1) >> 1;
                        if (s_base[mid] <= j) l = mid;
                        else h = mid - 1;
                    }
                    ent[u] = sids[s_lo[l] + (j - s_base[l])];   // entry p*b + t'
                    band[u] = t0 + l;
                }
            }
#pragma unroll
            for (int u = 0; u < kU; u++) {
                const int32_t id = ent[u] >= 0 ? ent[u] / b : 0;
                if (ent[u] >= 0 && ent[u] - id * b == band[u]) atomicOr(&bits[id >> 5], 1u << (id & 31));
            }
        }
        __syncthreads();
    }
    int64_t c = 0;
    if constexpr (kLds) {
        for (int64_t i = tid; i < words; i += kThreads) {
            const uint32_t v = s_row[i];
            row[i] = v;
            c += __popc(v);
        }
    } else {
        constexpr int kC = 8;                   // words in flight a thread
        for (int64_t i0 = tid; i0 < words; i0 += kThreads * kC) {
            uint32_t v[kC];
#pragma unroll
            for (int u = 0; u < kC; u++) {
                const int64_t i = i0 + kThreads * u;
                v[u] = __hip_atomic_load(&row[i < words ? i : i0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int u = 0; u < kC; u++) c += i0 + kThreads * u < words ? __popc(v[u]) : 0;
        }
    }
    c = wave_sum_i64(c);
    if (lane == 0) s_w[wave] = c;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kThreads / 64; w++) c += s_w[w];
        counts[q] = c;
    }
}

// Every query, a workgroup each, with rows in LDS.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_mark_row(const uint64_t *__restrict__ skeys,
                                                          const int32_t *__restrict__ sids, int64_t n_entries,
                                                          const uint64_t *__restrict__ qkeys, int32_t b,
                                                          uint32_t *bitmap, int64_t words,
                                                          int64_t *__restrict__ counts)
{
    mark_row<true, kThreads>(skeys, sids, n_entries, qkeys, blockIdx.x, b, bitmap, words, counts);
}

// The queries that the sparse passes left (dense), taken in turn (a kernel of
// its own: as one, the loop's registers cost the other a tenth).
template <bool kLds, int kThreads>
__global__ __launch_bounds__(kThreads) void k_mark_dense(const uint64_t *__restrict__ skeys,
                                                         const int32_t *__restrict__ sids, int64_t n_entries,
                                                         const uint64_t *__restrict__ qkeys, int64_t nq, int32_t b,
                                                         uint32_t *bitmap, int64_t words,
                                                         int64_t *__restrict__ counts,
                                                         const int32_t *__restrict__ dense)
{
    for (int64_t q = blockIdx.x; q < nq; q += gridDim.x) {
        if (!dense[q]) continue;
        mark_row<kLds, kThreads>(skeys, sids, n_entries, qkeys, q, b, bitmap, words, counts);
        __syncthreads();
    }
}

// Sorts L[0, cnt) in place (bitonic, padded with INT32_MAX to a power of
// two of at most kSparseCap) and keeps each value once; returns the new
// length.  One wavefront.
__device__ int sort_unique(int32_t *L, int cnt, int lane)
{
    int P = 64;
    while (P < cnt) P <<= 1;
    for (int i = cnt + lane; i < P; i += 64) L[i] = INT32_MAX;
    wave_lds_fence();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = lane; i < P; i += 64) {
                const int x = i ^ j;
                if (x > i) {
                    const int32_t a = L[i], c = L[x];
                    if ((a > c) == ((i & k) == 0)) { L[i] = c; L[x] = a; }
                }
            }
            wave_lds_fence();
        }
    }
    // in place: a chunk's values are read before any of its writes, and
    // writes land at or below the positions already read
    int u = 0;
    for (int i0 = 0; i0 < cnt; i0 += 64) {
        const int i = i0 + lane;
        const bool live = i < cnt;
        const int32_t v = live ? L[i] : 0;
        const bool first = live && (i == 0 || L[i - 1] != v);
        wave_lds_fence();
        const uint64_t fm = __ballot(first);
        if (first) {
            const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fm >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)fm, 0u));
            L[u + r] = v;
        }
        u += __popcll(fm);
        wave_lds_fence();
    }
    return u;
}

// Bitonic sort of 64 R values held R to a lane (element i = R lane + r, a
// blocked layout), ascending, in registers: steps within a lane swap
// registers, steps across lanes exchange with __shfl_xor.  R is 16 or 32.
template <int R>
__device__ __forceinline__ void sort_regs(int32_t (&v)[R], int lane)
{
#pragma unroll
    for (int k = 2; k <= 64 * R; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= R) {
                const int lj = j / R;                   // partner lane offset
                const bool lower = (lane & lj) == 0;
#pragma unroll
                for (int r = 0; r < R; r++) {
                    const bool up = ((R * lane + r) & k) == 0;
                    const int32_t o = __shfl_xor(v[r], lj, 64);
                    const int32_t lo = min(v[r], o), hi = max(v[r], o);
                    v[r] = (lower == up) ? lo : hi;
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; r++) {
                    if ((r & j) == 0) {
                        const bool up = ((R * lane + r) & k) == 0;
                        const int32_t a = v[r], b = v[r | j];
                        const int32_t lo = min(a, b), hi = max(a, b);
                        v[r] = up ? lo : hi;
                        v[r | j] = up ? hi : lo;
                    }
                }
            }
        }
    }
}

constexpr int kBigCap = 16384;

// Gather pass, one wavefront per query (four per block): the query's
// same-band bucket entries, in bucket order with repeats, written to the
// start of its own bitmap row; raw[q] = their number.  A query with more
// than `cap` entries in its buckets gets dense[q] = 1 (the bitmap takes it).
//
// Lane t takes band t's key: an interpolation search gives its bucket's
// first entry, a galloping search its end.  The bucket lengths' prefix
// sum then spreads every entry of the 64 buckets over the lanes, 64 entries
// a step with independent loads, so the walk takes (entries / 64) steps
// instead of as many as the longest bucket holds.
__global__ __launch_bounds__(256) void k_sparse(const uint64_t *__restrict__ skeys,
                                                const int32_t *__restrict__ sids, int64_t n_entries,
                                                const uint64_t *__restrict__ qkeys, int64_t nq, int32_t b,
                                                int32_t *__restrict__ dense, int64_t *__restrict__ raw,
                                                uint32_t *__restrict__ bitmap, int64_t words, int cap)
{
    __shared__ int32_t sbase[4][65];     // exclusive prefix of the bucket lengths, then the total
    __shared__ int64_t slo[4][64];       // each lane's bucket start
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nq) return;                       // wavefront-uniform; no block barriers below
    int32_t *row = reinterpret_cast<int32_t *>(bitmap + q * words);
    int32_t *base = sbase[wave];
    int64_t *los = slo[wave];
    int cnt = 0;
    bool over = false;
    for (int32_t t0 = 0; t0 < b && !over; t0 += 64) {
        const int32_t t = t0 + lane;
        const bool live = t < b && n_entries > 0;
        const uint64_t key = live ? qkeys[q * b + t] : 0ull;
        int64_t lo = 0, hi = 0;
        if (live) {
            lo = lower_bound_interp(skeys, n_entries, key);
            hi = bucket_end(skeys, n_entries, key, lo);
        }
        // a bucket longer than the list sends the query to the bitmap (which
        // is exact in every case)
        const int64_t len64 = hi - lo;
        if (__ballot(len64 > cap) != 0) {
            over = true;
            break;
        }
        const int len = (int)len64;
        // inclusive scan over the wavefront (64 x 16384 fits an int)
        int inc = len;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(inc, o, 64);
            if (lane >= o) inc += v;
        }
        base[lane] = inc - len;
        los[lane] = lo;
        const int total = __shfl(inc, 63, 64);
        if (cnt + total > cap) {               // wavefront-uniform
            over = true;
            break;
        }
        if (lane == 63) base[64] = total;
        wave_lds_fence();
        // every entry of the 64 buckets, one per lane per step (band lane
        // tl of entry j is the last with base[tl] <= j); the entries of
        // kWalk steps are loaded before any is used, so the walk costs
        // total / (64 kWalk) round trips to memory
        constexpr int kWalk = 8;
        for (int j00 = 0; j00 < total; j00 += 64 * kWalk) {
            int32_t ent[kWalk];
            int band[kWalk];
#pragma unroll
            for (int u = 0; u < kWalk; u++) {
                const int j = j00 + 64 * u + lane;
                ent[u] = -1;
                band[u] = 0;
                if (j < total) {
                    int l = 0, h = 63;         // base[l] <= j < base[h + 1]
                    while (l < h) {
                        const int mid = (l + h + 1) >> 1;
                        if (base[mid] <= j) l = mid;
                        else h = mid - 1;
                    }
                    ent[u] = sids[los[l] + (j - base[l])];   // entry p*b + t'
                    band[u] = t0 + l;
                }
            }
#pragma unroll
            for (int u = 0; u < kWalk; u++) {
                const int32_t id = ent[u] >= 0 ? ent[u] / b : 0;
                const bool ok = ent[u] >= 0 && ent[u] - id * b == band[u];
                const uint64_t om = __ballot(ok);
                const int n_new = __popcll(om);
                const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(om >> 32),
                                                                __builtin_amdgcn_mbcnt_lo((uint32_t)om, 0u));
                if (ok) row[cnt + rank] = id;
                cnt += n_new;
            }
        }
        wave_lds_fence();                      // base/los are rewritten by the next band chunk
    }
    if (lane == 0) {
        dense[q] = over ? 1 : 0;
        raw[q] = over ? 0 : cnt;
    }
}

// Multiplicative hash of a polygon id to a slot of a 2^bits table.
__device__ __forceinline__ int id_slot(int32_t id, int bits)
{
    return (int)(((uint32_t)id * 2654435761u) >> (32 - bits));
}

// Inserts v into an open-addressing set T of 2^bits slots (-1 = empty) by
// linear probing; returns true if v was not there yet.  Needs an empty slot.
__device__ __forceinline__ bool set_insert(int32_t *T, int bits, int32_t v)
{
    int h = id_slot(v, bits);
    const int mask = (1 << bits) - 1;
    for (;;) {
        const int32_t old = atomicCAS(&T[h], -1, v);
        if (old == -1) return true;
        if (old == v) return false;
        h = (h + 1) & mask;
    }
}

constexpr int kSetBits = 12;                 // wavefront pass: 4096 slots
constexpr int kSetMax = 3072;                // ... filled to at most 3/4
constexpr int kBigSetBits = 14;              // block pass: 16384 slots
constexpr int kBigSetMax = 12288;
static_assert((1 << kSetBits) == kSparseCap && (1 << kBigSetBits) == kBigCap, "set sizes");

// Sort pass for short lists, one wavefront per query (four per block): a
// query's raw list of at most kSparseCap entries, read from its row 64 at a
// time, goes into an LDS hash set (each polygon once); the set's members
// are moved to its front, sorted (bitonic) and written back; counts[q] =
// the list's length.  A list with more than kSetMax distinct polygons is
// sorted whole instead (its repeats dropped after the sort).
__global__ __launch_bounds__(256) void k_sparse_sort(const int32_t *__restrict__ dense, int64_t nq,
                                                     int64_t *__restrict__ counts, uint32_t *__restrict__ bitmap,
                                                     int64_t words)
{
    __shared__ int32_t lists[4][kSparseCap];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nq || dense[q]) return;           // wavefront-uniform
    const int cnt = (int)counts[q];            // the raw count of the gather pass
    if (cnt > kSparseCap) return;              // the block pass takes it
    int32_t *T = lists[wave];
    int32_t *row = reinterpret_cast<int32_t *>(bitmap + q * words);
    for (int i = lane; i < kSparseCap; i += 64) T[i] = -1;
    wave_lds_fence();
    int uniq = 0;
    bool whole = false;
    // eight of a lane's entries are loaded together, then inserted
    for (int i0 = 0; i0 < cnt && !whole; i0 += 8 * 64) {
        int32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int i = i0 + 64 * u + lane;
            v[u] = i < cnt ? row[i] : -1;
        }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            if (uniq + 64 > kSetMax) {         // wavefront-uniform: keep the set below 3/4 full
                whole = true;
                break;
            }
            const bool fresh = v[u] >= 0 && set_insert(T, kSetBits, v[u]);
            uniq += __popcll(__ballot(fresh));
        }
    }
    wave_lds_fence();
    int u;
    if (whole) {
        for (int i = lane; i < cnt; i += 64) T[i] = row[i];
        wave_lds_fence();
        u = sort_unique(T, cnt, lane);
    } else {
        // members to the front, in place (a chunk reads before it writes,
        // and writes land at or below what it read)
        int m = 0;
        for (int i0 = 0; i0 < kSparseCap; i0 += 64) {
            const int32_t v = T[i0 + lane];
            const bool keep = v != -1;
            wave_lds_fence();
            const uint64_t km = __ballot(keep);
            if (keep) {
                const int r = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(km >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
                T[m + r] = v;
            }
            m += __popcll(km);
            wave_lds_fence();
        }
        // the members are distinct: sorted in registers when they fit
        // (1,024 or 2,048 of them), else in LDS
        if (m <= 1024) {
            int32_t v[16];
#pragma unroll
            for (int r = 0; r < 16; r++) v[r] = 16 * lane + r < m ? T[16 * lane + r] : INT32_MAX;
            sort_regs<16>(v, lane);
#pragma unroll
            for (int r = 0; r < 16; r++)
                if (16 * lane + r < m) row[16 * lane + r] = v[r];
            if (lane == 0) counts[q] = m;
            return;
        }
        if (m <= 2048) {
            int32_t v[32];
#pragma unroll
            for (int r = 0; r < 32; r++) v[r] = 32 * lane + r < m ? T[32 * lane + r] : INT32_MAX;
            sort_regs<32>(v, lane);
#pragma unroll
            for (int r = 0; r < 32; r++)
                if (32 * lane + r < m) row[32 * lane + r] = v[r];
            if (lane == 0) counts[q] = m;
            return;
        }
        u = sort_unique(T, m, lane);
    }
    for (int i = lane; i < u; i += 64) row[i] = T[i];
    if (lane == 0) counts[q] = u;
}

// Bitonic sort of 4096 values over a 1024-thread block, thread t holding
// positions 4t .. 4t + 3: partners in the same thread are swapped in
// registers, partners in the same wavefront exchanged by shuffles, and the
// ten steps whose partners sit in another wavefront go through L (a write,
// a barrier, a read, a barrier).
__device__ void sort_block4096(int32_t (&v)[4], int32_t *L, int tid)
{
    const int lane = tid & 63;
    for (int k = 2; k <= 4096; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            if (j >= 256) {
#pragma unroll
                for (int r = 0; r < 4; r++) L[4 * tid + r] = v[r];
                __syncthreads();
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int i = 4 * tid + r;
                    const int32_t o = L[i ^ j];
                    const bool keep_min = ((i & j) == 0) == ((i & k) == 0);
                    v[r] = keep_min ? min(v[r], o) : max(v[r], o);
                }
                __syncthreads();
            } else if (j >= 4) {
                const int lj = j >> 2;
                const bool lower = (lane & lj) == 0;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const bool up = ((4 * tid + r) & k) == 0;
                    const int32_t o = __shfl_xor(v[r], lj, 64);
                    v[r] = (lower == up) ? min(v[r], o) : max(v[r], o);
                }
            } else {
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    if ((r & j) == 0) {
                        const bool up = ((4 * tid + r) & k) == 0;
                        const int32_t x = v[r], y = v[r | j];
                        v[r] = up ? min(x, y) : max(x, y);
                        v[r | j] = up ? max(x, y) : min(x, y);
                    }
                }
            }
        }
    }
}

// Block-wide exclusive prefix of one int per thread (1024 threads); *total
// gets the sum.  sw holds 16 ints.
__device__ __forceinline__ int block_excl_scan1024(int x, int *sw, int tid, int *total)
{
    const int lane = tid & 63, wave = tid >> 6;
    const int incl = wave_incl_scan32(x);
    if (lane == 63) sw[wave] = incl;
    __syncthreads();
    int pre = incl - x, tot = 0;
#pragma unroll
    for (int w = 0; w < 16; w++) {
        const int y = sw[w];
        pre += w < wave ? y : 0;
        tot += y;
    }
    *total = tot;
    return pre;
}

// Sort pass for long lists, one block of 1024 threads per query with more
// than kSparseCap raw entries (at most kBigCap): the raw list is loaded
// whole (16 entries a thread, all in flight together), inserted into an LDS
// hash set of 16384 slots (each polygon once), the set's members moved to
// the front (a block-wide scan places them) and sorted: up to 4096 of them
// in registers, more in LDS.  More than kBigSetMax distinct polygons: the
// raw list is sorted whole in LDS and its repeats dropped.
__global__ __launch_bounds__(1024) void k_sparse_sort_big(const int32_t *__restrict__ dense,
                                                          int64_t *__restrict__ counts,
                                                          uint32_t *__restrict__ bitmap, int64_t words)
{
    __shared__ int32_t L[kBigCap];
    __shared__ int sw[16];
    __shared__ int s_uniq;
    const int64_t q = blockIdx.x;
    if (dense[q]) return;
    const int cnt = (int)counts[q];
    if (cnt <= kSparseCap) return;             // the wavefront pass took it
    const int tid = threadIdx.x, lane = tid & 63;
    int32_t *row = reinterpret_cast<int32_t *>(bitmap + q * words);
    int32_t raw[kBigCap / 1024];
#pragma unroll
    for (int u = 0; u < kBigCap / 1024; u++) {
        const int i = u * 1024 + tid;
        raw[u] = i < cnt ? row[i] : -1;
    }
    for (int i = tid; i < kBigCap; i += 1024) L[i] = -1;
    if (tid == 0) s_uniq = 0;
    __syncthreads();
    bool whole = false;
#pragma unroll
    for (int u = 0; u < kBigCap / 1024; u++) {
        if (u * 1024 >= cnt) break;             // block-uniform
        if (s_uniq + 1024 > kBigSetMax) {     // block-uniform (read after a barrier)
            whole = true;
            break;
        }
        const bool fresh = raw[u] >= 0 && set_insert(L, kBigSetBits, raw[u]);
        const int nf = __popcll(__ballot(fresh));
        if (lane == 0 && nf) atomicAdd(&s_uniq, nf);
        __syncthreads();
    }
    __syncthreads();
    int n;                                      // entries to sort at the front of L
    if (whole) {
        for (int i = tid; i < cnt; i += 1024) L[i] = row[i];
        n = cnt;
    } else {
        // members to the front: thread tid owns slots [16 tid, 16 tid + 16)
        int32_t v[16];
        int mine = 0;
#pragma unroll
        for (int k = 0; k < 16; k++) {
            v[k] = L[16 * tid + k];
            mine += v[k] != -1;
        }
        int at = block_excl_scan1024(mine, sw, tid, &n);
        __syncthreads();                        // every slot read before any is rewritten
#pragma unroll
        for (int k = 0; k < 16; k++)
            if (v[k] != -1) L[at++] = v[k];
        __syncthreads();
        if (n <= 4096) {
            // distinct ids: sorted in registers and written out as they are
            int32_t w[4];
#pragma unroll
            for (int r = 0; r < 4; r++) w[r] = 4 * tid + r < n ? L[4 * tid + r] : INT32_MAX;
            __syncthreads();                    // L is reused by the sort's cross-wavefront steps
            sort_block4096(w, L, tid);
#pragma unroll
            for (int r = 0; r < 4; r++)
                if (4 * tid + r < n) row[4 * tid + r] = w[r];
            if (tid == 0) counts[q] = n;
            return;
        }
    }
    int P = 1;
    while (P < n) P <<= 1;
    for (int i = n + tid; i < P; i += 1024) L[i] = INT32_MAX;
    __syncthreads();
    for (int k = 2; k <= P; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < P; i += 1024) {
                const int x = i ^ j;
                if (x > i) {
                    const int32_t a = L[i], c = L[x];
                    if ((a > c) == ((i & k) == 0)) { L[i] = c; L[x] = a; }
                }
            }
            __syncthreads();
        }
    }
    // thread tid owns positions [tid * per, (tid + 1) * per); the first of
    // each run of equal values is kept
    const int per = (n + 1023) / 1024;
    const int i0 = tid * per, i1 = min(n, i0 + per);
    int mine = 0;
    for (int i = i0; i < i1; i++) mine += (i == 0 || L[i - 1] != L[i]) ? 1 : 0;
    int total;
    int u = block_excl_scan1024(mine, sw, tid, &total);
    for (int i = i0; i < i1; i++)
        if (i == 0 || L[i - 1] != L[i]) row[u++] = L[i];
    if (tid == 0) counts[q] = total;
}

// Exclusive prefix of counts[0..nq) into off[0..nq], single block, in
// tiles of 8192: each thread adds 8 consecutive counts, a wavefront scan of
// those sums and a pass over the 16 wavefront totals place every thread.
// With `overflow` (graph-captured lookups): if the total passes cap, raise
// the flag and empty every query's range so that later stages see none.
__global__ __launch_bounds__(1024) void k_offsets(int64_t *__restrict__ off, int64_t nq, int64_t cap,
                                                  int32_t *__restrict__ overflow)
{
    constexpr int kPer = 8;
    __shared__ int64_t s_w[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t carry = 0;
    for (int64_t t0 = 0; t0 < nq; t0 += 1024 * kPer) {
        const int64_t base = t0 + (int64_t)threadIdx.x * kPer;
        int64_t v[kPer];
        int64_t sum = 0;
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            v[u] = base + u < nq ? off[base + u] : 0;
            sum += v[u];
        }
        const int64_t incl = wave_incl_scan64(sum);
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int64_t pre = carry + incl - sum, tot = 0;
#pragma unroll
        for (int w = 0; w < 16; w++) {
            const int64_t x = s_w[w];
            pre += w < wave ? x : 0;
            tot += x;
        }
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            if (base + u < nq) off[base + u] = pre;
            pre += v[u];
        }
        carry += tot;
        __syncthreads();
    }
    const bool over = overflow && carry > cap;
    if (over)
        for (int64_t q = threadIdx.x; q < nq; q += 1024) off[q] = 0;
    if (threadIdx.x == 0) {
        off[nq] = over ? 0 : carry;
        if (overflow) overflow[0] = over ? 1 : 0;
    }
}

// One block per query: its list to off[q] (nothing when the capacity flag is
// raised), copied from its row if the sparse passes took it, else (dense
// null: every query) the row's set bits in ascending order.  The row is read in tiles of 4096 words, 16 consecutive words a thread: one
// block-wide scan of the threads' bit counts per tile places every thread's
// output.
__global__ __launch_bounds__(256) void k_emit(const uint32_t *__restrict__ bitmap, int64_t words,
                                              const int64_t *__restrict__ off,
                                              int32_t *__restrict__ ids, const int32_t *__restrict__ dense,
                                              const int32_t *__restrict__ overflow)
{
    constexpr int kPer = 16;
    __shared__ int32_t s_w[4];
    const int64_t q = blockIdx.x;
    if (overflow && overflow[0]) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t *row = bitmap + q * words;
    int64_t base = off[q];
    if (dense && !dense[q]) {
        const int64_t n = off[q + 1] - base;
        for (int64_t i = threadIdx.x; i < n; i += blockDim.x) ids[base + i] = (int32_t)row[i];
        return;
    }
    for (int64_t w0 = 0; w0 < words; w0 += 256 * kPer) {
        const int64_t w = w0 + (int64_t)threadIdx.x * kPer;
        uint32_t bits[kPer];
        int32_t c = 0;
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            bits[i] = w + i < words ? row[w + i] : 0u;
            c += __popc(bits[i]);
        }
        const int32_t incl = wave_incl_scan32(c);
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        int64_t pos = base + incl - c;
#pragma unroll
        for (int v = 0; v < 4; v++) {
            pos += v < wave ? s_w[v] : 0;
            base += s_w[v];
        }
#pragma unroll
        for (int i = 0; i < kPer; i++) {
            uint32_t v = bits[i];
            while (v) {
                const int bit = __builtin_ctz(v);
                ids[pos++] = (int32_t)((w + i) * 32 + bit);
                v &= v - 1;
            }
        }
        __syncthreads();
    }
}

// Workspace: dense flags [nq], counts [nq], bitmap rows [nq][words].
struct QueryWs {
    int32_t *dense;
    int64_t *counts;
    uint32_t *bitmap;
};

QueryWs carve_query(Carve &cv, int64_t nq, int64_t words)
{
    QueryWs w{};
    w.dense = cv.take<int32_t>((size_t)nq);
    w.counts = cv.take<int64_t>((size_t)nq);
    w.bitmap = cv.take<uint32_t>((size_t)(nq * words));
    return w;
}

// A query's bitmap fits LDS while the data set has up to 32 kRowMost polygons.
// Building it there (one launch) is the faster way as long as the queries run
// at once or the rows are short; else the queries' lists are gathered and
// sorted (three launches, work in proportion to the lists).  Measured, rows
// against lists: 140,000 polygons (4,375 words) and 10,000 queries 244 and 268
// us; 300,000 (9,375 words) 1,000 queries 76 and 76, 2,500 147 and 118;
// 1,000,000 (31,250 words) 200 queries 73 and 92, 1,000 225 and 114.
constexpr int64_t kRowShort = 5120, kRowMost = 32768;
static_assert(kRowShort >= kSparseCap, "a sparse list is kept in its query's bitmap row");
static_assert(kBigCap <= 16384 && kSparseCap <= kBigCap, "list caps");

// Rows of this many words that are on chip at once.
inline int64_t rows_at_once(int64_t words) { return cu_count() * ((int64_t)(160 << 10) / (words * 4 + 6144)); }

inline bool use_row(int64_t nq, int64_t words)
{
    if (words <= kRowShort) return true;
    return words <= kRowMost && nq <= rows_at_once(words);
}

// Lets k_mark_row have rows of any size that use_row gives it.  The setting is
// the device's for the whole process, so it is the largest, made once: with
// each call's own size, threads with data sets of different sizes could launch
// by the other's.
polymh_status allow_rows()
{
    static std::mutex mu;
    static bool done[64] = {false};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return set_error(POLYMH_EDEVICE, "query: no current device");
    std::lock_guard<std::mutex> lk(mu);
    if (done[dev]) return POLYMH_OK;
    for (const void *f : {reinterpret_cast<const void *>(&k_mark_row<kRowTeam>),
                          reinterpret_cast<const void *>(&k_mark_row<kRowThreads>),
                          reinterpret_cast<const void *>(&k_mark_dense<true, kRowTeam>),
                          reinterpret_cast<const void *>(&k_mark_dense<true, kRowThreads>)}) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kRowMost * 4);
        if (e != hipSuccess) return set_error(POLYMH_EDEVICE, "query: rows on chip: %s", hipGetErrorString(e));
    }
    done[dev] = true;
    return POLYMH_OK;
}

// Lengths of every query's list into counts, and what k_emit reads of them into
// the workspace.
polymh_status lookup_counts(const uint64_t *skeys, const int32_t *sids, int64_t n_entries, int64_t words,
                   const uint64_t *qkeys, int64_t nq, int32_t b, const QueryWs &w, int64_t *counts, hipStream_t s)
{
    if (use_row(nq, words)) {
        const bool team = nq <= cu_count();
        if (const polymh_status st = words * 4 > 40 << 10 ? allow_rows() : POLYMH_OK) return st;
        if (team)
            hipLaunchKernelGGL((k_mark_row<kRowTeam>), dim3((unsigned)nq), dim3(kRowTeam), (size_t)words * 4, s,
                               skeys, sids, words > 0 ? n_entries : 0, qkeys, b, w.bitmap, words, counts);
        else
            hipLaunchKernelGGL((k_mark_row<kRowThreads>), dim3((unsigned)nq), dim3(kRowThreads),
                               (size_t)words * 4, s, skeys, sids, words > 0 ? n_entries : 0, qkeys, b, w.bitmap, words,
                               counts);
        return POLYMH_OK;
    }
    // A list is sorted by a block while its row does not fit LDS (4 M polygons,
    // lists of 4,800: 1,000 queries 407 us); else the row costs less (300,000
    // polygons, 3,000 queries with lists of 4,800: 296 us, sorted 968; 1 M
    // polygons 630 and 976).
    const int cap = words > kRowMost ? kBigCap : kSparseCap;
    hipLaunchKernelGGL(k_sparse, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, skeys, sids, n_entries,
                       qkeys, nq, b, w.dense, counts, w.bitmap, words, (int)std::min<int64_t>(words, cap));
    hipLaunchKernelGGL(k_sparse_sort, dim3((unsigned)((nq + 3) / 4)), dim3(256), 0, s, w.dense, nq, counts,
                       w.bitmap, words);
    if (cap > kSparseCap) hipLaunchKernelGGL(k_sparse_sort_big, dim3((unsigned)nq), dim3(1024), 0, s, w.dense, counts, w.bitmap,
                       words);
    // the queries that they left: rows on chip where they fit (as many
    // workgroups as are there at once take them in turn), else in memory
    if (words <= kRowMost) {
        if (const polymh_status st = allow_rows()) return st;
        const int64_t at_once = rows_at_once(words);
        if (at_once <= cu_count())
            hipLaunchKernelGGL((k_mark_dense<true, kRowTeam>), dim3((unsigned)std::min(nq, at_once)), dim3(kRowTeam),
                               (size_t)words * 4, s, skeys, sids, n_entries, qkeys, nq, b, w.bitmap, words, counts,
                               w.dense);
        else
            hipLaunchKernelGGL((k_mark_dense<true, kRowThreads>), dim3((unsigned)std::min(nq, at_once)),
                               dim3(kRowThreads), (size_t)words * 4, s, skeys, sids, n_entries, qkeys, nq, b, w.bitmap,
                               words, counts, w.dense);
    } else if (nq <= 4 * cu_count()) {
        // few workgroups a CU: 4 M polygons, a list of 32,000: 209 us, with 256
        // threads 342
        hipLaunchKernelGGL((k_mark_dense<false, kRowTeam>), dim3((unsigned)nq), dim3(kRowTeam), 0, s, skeys, sids,
                           n_entries, qkeys, nq, b, w.bitmap, words, counts, w.dense);
    } else {
        hipLaunchKernelGGL((k_mark_dense<false, kRowThreads>), dim3((unsigned)nq), dim3(kRowThreads), 0, s, skeys, sids,
                           n_entries, qkeys, nq, b, w.bitmap, words, counts, w.dense);
    }
    return POLYMH_OK;
}

void lookup_emit(int64_t words, int64_t nq, const QueryWs &w, int64_t *off, int32_t *ids, const int32_t *overflow,
                 hipStream_t s)
{
    if (words > 0)
        hipLaunchKernelGGL(k_emit, dim3((unsigned)nq), dim3(256), 0, s, w.bitmap, words, off, ids,
                           use_row(nq, words) ? nullptr : w.dense, overflow);
}

}  // namespace

polymh_status launch_query_capped(const uint64_t *skeys, const int32_t *sids, int64_t n_entries,
                                  int64_t n_data, const uint64_t *qkeys, int64_t nq, int32_t b,
                                  void *ws, size_t ws_bytes, int64_t *cand_off, int32_t *cand_ids,
                                  int64_t cand_cap, int32_t *overflow, hipStream_t s)
{
    const int64_t words = (n_data + 31) / 32;
    Carve cv{static_cast<char *>(ws), ws_bytes};
    const QueryWs w = carve_query(cv, nq, words);
    if (!cv.ok)
        return set_error(POLYMH_ECAPACITY, "query_capped: workspace of %zu bytes, need %zu", ws_bytes, cv.used);
    if (nq > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "query_capped: too many queries");
    if (nq > 0)
        if (const polymh_status st = lookup_counts(skeys, sids, n_entries, words, qkeys, nq, b, w, cand_off, s)) return st;
    hipLaunchKernelGGL(k_offsets, dim3(1), dim3(1024), 0, s, cand_off, nq, cand_cap, overflow);
    if (nq > 0) lookup_emit(words, nq, w, cand_off, cand_ids, overflow, s);
    return check_launch("query_capped");
}

polymh_status launch_offsets(int64_t *off, int64_t nq, hipStream_t s)
{
    hipLaunchKernelGGL(k_offsets, dim3(1), dim3(1024), 0, s, off, nq, (int64_t)0, (int32_t *)nullptr);
    return check_launch("offsets");
}

size_t query_workspace_bytes(int64_t n_data, int64_t nq)
{
    const int64_t words = (n_data + 31) / 32;
    Carve cv{nullptr, 0};
    carve_query(cv, nq, words);
    return align_up(cv.used, 256) + 256;
}

polymh_status launch_query(const uint64_t *skeys, const int32_t *sids, int64_t n_entries,
                           int64_t n_data, const uint64_t *qkeys, int64_t nq, int32_t b, void *ws,
                           size_t ws_bytes, int64_t *cand_off, int32_t *cand_ids, hipStream_t s)
{
    const int64_t words = (n_data + 31) / 32;
    Carve cv{static_cast<char *>(ws), ws_bytes};
    const QueryWs w = carve_query(cv, nq, words);
    if (!cv.ok)
        return set_error(POLYMH_ECAPACITY, "query: workspace of %zu bytes, need %zu", ws_bytes, cv.used);
    if (nq == 0) {
        hipLaunchKernelGGL(k_offsets, dim3(1), dim3(1024), 0, s, cand_off, (int64_t)0, (int64_t)0,
                           (int32_t *)nullptr);
        return check_launch("query");
    }
    if (nq > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "query: too many queries");
    // with offsets from the first phase (the caller's), the lengths go to the
    // workspace
    int64_t *counts = cand_ids ? w.counts : cand_off;
    if (const polymh_status st = lookup_counts(skeys, sids, n_entries, words, qkeys, nq, b, w, counts, s)) return st;
    if (!cand_ids)
        hipLaunchKernelGGL(k_offsets, dim3(1), dim3(1024), 0, s, cand_off, nq, (int64_t)0, (int32_t *)nullptr);
    else
        lookup_emit(words, nq, w, cand_off, cand_ids, nullptr, s);
    return check_launch("query");
}

}  // namespace polymh
