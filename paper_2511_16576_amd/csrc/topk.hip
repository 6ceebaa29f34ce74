// Per-query top-k by (J descending, id ascending): Def. 1's K nearest
// neighbours under the Jaccard distance 1 - J.
//
// One workgroup per query narrows the list to at most `keep` entries that
// hold the top k, by a radix selection on the key (J, id): each step counts a
// digit of up to 11 bits over the entries that share the digits chosen so far
// and goes on in the digit where the k-th best falls.  The entries left are
// ranked by counting, for each, the ones before it.  Bound: the latency of
// the steps, typically two counts, one gather and one ranking whatever k is,
// where selecting one entry a round takes k passes over the list: 64 lists of
// 11,800 at k = 100 take 35 us (1,175 by rounds), 10,000 lists of 650 at
// k = 10 88 us (157 by rounds).  Where a step leaves no entry out, the next one
// starts at the highest bit in which they differ, so that equal J cost one
// count rather than four: 5,000 lists of 3,000 at k = 10 103 us where all J are
// equal and 163 where they take eight values (301 and 292 digit by digit).
#include "internal.hpp"

#include <algorithm>
#include <cfloat>

namespace polymh {

namespace {

constexpr int kBins = 2048;

__device__ __forceinline__ bool better(double ja, int32_t ia, double jb, int32_t ib)
{
    return ja > jb || (ja == jb && ia < ib);
}

// J as an integer that ascends as J descends (finite J, no negative zero).
__device__ __forceinline__ uint64_t key_of(double j)
{
    const uint64_t u = (uint64_t)__double_as_longlong(j);
    return (u >> 63) ? u : ~(u | 1ull << 63);
}
__device__ __forceinline__ double value_of(uint64_t k)
{
    return __longlong_as_double((long long)((k >> 63) ? k : ~k & ~(1ull << 63)));
}

// One selection a round: round r takes the best entry strictly after the
// (r-1)-th in the order.  Infinite J above every finite one and NaN are never
// taken, and an entry given twice is taken once.
__device__ void select_by_rounds(const int32_t *__restrict__ ids, const double *__restrict__ js, int64_t n, int32_t k,
                                 double *s_j, int32_t *s_i, int32_t *__restrict__ top_ids, double *__restrict__ top_j)
{
    double pj = DBL_MAX;
    int32_t pi = -1;
    for (int r = 0; r < k; r++) {
        double bj = -DBL_MAX;
        int32_t bi = -1;
        for (int64_t c = threadIdx.x; c < n; c += blockDim.x) {
            const double j = js[c];
            const int32_t i = ids[c];
            const bool after = j < pj || (j == pj && i > pi);
            if (after && (bi < 0 || better(j, i, bj, bi))) {
                bj = j;
                bi = i;
            }
        }
        s_j[threadIdx.x] = bj;
        s_i[threadIdx.x] = bi;
        __syncthreads();
        for (int o = (int)blockDim.x / 2; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) {
                const double oj = s_j[threadIdx.x + o];
                const int32_t oi = s_i[threadIdx.x + o];
                if (oi >= 0 && (s_i[threadIdx.x] < 0 || better(oj, oi, s_j[threadIdx.x], s_i[threadIdx.x]))) {
                    s_j[threadIdx.x] = oj;
                    s_i[threadIdx.x] = oi;
                }
            }
            __syncthreads();
        }
        pj = s_j[0];
        pi = s_i[0];
        if (threadIdx.x == 0) {
            top_ids[r] = pi;
            top_j[r] = pi >= 0 ? pj : 0.0;
        }
        __syncthreads();
        if (pi < 0) {
            for (int rr = r + 1 + threadIdx.x; rr < k; rr += blockDim.x) {
                top_ids[rr] = -1;
                top_j[rr] = 0.0;
            }
            break;
        }
    }
}

// keep >= 2 k: at most this many entries are ranked.
__global__ __launch_bounds__(1024) void k_topk(const int64_t *__restrict__ off, const int32_t *__restrict__ ids,
                                               const double *__restrict__ js, int32_t k, int32_t keep,
                                               int32_t *__restrict__ top_ids, double *__restrict__ top_j)
{
    extern __shared__ uint64_t s_mem[];
    uint64_t *s_k = s_mem;                                        // [keep]
    int32_t *s_id = reinterpret_cast<int32_t *>(s_mem + keep);    // [keep]
    uint32_t *s_bin = reinterpret_cast<uint32_t *>(s_id + keep);  // [kBins]
    __shared__ uint32_t s_wave[16], s_count, s_digit, s_below, s_in;
    __shared__ int32_t s_id_most;
    __shared__ unsigned long long s_and, s_or;
    const int64_t q = blockIdx.x;
    const int64_t a = off[q], n = off[q + 1] - a;
    ids += a;
    js += a;
    top_ids += q * k;
    top_j += q * k;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;

    bool odd = n > INT32_MAX;
    int shift = 64, id_shift = 32;      // digits chosen so far end here
    uint64_t pre = 0, all_and = ~0ull, all_or = 0;
    uint32_t id_pre = 0, below = 0, left_in = (uint32_t)n;
    int32_t id_most = 0;
    if (tid == 0) {
        s_and = ~0ull;
        s_or = 0;
        s_id_most = 0;
    }
    // bits of J from the top, then bits of the id
    while (n > keep) {
        const bool first_step = shift == 64, on_id = shift == 0;
        if (on_id && id_shift == 32) {
            // the ids' own bits
            id_most = wave_max32(id_most);
            if (lane == 0) atomicMax(&s_id_most, id_most);
            __syncthreads();
            id_shift = 32 - __builtin_clz((uint32_t)s_id_most | 1u);
        }
        if (on_id && id_shift == 0) {   // more than `keep` copies of one entry
            odd = true;
            break;
        }
        const int hi = on_id ? id_shift : shift, lo = hi > 11 ? hi - 11 : 0;
        const uint32_t mask = (1u << (hi - lo)) - 1;
        for (int b = tid; b < kBins; b += nt) s_bin[b] = 0;
        __syncthreads();
        for (int64_t c = tid; c < n; c += nt) {
            const double j = js[c];
            const int32_t id = ids[c];
            const uint64_t key = key_of(j);
            if (first_step) {
                odd |= !(fabs(j) <= DBL_MAX) || key == 1ull << 63 || id < 0;
                id_most = max(id_most, id);
            }
            const bool in = on_id ? key == pre && (uint32_t)id >> id_shift == id_pre : first_step || key >> shift == pre;
            if (!on_id && in) {
                all_and &= key;
                all_or |= key;
            }
            // the lanes that share the first one's digit are counted together
            // (many J are 0), the others one by one: 5,000 lists of 500 zeros
            // at k = 100 129 us, 183 with every lane on its own; three turns
            // of it cost random J more than they give
            const uint32_t d = (uint32_t)((on_id ? (uint64_t)(uint32_t)id : key) >> lo) & mask;
            uint64_t left = __ballot(in);
            if (left != 0) {
                const int first = __builtin_ctzll(left);
                const uint64_t same = left & __ballot(d == (uint32_t)__builtin_amdgcn_readlane((int)d, first));
                if (lane == first) atomicAdd(&s_bin[d], (uint32_t)__popcll(same));
                left &= ~same;
            }
            if (__builtin_amdgcn_inverse_ballot_w64(left)) atomicAdd(&s_bin[d], 1u);
        }
        if (first_step ? __syncthreads_or(odd) : (__syncthreads(), 0)) {
            odd = true;
            break;
        }
        // the digit in which the k-th entry falls
        const int per = kBins / nt;     // 2 to 32 bins a thread
        uint32_t sum = 0;
        for (int b = 0; b < per; b++) sum += s_bin[tid * per + b];
        const uint32_t incl = (uint32_t)wave_incl_scan32((int)sum);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        uint32_t at = incl - sum + below;
        for (int w = 0; w < wave; w++) at += s_wave[w];
        if (at < (uint32_t)k && at + sum >= (uint32_t)k) {
            int b = tid * per;
            while (at + s_bin[b] < (uint32_t)k) at += s_bin[b++];
            s_digit = (uint32_t)b;
            s_below = at;
            s_in = s_bin[b];
        }
        __syncthreads();
        below = s_below;
        const uint32_t in = s_in;
        if (on_id) {
            id_pre = id_pre << (hi - lo) | s_digit;
            id_shift = lo;
        } else {
            pre = (first_step ? 0ull : pre << (hi - lo)) | s_digit;
            shift = lo;
            // none left out: on to the highest bit in which they differ
            if (in == left_in && shift > 0) {
                for (int o = 32; o > 0; o >>= 1) {
                    all_and &= __shfl_xor(all_and, o, 64);
                    all_or |= __shfl_xor(all_or, o, 64);
                }
                if (lane == 0) {
                    atomicAnd(&s_and, all_and);
                    atomicOr(&s_or, all_or);
                }
                __syncthreads();
                const uint64_t differ = s_and ^ s_or;
                shift = differ ? 64 - __builtin_clzll(differ) : 0;
                pre = s_and >> shift;
                __syncthreads();
                if (tid == 0) {
                    s_and = ~0ull;
                    s_or = 0;
                }
            }
            all_and = ~0ull;
            all_or = 0;
            left_in = in;
        }
        __syncthreads();
        if (below + in <= (uint32_t)keep) break;
    }
    // the entries up to the chosen prefix
    if (tid == 0) s_count = 0;
    __syncthreads();
    if (!odd) {
        for (int64_t c = tid; c < n; c += nt) {
            const double j = js[c];
            const int32_t id = ids[c];
            const uint64_t key = key_of(j);
            if (n <= keep) odd |= !(fabs(j) <= DBL_MAX) || key == 1ull << 63 || id < 0;
            const uint64_t kp = shift == 64 ? 0ull : key >> shift;
            const bool in = kp < pre || (kp == pre && (shift > 0 || id_shift == 32 || (uint32_t)id >> id_shift <= id_pre));
            if (in) {
                const uint32_t at = atomicAdd(&s_count, 1u);
                s_k[at] = key;
                s_id[at] = id;
            }
        }
    }
    odd = __syncthreads_or(odd);
    const int m = (int)s_count;
    if (!odd) {
        for (int t = tid; t < m; t += nt) {
            const uint64_t key = s_k[t];
            const int32_t id = s_id[t];
            int rank = 0, same = 0;
            for (int u = 0; u < m; u++) {
                const uint64_t ku = s_k[u];
                const int32_t iu = s_id[u];
                rank += (ku < key || (ku == key && iu < id)) ? 1 : 0;
                same += (ku == key && iu == id) ? 1 : 0;
            }
            odd |= same > 1;
            if (rank < k) {
                top_ids[rank] = id;
                top_j[rank] = value_of(key);
            }
        }
        for (int r = m + tid; r < k; r += nt) {
            top_ids[r] = -1;
            top_j[r] = 0.0;
        }
    }
    if (__syncthreads_or(odd))
        select_by_rounds(ids, js, n, k, reinterpret_cast<double *>(s_mem), reinterpret_cast<int32_t *>(s_mem + nt),
                         top_ids, top_j);
}

// The first few entries by rounds alone (a kernel of its own, as the registers
// and the LDS of the one above cost it a fifth).
__global__ __launch_bounds__(1024) void k_topk_few(const int64_t *__restrict__ off, const int32_t *__restrict__ ids,
                                                   const double *__restrict__ js, int32_t k,
                                                   int32_t *__restrict__ top_ids, double *__restrict__ top_j)
{
    extern __shared__ uint64_t s_mem[];
    const int64_t q = blockIdx.x, a = off[q], n = off[q + 1] - a;
    select_by_rounds(ids + a, js + a, n, k, reinterpret_cast<double *>(s_mem),
                     reinterpret_cast<int32_t *>(s_mem + blockDim.x), top_ids + q * k, top_j + q * k);
}

}  // namespace

polymh_status launch_topk(const int64_t *off, const int32_t *ids, const double *js, int64_t nq,
                          int32_t k, int32_t *top_ids, double *top_j, hipStream_t s)
{
    if (nq == 0) return POLYMH_OK;
    if (nq > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "topk: too many queries");
    // few lists: each spread over a CU's SIMDs; many: more lists in flight
    const int threads = nq < 1024 ? 1024 : 256;
    // up to four entries by rounds: 5,000 lists of 300 at k = 1, 2 and 4 take 22,
    // 28 and 42 us (47 by digits), of 3,000 44, 71 and 122 (110); one of 100,000
    // 38, 62 and 112 (119); at k = 6 digits win (47 against 52, 110 against 173)
    if (k <= 4) {
        hipLaunchKernelGGL(k_topk_few, dim3((unsigned)nq), dim3(threads), (size_t)threads * 12, s, off, ids, js, k, top_ids,
                           top_j);
        return check_launch("topk");
    }
    // ranking takes the square of what is kept: 5,000 lists of 200 and of 500 at
    // k = 10 take 54 and 49 us with 128, 71 and 91 with 256; with 64, lists of
    // few values need a step more (10,000 of 650 and eight values 140, 117 us)
    const int keep = std::max(128, 2 * k);
    const size_t lds = std::max((size_t)keep * 12 + kBins * sizeof(uint32_t), (size_t)threads * 12);
    hipLaunchKernelGGL(k_topk, dim3((unsigned)nq), dim3(threads), lds, s, off, ids, js, k, keep, top_ids, top_j);
    return check_launch("topk");
}

}  // namespace polymh
