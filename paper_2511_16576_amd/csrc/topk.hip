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
// 11,800 at k = 100 take 34 us (1,176 by rounds), 10,000 lists of 650 at
// k = 10 85 us (157 by rounds).  Up to three or four entries go by rounds.
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
    const int64_t q = blockIdx.x;
    const int64_t a = off[q], n = off[q + 1] - a;
    ids += a;
    js += a;
    top_ids += q * k;
    top_j += q * k;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, wave = tid >> 6;

    // The first few by rounds: 5,000 lists of 3,000 at k = 1 46 us (98 by
    // digits, 276 if J takes 8 values), at k = 3 103 (98, 275), at k = 4 122
    // (99, 278); one list of 100,000 37 and 86 us at k = 1 and 3 (113).  Short
    // lists wait on the digits' steps rather than on memory and gain a little
    // longer: 5,000 lists of 300 and of 500 at k = 4 49 and 52 us (65, 86), but
    // at k = 8 83 and 87 (65, 86).
    if (k <= 3 || (k == 4 && n <= 512)) {
        select_by_rounds(ids, js, n, k, reinterpret_cast<double *>(s_mem), reinterpret_cast<int32_t *>(s_mem + nt),
                         top_ids, top_j);
        return;
    }
    bool odd = n > INT32_MAX;
    int shift = 64, id_shift = 32;      // digits chosen so far end here
    uint64_t pre = 0;
    uint32_t id_pre = 0, below = 0;
    // s: bits of J from the top, then bits of the id
    for (int step = 0; n > keep && step < 9; step++) {
        const bool on_id = step >= 6;
        const int hi = on_id ? id_shift : shift, lo = hi > 11 ? hi - 11 : 0;
        const uint32_t mask = (1u << (hi - lo)) - 1;
        for (int b = tid; b < kBins; b += nt) s_bin[b] = 0;
        __syncthreads();
        for (int64_t c = tid; c < n; c += nt) {
            const double j = js[c];
            const int32_t id = ids[c];
            const uint64_t key = key_of(j);
            if (step == 0) odd |= !(fabs(j) <= DBL_MAX) || key == 1ull << 63 || id < 0;
            const bool in = on_id ? key == pre && (id_shift == 32 || (uint32_t)id >> id_shift == id_pre)
                                  : shift == 64 || key >> shift == pre;
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
        if (step == 0 ? __syncthreads_or(odd) : (__syncthreads(), 0)) {
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
            id_pre = (id_shift == 32 ? 0u : id_pre << (hi - lo)) | s_digit;
            id_shift = lo;
        } else {
            pre = (shift == 64 ? 0ull : pre << (hi - lo)) | s_digit;
            shift = lo;
        }
        __syncthreads();
        if (below + in <= (uint32_t)keep) break;
        odd = step == 8;                // more than `keep` copies of one entry
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

}  // namespace

polymh_status launch_topk(const int64_t *off, const int32_t *ids, const double *js, int64_t nq,
                          int32_t k, int32_t *top_ids, double *top_j, hipStream_t s)
{
    if (nq == 0) return POLYMH_OK;
    if (nq > 0x7fffffffLL) return set_error(POLYMH_EINVAL, "topk: too many queries");
    // few lists: each spread over a CU's SIMDs; many: more lists in flight
    const int threads = nq < 1024 ? 1024 : 256;
    const int keep = std::max(256, 2 * k);
    const size_t lds = std::max((size_t)keep * 12 + kBins * sizeof(uint32_t), (size_t)threads * 12);
    hipLaunchKernelGGL(k_topk, dim3((unsigned)nq), dim3(threads), lds, s, off, ids, js, k, keep, top_ids, top_j);
    return check_launch("topk");
}

}  // namespace polymh
