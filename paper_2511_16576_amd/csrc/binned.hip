// Shared-sample binned signing: the signatures of Alg. 1 / Def. 2, bit for
// bit, without walking every (polygon, hash) stream.  All polygons read the
// same point stream per hash (Sec. 3.2's fixed-seed generators), so the
// samples j < horizon of every hash are drawn once, in chunks of C, and each
// chunk's samples of a group of up to 256 hashes are grouped by cell of a
// 2^b x 2^b grid over B.  A polygon visits the chunks in order and, in each,
// the samples of the cells its MBR meets, which are one stretch of memory a
// grid row: those inside the MBR whose hash has no hit yet are tested for
// membership, and the smallest inside index of a hash is its first hit (every
// sample inside the polygon lies in its MBR, hence in those cells).  Units
// with no hit below the horizon are walked from the start by the per-unit
// kernel, so every value equals Alg. 1's.
//
// Polygons whose expected walk is short (|B| / area below a threshold) are
// left to the walk altogether: a first-hit index near N_B / N_P is cheaper
// to draw than to look up.
//
// Lookup layout: one workgroup per (polygon, group of hashes), lane = sample,
// so all lanes read one stretch whatever hashes it holds, the polygon's edges
// are staged once in LDS and every membership test reads them as broadcasts;
// samples inside the MBR are queued per wavefront and tested 64 at a time,
// one point per lane.  Bound: VALU issue (about 70% busy).  2 M polygons of
// 22 vertices at k = 256: 33 ms; 76 with bins a hash, lane = hash (64 places
// of memory a read, and a wavefront as slow as the hash with most samples),
// and 100 before the polygons were ordered along the plane.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "internal.hpp"
#include "sign_common.hpp"

namespace polymh {

namespace {

constexpr int kRecBatch = 128;      // points tested together against edges with their products
constexpr int kQueue = 256;        // per-wavefront queue of membership tests
constexpr int kGroup = 256;        // hashes a lookup workgroup at most, see group_hashes
constexpr int kBinLog = 13;        // log2 of the samples a workgroup of k_bin takes
constexpr uint32_t kNone = 0xffffffffu;
constexpr int kXcds = 8;           // workgroups are handed to the XCDs in turn

struct BinArgs {
    uint64_t seed;
    int32_t k;
    int32_t hashes;                // of a group
    uint32_t horizon;              // samples per hash (j < horizon), <= cap
    int32_t nchunks;
    int32_t lchunk;                // chunk C = 2^lchunk samples
    int32_t bits;                  // grid side 2^bits (0..6)
    int32_t sbx, sby;              // cell of offset o: o >> sb
    uint32_t wx, wy;
    int32_t shx, shy;
    uint32_t per;                  // samples of a (group, chunk): hashes of a group << lchunk
    int32_t parts;                 // k_bin files by this many parts of the plane: grid rows, or cells
    int32_t by_row;                // ... rows, which k_bin_row then files by cell
    uint2 *xy;                     // [groups][nchunks][per] lattice offsets, grouped by cell
    uint32_t *meta;                // hash in the group << 24 | index in the chunk
    int32_t cbits, csx;            // columns of a row: 2^cbits, that of offset o: o >> csx
    uint2 *range;                  // [groups][nchunks][rows][columns] first and past-the-end place
    uint32_t *cursor;              // [groups][nchunks][parts] counts, then next free place
    int64_t list0;                 // k_bin_row's first (group, chunk)
};

constexpr int kBinSamples = 1 << kBinLog;

// State of hash h's stream, which sample j's numbers come from.
__device__ __forceinline__ uint64_t stream_key(const BinArgs &A, int h)
{
    return mix64(A.seed + (uint64_t)(h + 1) * kGamma);
}
template <bool POW2>
__device__ __forceinline__ uint2 sample_at(const BinArgs &A, uint64_t key, uint64_t j)
{
    const uint64_t r = mix64(key + (j + 1) * kGamma);
    return make_uint2(lattice<POW2>((uint32_t)(r >> 32), A.wx, A.shx), lattice<POW2>((uint32_t)r, A.wy, A.shy));
}

enum BinTo { kCount = 0, kToRows = 1, kToCells = 2 };

// k_bin counts or files some hashes' samples of a chunk by part: counted in
// LDS, one global atomic a part, and where they are filed first ordered in
// LDS, so that a part's samples are written together.  By row, only the four
// bytes of hash and index are: k_bin_row draws the sample again, which costs
// less than the eight bytes written and read.  117 M samples take 0.20 ms to
// count, 0.28 to file by row and 0.40 by column (with the bytes 0.20, 0.53 and
// 0.65), against 3.2 written one by one to the 4,096 cells.  The order inside
// a part does not matter.
template <bool POW2, BinTo TO>
__global__ __launch_bounds__(1024) void k_bin(BinArgs A)
{
    constexpr int kPer = kBinSamples / 1024;
    constexpr bool PLACE = TO != kCount, XY = TO == kToCells;
    __shared__ uint32_t s_cnt[256], s_start[256];
    __shared__ uint32_t s_w[16];
    __shared__ uint2 s_xy[XY ? kBinSamples : 1];
    __shared__ uint32_t s_meta[PLACE ? kBinSamples : 1];
    __shared__ uint8_t s_part[PLACE ? kBinSamples : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, c = blockIdx.x;
    // kBinSamples >> lchunk hashes of the chunk, or a stretch of one hash's
    const int lh = kBinLog - A.lchunk;
    const int h0 = lh >= 0 ? (int)blockIdx.y << lh : (int)(blockIdx.y >> -lh);
    const uint32_t i0 = lh >= 0 ? 0u : (blockIdx.y & ((1u << -lh) - 1)) << kBinLog;
    const int g = h0 / A.hashes;
    const size_t gc = (size_t)g * A.nchunks + c;
    if (tid < 256) s_cnt[tid] = 0;
    __syncthreads();
    uint2 o[kPer];
    uint32_t meta[kPer], rank[kPer];
    int part[kPer];
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint32_t e = (uint32_t)(u * 1024 + tid);
        const int h = h0 + (lh >= 0 ? (int)(e >> A.lchunk) : 0);
        const uint32_t i = i0 + (lh >= 0 ? e & ((1u << A.lchunk) - 1) : e);
        const uint64_t j = ((uint64_t)c << A.lchunk) + i;
        part[u] = -1;
        if (h < A.k && j < A.horizon) {
            o[u] = sample_at<POW2>(A, stream_key(A, h), j);
            // 64-bit shifts: a 2^32-wide side with one cell shifts by 32
            const int cy = (int)((uint64_t)o[u].y >> A.sby);
            part[u] = A.by_row ? cy : cy << A.bits | (int)((uint64_t)o[u].x >> A.sbx);
            meta[u] = (uint32_t)(h - g * A.hashes) << 24 | i;
            rank[u] = atomicAdd(&s_cnt[part[u]], 1u);
        }
    }
    __syncthreads();
    uint32_t *cursor = A.cursor + gc * A.parts;
    if constexpr (!PLACE) {
        if (tid < A.parts && s_cnt[tid]) atomicAdd(&cursor[tid], s_cnt[tid]);
    } else {
        const uint32_t cnt = tid < A.parts ? s_cnt[tid] : 0u;
        const uint32_t incl = (uint32_t)wave_incl_scan32((int)cnt);
        if (lane == 63) s_w[wave] = incl;
        __syncthreads();
        uint32_t at = incl - cnt;
        for (int w = 0; w < min(wave, 4); w++) at += s_w[w];
        if (tid < 256) {
            s_start[tid] = at;
            // where a part's stretch goes, less where it starts here
            s_cnt[tid] = (cnt ? atomicAdd(&cursor[tid], cnt) : 0u) - at;
        }
        uint32_t total = 0;
        for (int w = 0; w < 4; w++) total += s_w[w];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPer; u++) {
            if (part[u] >= 0) {
                const uint32_t p = s_start[part[u]] + rank[u];
                if (XY) s_xy[p] = o[u];
                s_meta[p] = meta[u];
                s_part[p] = (uint8_t)part[u];
            }
        }
        __syncthreads();
        const size_t base = gc * A.per;
        for (uint32_t e = tid; e < total; e += 1024) {
            const size_t p = base + s_cnt[s_part[e]] + e;
            if (XY) A.xy[p] = s_xy[e];
            A.meta[p] = s_meta[e];
        }
    }
}

// Counts to starts, a wavefront a (group, chunk); where the parts are cells,
// their ranges too.
__global__ __launch_bounds__(256) void k_bin_scan(BinArgs A, int64_t lists)
{
    const int lane = threadIdx.x & 63;
    const int64_t l = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (l >= lists) return;
    uint32_t *cursor = A.cursor + l * A.parts;
    uint32_t carry = 0;
    for (int t0 = 0; t0 < A.parts; t0 += 64) {
        const int t = t0 + lane;
        const uint32_t c = t < A.parts ? cursor[t] : 0u;
        const uint32_t incl = (uint32_t)wave_incl_scan32((int)c);
        if (t < A.parts) {
            cursor[t] = carry + incl - c;
            if (!A.by_row) A.range[l * A.parts + t] = make_uint2(carry + incl - c, carry + incl);
        }
        carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
}

// One workgroup a (group, chunk, grid row): its samples by column, hash and
// index in place, kPer a thread in registers and ordered in LDS before they
// are written.
// Columns are a quarter of a cell wide, so that a stretch ends near the MBR's
// sides.  cursor holds the rows' ends by now.  A row of more samples than
// the threads hold (the hashes spread them evenly: none) stays as it is, and
// each of its columns is the whole row.
template <bool POW2, int kPer>
__global__ __launch_bounds__(1024) void k_bin_row(BinArgs A)
{
    constexpr uint32_t kMost = kPer * 1024;
    __shared__ uint64_t s_key[kGroup];
    __shared__ uint2 s_xy[kMost];
    __shared__ uint32_t s_meta[kMost];
    __shared__ uint32_t s_cnt[256], s_w[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row = blockIdx.x, side = 1 << A.cbits;
    const size_t gc = blockIdx.y;
    const uint32_t *ends = A.cursor + gc * A.parts;
    const uint32_t e0 = row ? ends[row - 1] : 0u, e1 = ends[row], n = e1 - e0;
    uint2 *xy = A.xy + gc * A.per + e0;
    uint32_t *meta = A.meta + gc * A.per + e0;
    uint2 *range = A.range + (gc << (A.bits + A.cbits)) + (row << A.cbits);
    const int64_t list = A.list0 + blockIdx.y, g = list / A.nchunks, c0 = (list - g * A.nchunks) << A.lchunk;
    if (tid < kGroup) s_key[tid] = stream_key(A, (int)g * A.hashes + tid);
    __syncthreads();
    auto sample = [&](uint32_t m) { return sample_at<POW2>(A, s_key[m >> 24], (uint64_t)c0 + (m & 0xffffffu)); };
    if (n > kMost) {
        if (tid < side) range[tid] = make_uint2(e0, e1);
        for (uint32_t e = tid; e < n; e += 1024) xy[e] = sample(meta[e]);
        return;
    }
    uint2 o[kPer];
    uint32_t m[kPer], rank[kPer];
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint32_t e = (uint32_t)(u * 1024 + tid);
        m[u] = e < n ? meta[e] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kPer; u++) o[u] = sample(m[u]);
    if (tid < 256) s_cnt[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; u++)
        rank[u] = (uint32_t)(u * 1024 + tid) < n ? atomicAdd(&s_cnt[o[u].x >> A.csx], 1u) : 0u;
    __syncthreads();
    const uint32_t c = tid < 256 ? s_cnt[tid] : 0u, incl = (uint32_t)wave_incl_scan32((int)c);
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    if (tid < 256) {
        uint32_t at = incl - c;
        for (int w = 0; w < wave; w++) at += s_w[w];
        s_cnt[tid] = at;
        if (tid < side) range[tid] = make_uint2(e0 + at, e0 + at + c);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        if ((uint32_t)(u * 1024 + tid) < n) {
            const uint32_t p = s_cnt[o[u].x >> A.csx] + rank[u];
            s_xy[p] = o[u];
            s_meta[p] = m[u];
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        const uint32_t e = (uint32_t)(u * 1024 + tid);
        if (e < n) {
            xy[e] = s_xy[e];
            meta[e] = s_meta[e];
        }
    }
}

struct LookupArgs {
    const int32_t *xy;
    const int64_t *off;
    const int32_t *mbr;
    const uint32_t *flags;
    const int64_t *area2;
    float need;                    // samples of a hash that hold the first hits, times the area
    const uint2 *bxy;              // the bins, see BinArgs
    const uint32_t *bmeta;
    const uint2 *brange;
    uint32_t per;
    uint32_t *sig;
    uint32_t *unresolved;          // [n] 1: a hash needs the walk, 2: the whole polygon is walked
    int32_t hashes;                // of a group
    const int32_t *order;          // [n] polygons in the order their workgroups start
    int32_t by_place;              // the order is along the plane: a stretch of it an XCD
    int64_t n;
    int32_t k;
    uint32_t cap, horizon;
    int32_t nchunks, lchunk, bits, cbits, csx, sby;
    int32_t bx0, by0, bx1, by1;
    int32_t lds_edges;
};

enum TestMode { kTestRec = 0, kTestLds = 1, kTestStream = 2, kTestWide = 3 };

// Lane-serial crossing-number test of the lane's own point; every lane walks
// the same edge sequence, so the edge reads are broadcasts.
template <int MODE>
__device__ __forceinline__ bool inside_lane(const int4 *s_edges, const int32_t *pxy, int32_t n,
                                            int32_t px, int32_t py)
{
    bool odd = false;
    for (int e = 0; e < n; e++) {
        if constexpr (MODE == kTestLds) {
            odd ^= crosses_fp64(s_edges[e], px, py);
        } else {
            const int f = (e + 1 == n) ? 0 : e + 1;
            if constexpr (MODE == kTestStream) {
                const int2 a = *reinterpret_cast<const int2 *>(pxy + 2 * e);
                const int2 b = *reinterpret_cast<const int2 *>(pxy + 2 * f);
                odd ^= crosses_fp64(make_edge(a.x, a.y, b.x, b.y), px, py);
            } else {
                odd ^= crosses_i128(pxy + 2 * e, pxy + 2 * f, px, py);
            }
        }
    }
    return odd;
}

// Crossing-number test of each lane's point against edges read from memory
// 64 at a time, one edge per lane in one coalesced load, and handed to every
// lane by readlane (a load per edge made each step wait on memory).  Every
// lane of the wavefront takes part.
__device__ __forceinline__ bool inside_stream_block(const int32_t *pxy, int32_t n, int32_t px, int32_t py,
                                                    int lane)
{
    bool odd = false;
    for (int e0 = 0; e0 < n; e0 += 64) {
        const int e = e0 + lane < n ? e0 + lane : 0;
        const int f = (e + 1 == n) ? 0 : e + 1;
        const int2 a = *reinterpret_cast<const int2 *>(pxy + 2 * e);
        const int2 b = *reinterpret_cast<const int2 *>(pxy + 2 * f);
        const int4 ed = make_edge(a.x, a.y, b.x, b.y);
        const int cnt = min(64, n - e0);
        for (int t = 0; t < cnt; t++) {
            const int4 et = make_int4(__builtin_amdgcn_readlane(ed.x, t), __builtin_amdgcn_readlane(ed.y, t),
                                      __builtin_amdgcn_readlane(ed.z, t), __builtin_amdgcn_readlane(ed.w, t));
            odd ^= crosses_fp64(et, px, py);
        }
    }
    return odd;
}

// Per-wavefront state of one polygon's lookup.
struct Scan {
    uint32_t mx0, my0, mwx, mwy;   // MBR inside B: corner as a lattice offset, width - 1, height - 1
    int32_t x0, y0;                // the MBR's corner
    uint32_t *queue;               // samples inside the MBR: chunk of the round << sub_shift | place in it
    uint32_t *s_best;              // smallest inside index a hash of the workgroup
    int head, tail;
    // this round's bins
    const uint2 *xy;
    const uint32_t *meta;
    int c0, sub_shift;
};

// A queued sample again: its lattice offset, hash and index.  (Queued by its
// place alone, four bytes, the queues of a workgroup that tests two points a
// lane leave room for seven workgroups a CU; with the sample's 16 bytes for
// four: 2 million polygons of 256 hashes 46.3 ms instead of 56.5.)
__device__ __forceinline__ uint4 queued(const LookupArgs &A, const Scan &S, int q)
{
    const uint32_t en = S.queue[(S.head + q) & (kQueue - 1)];
    const uint32_t at = en & ((1u << S.sub_shift) - 1);
    const uint2 o = S.xy[at];
    const uint32_t m = S.meta[at];
    return make_uint4(o.x, o.y, m >> 24, ((uint32_t)(S.c0 + (int)(en >> S.sub_shift)) << A.lchunk) + (m & 0xffffffu));
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
}

// Test POINTS * 64 queued points, POINTS a lane, against edges with their
// products taken out, and lower their hashes' best index (entries past count
// are tested again as the first one and dropped).  The edge reads are
// broadcasts, 16 cycles of the LDS an edge, three times what four SIMDs need
// for one point a lane: two points share them (46.3 ms, one point 49.5).
template <int POINTS>
__device__ __forceinline__ void drain_rec(const LookupArgs &A, const EdgeRec *rec, int32_t n, const Scan &S, int count,
                                          int lane)
{
    uint4 o[POINTS];
    int32_t ry[POINTS];
    double dx[POINTS], dy[POINTS];
    uint64_t odd[POINTS];
#pragma unroll
    for (int u = 0; u < POINTS; u++) {
        const int at = 64 * u + lane;
        o[u] = queued(A, S, at < count ? at : 0);
        ry[u] = (int32_t)((uint32_t)A.by0 + o[u].y) - S.y0;
        dx[u] = (double)((int32_t)((uint32_t)A.bx0 + o[u].x) - S.x0);
        dy[u] = (double)ry[u];
        odd[u] = 0;
    }
    EdgeRec next = rec[0];
    for (int e = 1; e <= n; e++) {
        const EdgeRec r = next;
        next = rec[e < n ? e : 0];
#pragma unroll
        for (int u = 0; u < POINTS; u++) odd[u] ^= crosses_mask(r, ry[u], dx[u], dy[u]);
    }
#pragma unroll
    for (int u = 0; u < POINTS; u++) {
        const uint64_t in = odd[u] & __ballot(64 * u + lane < count);
        if (__builtin_amdgcn_inverse_ballot_w64(in)) atomicMin(&S.s_best[o[u].z], o[u].w);
    }
}

// Test up to 64 (kTestRec: 128) queued points and lower their hashes' best
// index.
template <int MODE>
__device__ __forceinline__ void drain(const LookupArgs &A, const int4 *s_edges, const int32_t *pxy, int32_t n,
                                      const Scan &S, int count, int lane)
{
    if constexpr (MODE == kTestRec) {
        const EdgeRec *rec = reinterpret_cast<const EdgeRec *>(s_edges);
        if (count > 64) drain_rec<2>(A, rec, n, S, count, lane);
        else drain_rec<1>(A, rec, n, S, count, lane);
        return;
    }
    // lanes past count test the first entry where every lane takes part
    if (MODE != kTestStream && lane >= count) return;
    const uint4 o = queued(A, S, lane < count ? lane : 0);
    const int32_t px = (int32_t)((uint32_t)A.bx0 + o.x), py = (int32_t)((uint32_t)A.by0 + o.y);
    bool in;
    if constexpr (MODE == kTestStream) in = inside_stream_block(pxy, n, px, py, lane) && lane < count;
    else in = inside_lane<MODE>(s_edges, pxy, n, px, py);
    if (in) atomicMin(&S.s_best[o.z], o.w);
}

// One sample a lane: those inside the MBR whose hash has no smaller index yet
// are queued, 64 (kTestRec: 128) waiting are tested.
template <int MODE>
__device__ __forceinline__ void take(const LookupArgs &A, const int4 *s_edges, const int32_t *pxy, int32_t n, Scan &S,
                                     uint2 o, uint32_t meta, uint32_t chunk_base, uint32_t place, int lane)
{
    const uint32_t hash = meta >> 24, j = chunk_base + (meta & 0xffffffu);
    const uint64_t mk = __ballot(o.x - S.mx0 <= S.mwx) & __ballot(o.y - S.my0 <= S.mwy) & __ballot(S.s_best[hash] > j);
    if (mk == 0) return;
    if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
        const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mk >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u));
        S.queue[(S.tail + rank) & (kQueue - 1)] = place;
    }
    S.tail += __popcll(mk);
    constexpr int kBatch = MODE == kTestRec ? kRecBatch : 64;
    if (S.tail - S.head >= kBatch) {
        wave_sync_lds();
        drain<MODE>(A, s_edges, pxy, n, S, kBatch, lane);
        S.head += kBatch;
        wave_sync_lds();
    }
}

// The chunks in rounds of some at a time: lane l of a wavefront knows the
// stretch of (chunk l / rows of the round, grid row l % rows), the
// wavefronts take 64 samples at a time in turn.  After a round, a hash with a
// hit is settled (all smaller indices have been seen); the workgroup is done
// when all are.  Rounds double what was read, as what is left open shrinks: the
// barriers and the ranges' latency are paid once a round, the samples of
// settled hashes read on the way cost one compare.  Every wavefront takes part; all
// arguments but `active`, tid and lane are wavefront-uniform.
//
// `need` samples a hash hold the first hits of all hashes of 31 workgroups in
// 32, so the first round takes the chunks that those fill: 2 M polygons of 22
// vertices 39.2 ms, 44.5 with eight chunks for all of them, 41.0 with eight at
// most.  Where they are less than most of one chunk, and it is a long one (at
// most 64 hashes, one wavefront), only they are tested at first; if a hash is
// then open, the chunk is read again, whole.  3,000 large polygons at 4 hashes
// take 317 us, 535 without the bound; 100 of 75 edges at 16 hashes 162, 274
// without it, 444 with longer chunks and rounds of eight too.  With 128 hashes,
// whose chunk is half as long, reading one twice costs more than that saves
// (3,000 large polygons 1,450 us, 1,657 with it).
template <int MODE>
__device__ void lookup_polygon(const LookupArgs &A, const int4 *s_edges, const int32_t *pxy, int32_t n, Scan &S, int cx0,
                               int cx1, int cy0, int cy1, bool active, int tid, int lane, int wave, int waves, int group, float need)
{
    const int rows = cy1 - cy0 + 1;              // at most 64
    // chunks a round at most: a round's samples are counted in 26 bits, or,
    // alone, a chunk's in 28
    const int most = max(1, min(64 / rows, (int)((1u << 26) / A.per)));
    S.sub_shift = most > 1 ? 26 : 31;
    const int sub = lane / rows, row = (cy0 + lane % rows) << A.cbits;
    int m = max(1, (int)fminf(ceilf(ldexpf(need, -A.lchunk)), (float)most));
    uint32_t bound = kNone;
    if (waves == 1 && need < 0.75f * (float)(1u << A.lchunk)) {
        bound = (uint32_t)need + 1;
        S.s_best[tid] = bound;
        __syncthreads();
    }
    for (int c0 = 0; c0 < A.nchunks;) {
        const size_t gc = (size_t)group * A.nchunks + c0;
        uint32_t e0 = 0, e1 = 0;
        if (sub < m && c0 + sub < A.nchunks) {
            const uint2 *range = A.brange + ((gc + sub) << (A.bits + A.cbits));
            // bounded also where the bins are not there
            e0 = min(range[row | cx0].x, A.per);
            e1 = min(range[row | cx1].y, A.per);
        }
        const int steps = e1 > e0 ? (int)((e1 - e0 + 63) / 64) : 0;
        const int incl = wave_incl_scan32(steps);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        // places count from the round's first sample
        const int skip = sub * (int)A.per;
        const int from = skip + (int)e0 - 64 * (incl - steps), last = skip + (int)e1 - 1;
        const uint32_t base = (uint32_t)(c0 + sub) << A.lchunk;
        S.xy = A.bxy + gc * A.per;
        S.meta = A.bmeta + gc * A.per;
        S.c0 = c0;
        S.head = S.tail = 0;
        // step t: its stretch is the first that ends after it; lanes past the
        // stretch's end take its last sample again, which changes nothing
        struct Step {
            uint2 o;
            uint32_t meta, base, place;
        } a{}, b{};
        auto load = [&](int t, Step &s) {
            const int l = __builtin_ctzll(__ballot(incl > t));
            const int at = min(__builtin_amdgcn_readlane(from, l) + 64 * t + lane, __builtin_amdgcn_readlane(last, l));
            s.base = (uint32_t)__builtin_amdgcn_readlane((int)base, l);
            __builtin_assume(at >= 0 && at < 1 << 28);
            s.o = S.xy[at];
            s.meta = S.meta[at];
            s.place = (uint32_t)at | (uint32_t)__builtin_amdgcn_readlane(sub, l) << S.sub_shift;
        };
        // two steps in flight
        int t = wave;
        if (t < total) load(t, a);
        if (t + waves < total) load(t + waves, b);
        while (t < total) {
            take<MODE>(A, s_edges, pxy, n, S, a.o, a.meta, a.base, a.place, lane);
            t += waves;
            if (t + waves < total) load(t + waves, a);
            if (t >= total) break;
            take<MODE>(A, s_edges, pxy, n, S, b.o, b.meta, b.base, b.place, lane);
            t += waves;
            if (t + waves < total) load(t + waves, b);
        }
        while (S.tail > S.head) {
            wave_sync_lds();
            const int left = min(MODE == kTestRec ? kRecBatch : 64, S.tail - S.head);
            drain<MODE>(A, s_edges, pxy, n, S, left, lane);
            S.head += left;
            wave_sync_lds();
        }
        __syncthreads();
        const bool open = active && S.s_best[tid] == bound;
        if (!__syncthreads_or(open)) break;
        if (bound != kNone) {
            if (open) S.s_best[tid] = kNone;
            bound = kNone;
            __syncthreads();
        } else {
            c0 += m;
            m = min(most, max(m, c0));
        }
    }
}

// One workgroup per (polygon, group of hashes), with a thread a hash rounded up
// to wavefronts.
__global__ __launch_bounds__(256) void k_bin_lookup(LookupArgs A)
{
    extern __shared__ int4 s_edges[];
    __shared__ uint32_t s_queue[4][kQueue];
    __shared__ uint32_t s_best[kGroup];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per = blockDim.x;
    const int groups = (A.k + A.hashes - 1) / A.hashes;
    // workgroups start in order of their index, index b on XCD b % kXcds
    int64_t at = blockIdx.x / groups;
    if (A.by_place) {
        const int64_t per_xcd = (A.n + kXcds - 1) / kXcds;
        at = at % kXcds * per_xcd + at / kXcds;
        if (at >= A.n) return;
    }
    // read through a vector load, made uniform so that what follows is scalar
    const int64_t p = __builtin_amdgcn_readfirstlane(A.order[at]);
    const int i = (int)(blockIdx.x % groups) * A.hashes + tid;
    const bool active = tid < A.hashes && i < A.k;
    if (A.unresolved[p] & 2u) return;    // walked (uniform per workgroup, before any barrier)
    const int64_t a = (int64_t)dpp::readlane64((uint64_t)A.off[p], 0);
    const int32_t n = __builtin_amdgcn_readfirstlane((int32_t)(A.off[p + 1] - a));
    const uint32_t fl = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.flags[p]);
    int4 mb = *reinterpret_cast<const int4 *>(A.mbr + 4 * p);
    mb.x = __builtin_amdgcn_readfirstlane(mb.x);
    mb.y = __builtin_amdgcn_readfirstlane(mb.y);
    mb.z = __builtin_amdgcn_readfirstlane(mb.z);
    mb.w = __builtin_amdgcn_readfirstlane(mb.w);
    uint32_t *out = A.sig + (size_t)p * (size_t)A.k;
    const bool empty = (fl & (kFlagFew | kFlagCollinear)) || mb.z < A.bx0 || mb.x > A.bx1 ||
                       mb.w < A.by0 || mb.y > A.by1;
    if (empty) {
        if (active) out[i] = 0u;
        return;
    }
    const int32_t *pxy = A.xy + 2 * a;
    // the cache holds lds_edges edges, or half as many with their products
    const int mode = (fl & kFlagWide) ? kTestWide
                                      : 2 * n <= A.lds_edges ? kTestRec : n <= A.lds_edges ? kTestLds : kTestStream;
    if (mode <= kTestLds) {
        for (int e = tid; e < n; e += per) {
            const int f = (e + 1 == n) ? 0 : e + 1;
            const int2 u = *reinterpret_cast<const int2 *>(pxy + 2 * e);
            const int2 v = *reinterpret_cast<const int2 *>(pxy + 2 * f);
            const int4 ed = make_edge(u.x, u.y, v.x, v.y);
            if (mode == kTestRec) reinterpret_cast<EdgeRec *>(s_edges)[e] = make_edge_rec(ed, mb.x, mb.y);
            else s_edges[e] = ed;
        }
    }
    __syncthreads();
    Scan S;
    S.mx0 = (uint32_t)max(mb.x, A.bx0) - (uint32_t)A.bx0;
    S.my0 = (uint32_t)max(mb.y, A.by0) - (uint32_t)A.by0;
    const uint32_t mx1 = (uint32_t)min(mb.z, A.bx1) - (uint32_t)A.bx0, my1 = (uint32_t)min(mb.w, A.by1) - (uint32_t)A.by0;
    S.mwx = mx1 - S.mx0;
    S.mwy = my1 - S.my0;
    S.x0 = mb.x;
    S.y0 = mb.y;
    S.queue = s_queue[wave];
    S.s_best = s_best;
    // 64-bit shifts: a 2^32-wide side with one cell shifts by 32
    const int cx0 = (int)((uint64_t)S.mx0 >> A.csx), cx1 = (int)((uint64_t)mx1 >> A.csx);
    const int cy0 = (int)((uint64_t)S.my0 >> A.sby), cy1 = (int)((uint64_t)my1 >> A.sby);
    for (int t = tid; t < kGroup; t += per) s_best[t] = kNone;
    __syncthreads();                 // the edges and the bests
    const int group = (int)(blockIdx.x % groups);
    const float area = 0.5f * fabsf((float)A.area2[p]);
    const float need = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(A.need / fmaxf(area, 0.5f))));
    if (mode == kTestRec)
        lookup_polygon<kTestRec>(A, s_edges, pxy, n, S, cx0, cx1, cy0, cy1, active, tid, lane, wave, per >> 6, group, need);
    else if (mode == kTestLds)
        lookup_polygon<kTestLds>(A, s_edges, pxy, n, S, cx0, cx1, cy0, cy1, active, tid, lane, wave, per >> 6, group, need);
    else if (mode == kTestStream)
        lookup_polygon<kTestStream>(A, s_edges, pxy, n, S, cx0, cx1, cy0, cy1, active, tid, lane, wave, per >> 6, group, need);
    else
        lookup_polygon<kTestWide>(A, s_edges, pxy, n, S, cx0, cx1, cy0, cy1, active, tid, lane, wave, per >> 6, group, need);
    const uint32_t best = active ? s_best[tid] : 0u;
    if (active) {
        if (best != kNone) out[i] = best + 1;
        else if (A.horizon >= A.cap) out[i] = 0u;
        else atomicOr(&A.unresolved[p], 1u);
    }
}

// Dispatch order of the polygons for the lookup, longest first.  A workgroup
// runs until the last of its 256 hashes has a hit, about ln(256) |B| / area
// samples a hash (capped at the horizon), read in rounds of a few round trips
// to memory, and tests about kTestSlack A_MBR / area samples a hash against
// its n edges.  Started last, the few polygons with the largest such cost set
// the launch's duration; started first, they overlap the rest.  A counting
// sort on a quantised estimate (descending; the order within a key is the
// arrival order, which affects only timing).  Walked and degenerate polygons,
// whose workgroups return at once, go last.
constexpr int kOrderCells = 4096;
constexpr int64_t kOrderMaxPolys = 65536;
// Samples of a hash tested, over the A_MBR / area up to its first hit: those
// queued before that hit was known.
constexpr double kTestSlack = 1.5;

__global__ __launch_bounds__(256) void k_order_count(const int64_t *__restrict__ area2,
                                                     const int64_t *__restrict__ off,
                                                     const int32_t *__restrict__ mbr,
                                                     const uint32_t *__restrict__ unresolved, int64_t n,
                                                     double box_area, double horizon,
                                                     uint16_t *__restrict__ key, int32_t *__restrict__ counts)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const double area = 0.5 * (double)(area2[p] < 0 ? -area2[p] : area2[p]);
        int k = kOrderCells - 1;
        if (!(unresolved[p] & 2u) && area > 0.0) {
            const int4 b = *reinterpret_cast<const int4 *>(mbr + 4 * p);
            const double a_mbr = ((double)b.z - (double)b.x + 1.0) * ((double)b.w - (double)b.y + 1.0);
            const double samples = fmin(horizon, 5.545 * box_area / area);   // ln(256) |B| / area
            const double tests = kTestSlack * a_mbr / area;
            const double est = samples / 256.0 + tests * (double)(off[p + 1] - off[p]) / 8.0;
            k = kOrderCells - 1 - (int)fmin(est, (double)(kOrderCells - 1));
        }
        key[p] = (uint16_t)k;
        // the last key (every walked polygon) is counted once a wavefront
        const bool last = k == kOrderCells - 1;
        const uint64_t m = __ballot(last);
        if (!last) atomicAdd(&counts[k], 1);
        else if ((int)(threadIdx.x & 63) == __builtin_ctzll(m)) atomicAdd(&counts[k], __popcll(m));
    }
}

// Dispatch order of a large launch: along the Z-order curve of the polygons'
// MBR centres (64 x 64 cells; walked polygons, whose workgroups return at once,
// among the others).  A (polygon, hash) unit reads a few lines of that hash's bins; polygons of one place read the same
// lines, and started together they find them in their XCD's L2.
// A counting sort: a block counts its stretch of the polygons in LDS and adds
// one number a cell to the totals (k_place_count), then reserves its range of
// every cell and fills it (k_place_scatter); the order inside a cell affects
// only timing.
__device__ __forceinline__ uint32_t spread_bits8(uint32_t v)
{
    v = (v | v << 4) & 0x0f0fu;
    v = (v | v << 2) & 0x3333u;
    return (v | v << 1) & 0x5555u;
}

constexpr int kPlaceThreads = 1024;

__global__ __launch_bounds__(kPlaceThreads) void k_place_count(const int32_t *__restrict__ mbr, int64_t n, int64_t per,
                                                               int32_t bx0, int32_t by0, int32_t bx1, int32_t by1,
                                                               int32_t sx, int32_t sy, uint16_t *__restrict__ key,
                                                               int32_t *__restrict__ counts)
{
    __shared__ int32_t s_cnt[kOrderCells];
    for (int c = threadIdx.x; c < kOrderCells; c += kPlaceThreads) s_cnt[c] = 0;
    __syncthreads();
    const int64_t end = min(n, (blockIdx.x + 1) * per);
    for (int64_t p = blockIdx.x * per + threadIdx.x; p < end; p += kPlaceThreads) {
        const int32_t *m = mbr + 4 * p;
        // the MBR's centre, brought into B, as an offset from its corner
        const int64_t x = min(max(((int64_t)m[0] + m[2]) >> 1, (int64_t)bx0), (int64_t)bx1) - bx0;
        const int64_t y = min(max(((int64_t)m[1] + m[3]) >> 1, (int64_t)by0), (int64_t)by1) - by0;
        const uint32_t c = spread_bits8((uint32_t)(x >> sx)) | spread_bits8((uint32_t)(y >> sy)) << 1;
        key[p] = (uint16_t)c;
        atomicAdd(&s_cnt[c], 1);
    }
    __syncthreads();
    for (int c = threadIdx.x; c < kOrderCells; c += kPlaceThreads)
        if (s_cnt[c]) atomicAdd(&counts[c], s_cnt[c]);
}

__global__ __launch_bounds__(kPlaceThreads) void k_place_scatter(const uint16_t *__restrict__ key, int64_t n, int64_t per,
                                                                 int32_t *__restrict__ cursor,
                                                                 int32_t *__restrict__ order)
{
    __shared__ int32_t s_cnt[kOrderCells];
    for (int c = threadIdx.x; c < kOrderCells; c += kPlaceThreads) s_cnt[c] = 0;
    __syncthreads();
    const int64_t begin = blockIdx.x * per, end = min(n, begin + per);
    for (int64_t p = begin + threadIdx.x; p < end; p += kPlaceThreads) atomicAdd(&s_cnt[key[p]], 1);
    __syncthreads();
    for (int c = threadIdx.x; c < kOrderCells; c += kPlaceThreads)
        if (s_cnt[c]) s_cnt[c] = atomicAdd(&cursor[c], s_cnt[c]);
    __syncthreads();
    for (int64_t p = begin + threadIdx.x; p < end; p += kPlaceThreads)
        order[atomicAdd(&s_cnt[key[p]], 1)] = (int32_t)p;
}

// Exclusive prefix of the kOrderCells counts in place (one block of 1024).
__global__ __launch_bounds__(1024) void k_order_scan(int32_t *__restrict__ counts)
{
    constexpr int kPer = kOrderCells / 1024;
    __shared__ int sw[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int v[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        v[u] = counts[kPer * tid + u];
        sum += v[u];
    }
    const int incl = wave_incl_scan32(sum);
    if (lane == 63) sw[wave] = incl;
    __syncthreads();
    int pre = incl - sum;
    for (int w = 0; w < wave; w++) pre += sw[w];
#pragma unroll
    for (int u = 0; u < kPer; u++) {
        counts[kPer * tid + u] = pre;
        pre += v[u];
    }
}

__global__ __launch_bounds__(256) void k_order_scatter(const uint16_t *__restrict__ key, int64_t n,
                                                       int32_t *__restrict__ cursor, int32_t *__restrict__ order)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const int k = key[p];
        // positions of the last key are claimed once a wavefront
        const bool last = k == kOrderCells - 1;
        const uint64_t m = __ballot(last);
        int pos;
        if (last) {
            const int leader = __builtin_ctzll(m);
            int base = 0;
            if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(&cursor[k], __popcll(m));
            base = __shfl(base, leader, 64);
            pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        } else {
            pos = atomicAdd(&cursor[k], 1);
        }
        order[pos] = (int32_t)p;
    }
}

// Flags: 2 for a polygon to walk whole, else 0 (twice the area exact from
// prepare).  With walk_ratio > 0 a polygon is walked when |B| < walk_ratio x
// area, or when its walk is expected to cost less than its lookup, in edge
// tests per hash: the walk draws about |B| / area points (kDrawTests edge
// tests each) and tests the about A_mbr / area of them inside the MBR against
// its n edges; the lookup tests about kTestSlack as many.  Either way the
// signature is the same.  A polygon beyond the lookup's LDS edge cache
// (walk_edges) is walked too, and in a small launch so is one whose lookup
// would test more than test_cap edges a hash: one lookup workgroup tests its
// 256 hashes' points with four wavefronts, a long serial run that sets a
// small launch's duration, where the walk spreads a polygon's hashes over
// many work items and each test over the lanes.  Degenerate polygons stay
// with the lookup, which signs them 0 at once.
constexpr double kDrawTests = 5.0;
constexpr double kLookupTestCap = 2048.0;

__global__ __launch_bounds__(256) void k_classify(const int64_t *__restrict__ area2,
                                                  const uint32_t *__restrict__ flags,
                                                  const int64_t *__restrict__ off,
                                                  const int32_t *__restrict__ mbr, int64_t n,
                                                  double box_area, double walk_ratio,
                                                  double walk_edges, double test_cap,
                                                  uint32_t *__restrict__ unresolved)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x) {
        const bool degenerate = (flags[p] & (kFlagFew | kFlagCollinear)) != 0;
        const double area = 0.5 * (double)(area2[p] < 0 ? -area2[p] : area2[p]);
        bool walk = false;
        if (!degenerate && walk_ratio > 0.0 && area > 0.0) {
            const int4 m = *reinterpret_cast<const int4 *>(mbr + 4 * p);
            const double a_mbr = ((double)m.z - (double)m.x + 1.0) * ((double)m.w - (double)m.y + 1.0);
            const double edges = (double)(off[p + 1] - off[p]);
            const double walk_cost = kDrawTests * box_area / area + edges * a_mbr / area;
            const double bin_cost = kTestSlack * edges * a_mbr / area;
            walk = box_area < walk_ratio * area || walk_cost < bin_cost || edges > walk_edges ||
                   bin_cost > test_cap;
        }
        unresolved[p] = walk ? 2u : 0u;
    }
}

// Polygons with an unresolved hash, or walked whole, listed for the walk.
__global__ __launch_bounds__(256) void k_unresolved_list(const uint32_t *__restrict__ unresolved, int64_t n,
                                                         int32_t *__restrict__ list, int32_t *__restrict__ count)
{
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += (int64_t)gridDim.x * blockDim.x)
        if (unresolved[p]) list[atomicAdd(count, 1)] = (int32_t)p;
}

__global__ __launch_bounds__(256) void k_zero_words(uint32_t *p, int64_t count)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = 0u;
}


int ceil_log2(uint64_t w)
{
    int l = 0;
    while ((1ull << l) < w) l++;
    return l;
}

int grid_for(int64_t items)
{
    int64_t g = (items + 255) / 256;
    return (int)(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

// Chunks of 256 to 1,024 samples a hash, a quarter of a sample per cell at
// the finest grid, so that a settled hash is found so early; more where a
// group has fewer than kGroup hashes, so that a chunk's cells hold enough of
// them together to fill a wavefront's reads, or for a horizon of many chunks:
// twice as many at 128 hashes, and from there on twice as many for every
// quarter of them, as what is read past the first hits grows too (a lookup of
// 16 hashes by 100 and 3,000 polygons takes 88 and 332 us, 111 and 364 with
// twice as many for every half).  A grid row of a chunk then holds 4,096 samples at most
// where k_bin_row files it, or half as many rows twice that.
constexpr int64_t kMostChunks = 65535;

int64_t chunks_of(uint32_t horizon, int lchunk) { return ((int64_t)horizon + ((int64_t)1 << lchunk) - 1) >> lchunk; }

bool horizon_fits(uint32_t horizon, int32_t bits)
{
    return chunks_of(horizon, std::min(12, std::max(8, 2 * bits))) <= kMostChunks;
}

int64_t hash_groups(int32_t k) { return (k + kGroup - 1) / kGroup; }

int chunk_log2(int32_t bits, int32_t k, uint32_t horizon)
{
    int l = std::max(8, bits + 4);
    // (a little more than half, which k_bin_row's threads still hold, as half)
    int halvings = 0;
    for (int64_t h = (k + hash_groups(k) - 1) / hash_groups(k); 2 * h <= kGroup + kGroup / 16; h *= 2) halvings++;
    l += std::min(halvings, (halvings + 2) / 2);
    while (chunks_of(horizon, l) > kMostChunks) l++;
    return l;
}

// Hashes of a group: k spread evenly, whole workgroups of k_bin, so that one
// hash more than a multiple of 256 does not cost the bins of 256.
int group_hashes(int32_t k, int lchunk)
{
    const int64_t groups = hash_groups(k);
    if (groups == 1) return k;
    const int64_t step = (int64_t)1 << std::max(0, kBinLog - lchunk);
    return (int)(((k + groups - 1) / groups + step - 1) / step * step);
}

// k_bin files straight by cell while its 8,192 samples leave 32 a cell.
bool bins_by_row(int32_t bits) { return bits > 4; }
// ... and k_bin_row by quarters of a cell where a cell has them.
int col_bits(int32_t bits, int lx) { return bits + (bins_by_row(bits) && lx >= bits + 2 ? 2 : 0); }
int64_t bin_parts(int32_t bits) { return (int64_t)1 << (bins_by_row(bits) ? bits : 2 * bits); }

// Samples of a (group, chunk).
int64_t group_samples(int32_t k, int lchunk) { return (int64_t)group_hashes(k, lchunk) << lchunk; }

struct BinnedWs {
    uint2 *xy;
    uint32_t *meta, *cursor;
    uint2 *range;
    uint32_t *unresolved;
    int32_t *list, *count;
    int32_t *order, *cell_counts;
    uint16_t *key;
};

BinnedWs carve_binned(Carve &c, int32_t k, uint32_t horizon, int32_t bits, int64_t n)
{
    const int lchunk = chunk_log2(bits, k, horizon);
    const int64_t nchunks = chunks_of(horizon, lchunk);
    const int64_t lists = hash_groups(k) * nchunks, samples = lists * group_samples(k, lchunk);
    const int64_t cells = (int64_t)1 << (2 * bits + (bins_by_row(bits) ? 2 : 0));
    BinnedWs w{};
    w.xy = c.take<uint2>((size_t)samples);
    w.meta = c.take<uint32_t>((size_t)samples);
    w.range = c.take<uint2>((size_t)(lists * cells));
    w.cursor = c.take<uint32_t>((size_t)(lists * bin_parts(bits)));
    w.unresolved = c.take<uint32_t>((size_t)n);
    w.list = c.take<int32_t>((size_t)n);
    w.count = c.take<int32_t>(1);
    w.order = c.take<int32_t>((size_t)n);
    w.cell_counts = c.take<int32_t>((size_t)kOrderCells);
    w.key = c.take<uint16_t>((size_t)n);
    return w;
}

}  // namespace

size_t binned_workspace_bytes(int32_t k, uint32_t horizon, int32_t bits, int64_t n)
{
    Carve c{nullptr, 0};
    carve_binned(c, k, horizon, bits, n);
    return align_up(c.used, 256);
}

polymh_status launch_sign_binned(const SignLaunch &L, const int64_t *area2, uint32_t horizon, int32_t bits,
                                 double walk_ratio, void *ws, size_t ws_bytes, hipStream_t s, bool rebin)
{
    const uint64_t wx = (uint64_t)((int64_t)L.box.xmax - L.box.xmin + 1);
    const uint64_t wy = (uint64_t)((int64_t)L.box.ymax - L.box.ymin + 1);
    const int lx = ceil_log2(wx), ly = ceil_log2(wy);
    const bool pow2 = (1ull << lx) == wx && (1ull << ly) == wy && lx >= 1 && ly >= 1;
    if (!horizon_fits(horizon, bits)) return set_error(POLYMH_EINVAL, "sign_binned: horizon too large");
    const int lchunk = chunk_log2(bits, L.k, horizon);
    const int64_t nchunks = chunks_of(horizon, lchunk);
    Carve cv{static_cast<char *>(ws), ws_bytes};
    BinnedWs w = carve_binned(cv, L.k, horizon, bits, L.n);
    if (!cv.ok)
        return set_error(POLYMH_ECAPACITY, "sign_binned: workspace of %zu bytes, need %zu", ws_bytes, cv.used);
    BinArgs B{};
    B.seed = L.seed;
    B.k = L.k;
    B.hashes = group_hashes(L.k, lchunk);
    B.horizon = horizon;
    B.nchunks = (int32_t)nchunks;
    B.lchunk = lchunk;
    B.bits = bits;
    B.sbx = lx > bits ? lx - bits : 0;
    B.sby = ly > bits ? ly - bits : 0;
    B.wx = (uint32_t)wx;
    B.wy = (uint32_t)wy;
    B.shx = pow2 ? 32 - lx : 0;
    B.shy = pow2 ? 32 - ly : 0;
    B.per = (uint32_t)group_samples(L.k, lchunk);
    B.xy = w.xy;
    B.meta = w.meta;
    B.range = w.range;
    B.cursor = w.cursor;
    B.parts = (int32_t)bin_parts(bits);
    B.by_row = bins_by_row(bits) ? 1 : 0;
    B.cbits = col_bits(bits, lx);
    B.csx = lx > B.cbits ? lx - B.cbits : 0;
    // without rebin the workspace already holds these bins (an earlier call
    // with the same arguments); the lookup clamps every stretch to its chunk,
    // so bins that are not there give wrong values, never a stray read
    if (rebin) {
        const int64_t lists = hash_groups(L.k) * nchunks;
        const int64_t ys = lchunk <= kBinLog ? (L.k + (1 << (kBinLog - lchunk)) - 1) >> (kBinLog - lchunk)
                                             : (int64_t)L.k << (lchunk - kBinLog);
        const dim3 bgrid((unsigned)nchunks, (unsigned)ys);
        hipLaunchKernelGGL(k_zero_words, dim3(grid_for(lists * B.parts)), dim3(256), 0, s, w.cursor, lists * B.parts);
        hipLaunchKernelGGL((pow2 ? k_bin<true, kCount> : k_bin<false, kCount>), bgrid, dim3(1024), 0, s, B);
        hipLaunchKernelGGL(k_bin_scan, dim3((unsigned)((lists + 3) / 4)), dim3(256), 0, s, B, lists);
        if (B.by_row)
            hipLaunchKernelGGL((pow2 ? k_bin<true, kToRows> : k_bin<false, kToRows>), bgrid, dim3(1024), 0, s, B);
        else
            hipLaunchKernelGGL((pow2 ? k_bin<true, kToCells> : k_bin<false, kToCells>), bgrid, dim3(1024), 0, s, B);
        // a row's samples, with room for what chance adds to them
        const double even = (double)B.per * std::ldexp(1.0, B.sby) / (double)wy;
        const bool narrow = even + 8.0 * std::sqrt(even) <= 5 * 1024;
        for (int64_t l0 = 0; B.by_row && l0 < lists; l0 += 65535) {
            BinArgs R = B;
            R.xy += l0 * B.per;
            R.meta += l0 * B.per;
            R.range += l0 << (bits + B.cbits);
            R.cursor += l0 * B.parts;
            const dim3 rgrid(1u << bits, (unsigned)std::min<int64_t>(65535, lists - l0));
            R.list0 = l0;
            if (narrow)
                hipLaunchKernelGGL((pow2 ? k_bin_row<true, 5> : k_bin_row<false, 5>), rgrid, dim3(1024), 0, s, R);
            else
                hipLaunchKernelGGL((pow2 ? k_bin_row<true, 12> : k_bin_row<false, 12>), rgrid, dim3(1024), 0, s, R);
        }
    }
    polymh_status st = check_launch("sign_binned: bin");
    if (st) return st;
    // one workgroup per (polygon, group of hashes)
    const int64_t per = (B.hashes + 63) / 64 * 64, groups = hash_groups(L.k);
    const int64_t units = L.n * groups;
    const double walk_edges = (double)L.cfg.lds_edges;
    // the order and the cap on a lookup's tests serve small launches, where a
    // few costly polygons set the duration; a large launch hides them
    const bool ordered = L.n <= kOrderMaxPolys;
    hipLaunchKernelGGL(k_classify, dim3(grid_for(L.n)), dim3(256), 0, s, area2, L.flags, L.off, L.mbr, L.n,
                       (double)wx * (double)wy, walk_ratio, walk_edges,
                       ordered ? kLookupTestCap : INFINITY, w.unresolved);
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(64), 0, s, reinterpret_cast<uint32_t *>(w.count), (int64_t)1);
    // the lookup's dispatch order (after the classification: in a small launch
    // walked polygons last)
    hipLaunchKernelGGL(k_zero_words, dim3(kOrderCells / 256), dim3(256), 0, s,
                       reinterpret_cast<uint32_t *>(w.cell_counts), (int64_t)kOrderCells);
    if (ordered) {
        hipLaunchKernelGGL(k_order_count, dim3(grid_for(L.n)), dim3(256), 0, s, area2, L.off, L.mbr, w.unresolved, L.n,
                           (double)wx * (double)wy, (double)horizon, w.key,
                           w.cell_counts);
        hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(1024), 0, s, w.cell_counts);
        hipLaunchKernelGGL(k_order_scatter, dim3(grid_for(L.n)), dim3(256), 0, s, w.key, L.n, w.cell_counts, w.order);
    } else {
        const int64_t blocks = std::min<int64_t>(cu_count(), (L.n + 4095) / 4096), each = (L.n + blocks - 1) / blocks;
        hipLaunchKernelGGL(k_place_count, dim3((unsigned)blocks), dim3(kPlaceThreads), 0, s, L.mbr, L.n, each,
                           L.box.xmin, L.box.ymin, L.box.xmax, L.box.ymax, lx > 6 ? lx - 6 : 0, ly > 6 ? ly - 6 : 0,
                           w.key, w.cell_counts);
        hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(1024), 0, s, w.cell_counts);
        hipLaunchKernelGGL(k_place_scatter, dim3((unsigned)blocks), dim3(kPlaceThreads), 0, s, w.key, L.n, each,
                           w.cell_counts, w.order);
    }
    polymh_status st0 = check_launch("sign_binned: order");
    if (st0) return st0;
    LookupArgs A{};
    A.xy = L.xy;
    A.off = L.off;
    A.mbr = L.mbr;
    A.flags = L.flags;
    A.area2 = area2;
    A.need = (float)(std::log(32.0 * B.hashes) * (double)wx * (double)wy);
    A.bxy = w.xy;
    A.bmeta = w.meta;
    A.brange = w.range;
    A.per = B.per;
    A.sig = L.sig;
    A.unresolved = w.unresolved;
    A.order = w.order;
    A.hashes = B.hashes;
    A.by_place = ordered ? 0 : 1;
    A.n = L.n;
    A.k = L.k;
    A.cap = L.cap;
    A.horizon = horizon;
    A.nchunks = (int32_t)nchunks;
    A.lchunk = lchunk;
    A.bits = bits;
    A.cbits = B.cbits;
    A.csx = B.csx;
    A.sby = B.sby;
    A.bx0 = L.box.xmin; A.by0 = L.box.ymin; A.bx1 = L.box.xmax; A.by1 = L.box.ymax;
    A.lds_edges = L.cfg.lds_edges;
    // by place, every XCD's stretch is rounded up (the workgroups past the
    // end return)
    const int64_t grid = ordered ? units : (L.n + kXcds - 1) / kXcds * kXcds * groups;
    if (grid > 0x7fffffff) return set_error(POLYMH_EINVAL, "sign_binned: too many work items");
    const size_t lds = (size_t)L.cfg.lds_edges * sizeof(int4);
    hipLaunchKernelGGL(k_bin_lookup, dim3((unsigned)grid), dim3((unsigned)per), lds, s, A);
    if ((st = check_launch("sign_binned: lookup"))) return st;
    if (horizon >= L.cap && walk_ratio <= 0.0) return POLYMH_OK;
    // the walk for polygons with a hash unresolved below the horizon, and
    // those left to it whole
    hipLaunchKernelGGL(k_unresolved_list, dim3(grid_for(L.n)), dim3(256), 0, s, w.unresolved, L.n, w.list, w.count);
    if ((st = check_launch("sign_binned: list"))) return st;
    SignLaunch W = L;
    W.order = w.list;
    W.n_dev = w.count;
    W.cfg.persistent = 1;
    // in a small launch the few polygons left to the walk are the costly
    // ones (many edges or deep hits) and set its duration: 8 hashes a work
    // item (one a wavefront) spread one polygon's hashes over many
    // workgroups (in a large launch that only multiplies the staging of the
    // many cheap walks of large polygons)
    if (units < 32768 && (W.cfg.hash_block <= 0 || W.cfg.hash_block > 8)) W.cfg.hash_block = 8;
    return launch_sign(W, s);
}

}  // namespace polymh
