// Ingest of a whole sampled block on the device: the index data of up to 32 small relations at once.
//
// A mini-batch block (Section 2.2 of the paper: the sampled k-hop neighbourhood, one bipartite graph per
// relation and hop) has a handful of relations of 10^3 .. 10^5 edges each.  The per-relation device
// pipeline costs twenty launches per relation, the host path a few hundred microseconds of CPU work and
// an upload (plus a download when the block was sampled on the device).  Here four launches build every
// relation of the block, from the caller's CSR to both schedules:
//
//   prep     rows: validation, offsets, 1/deg, degree counts; edges: validation, neighbour ids, the row of
//            every edge, counts per bucket of sources
//   spread   CSR rows placed by descending degree, their neighbours copied in that order; edges moved, stably,
//            to their buckets of sources
//   columns  a bucket's edges sorted, stably, by source in LDS: column offsets, the transpose's rows, degree counts
//   place    CSC rows placed like the CSR's
//
// What bounds it is latency: a launch is 4 to 8 us of a few dependent L2 accesses, whatever the block's size, and each
// launch after the first costs as much again in submission and gap.  So nothing is scanned over the whole block in a
// launch of its own: a relation has at most 64 or 128 workgroups a side, and each of them adds up the counts of all of
// them itself.  What a stage reads was mostly written by other XCDs a launch before and takes one to four microseconds to
// arrive: loads go in predicated rounds that are in flight together (a loop unrolled by 16 or 4 runs its remainder one load
// after the other), elements that two passes need stay in registers, and searches among row offsets are made by a
// wavefront, 64 places at a time, and then in LDS.  Whole calls for 14 relations of 2,000 / 5,000 / 40,000 edges: by the host path,
// with device arrays, 328 / 593 / 1,889 us; a chain of two radix sorts and two scans, 22 launches, 209 / 224 / 476; these
// four with the loads one by one 99 / 100 / 162, now 89 / 87 / 114.
//
// A relation's slice of every array is what the other ingest paths produce, bit for bit.  Everything is deterministic:
// integer atomics only count, every placement is by rank.  Where a workgroup of the first launch finds the caller's
// arrays malformed, the later launches leave that relation alone, and the fault is reported after the one
// synchronisation at the end; the first launch follows no offset or id that it has not clamped.
#include <algorithm>
#include <cstring>
#include <vector>

#include "heta_internal.h"

namespace heta {

namespace {

constexpr int kMaxBlockRels = 32;
constexpr int kRounds = 4;                    // elements per lane whose loads are in flight together
constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr int kMaxRowBlocks = 64;             // workgroups per relation over its destination rows, over its edges
constexpr int kMaxBuckets = 128;              // buckets of sources per relation
constexpr int kMaxRowsPer = 4096;             // rows per workgroup
constexpr int kMaxLow = 11;                   // a bucket holds 2^10 or 2^11 sources
constexpr int64_t kMaxElems = int64_t(1) << 18; // edges + rows of both sides of a relation: fewer (the caller's bound)
constexpr int kMaxHubs = kMaxElems / kHubMinDeg;
constexpr int kRowsInLds = 4096;              // offsets that a workgroup over edges searches in LDS
static_assert(kMaxElems <= int64_t(kMaxRowBlocks) * kMaxRowsPer && kMaxElems <= int64_t(kMaxBuckets) << kMaxLow, "a relation fits its workgroups");
static_assert(kMaxHubs <= 2 * kThreads, "hub rows of a workgroup: two per thread");
static_assert(kHubMinDeg == 2 * kThreads, "two degree buckets per thread beside the hubs'");

struct BlockPlan { // passed by value
    int n_rel;
    int32_t dst_off[kMaxBlockRels + 1], src_off[kMaxBlockRels + 1], edge_off[kMaxBlockRels + 1]; // a relation's rows and edges
    int32_t hub_off[2 * kMaxBlockRels + 1];    // chunk descriptors of schedule s (s < n_rel: CSR of relation s; else CSC of s - n_rel)
    int32_t hubptr_off[2 * kMaxBlockRels + 1]; // its chunk range array
    int32_t row_blk[kMaxBlockRels + 1], edge_blk[kMaxBlockRels + 1], src_blk[kMaxBlockRels + 1]; // a relation's workgroups
    int32_t rows_per[kMaxBlockRels], edges_per[kMaxBlockRels], low[kMaxBlockRels];               // elements of a workgroup; 2^low sources
    const int64_t *rowptr[kMaxBlockRels];
    const int32_t *col[kMaxBlockRels];
};

struct BlockBack { // per schedule, in page-locked host memory
    unsigned long long err; // CSR schedules
    uint32_t hub_edges, n_chunks;
    uint32_t rows[kDegHist + 1]; // rows of every capped degree
};

struct DegCounts { // of one workgroup's rows
    uint16_t rows[kHubMinDeg];
    uint32_t hub_rows, hub_edges, hub_chunks, pad;
};

struct BlockArrays { // passed by value
    // the arena; a relation's slice of an offset array has one more entry than rows
    int64_t *csr_ptr, *csr_sptr, *csc_ptr, *csc_sptr, *hub_chunk_ptr;
    HubChunk *hub_chunks;
    int32_t *csr_idx, *csr_sidx, *csc_idx, *csc_sidx, *csr_perm, *csc_perm;
    float *inv_deg;
    // scratch
    DegCounts *row_counts, *src_counts;   // per workgroup over rows / bucket
    uint16_t *bucket_counts;              // per workgroup over edges: kMaxBuckets
    uint32_t *bucket_start;               // per relation: kMaxBuckets + 1
    unsigned long long *err;              // per workgroup of the first launch
    uint32_t *row_of, *src_of;            // row of every CSR edge, source of every CSC edge
    uint2 *spread;                        // (source, row) by bucket
    BlockBack *back;
};

// largest i < n with off[i] <= x (off increasing, off[0] <= x)
__device__ __forceinline__ int seg_of(const int32_t *off, int n, int x)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// the last v in [lo, hi) with rp[v] <= x, lo if there is none
template <typename T> __device__ __forceinline__ int row_at(const T *rp, int lo, int hi, T x)
{
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (rp[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// the same by a whole wavefront, 64 places at a time: two or three accesses one after another instead of a dozen
__device__ __forceinline__ int row_at_wave(const int64_t *rp, int lo, int hi, int64_t x)
{
    const int lane = threadIdx.x & 63;
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64, at = lo + lane * step;
        const bool below = lane == 0 || (at < hi && rp[at] <= x);
        lo += (__popcll(__ballot(below)) - 1) * step; // malformed arrays: some place in [lo, hi) all the same
        hi = min(hi, lo + step);
    }
    return lo;
}

enum : unsigned long long { kBadPtr0 = 1, kBadDecrease = 2, kBadTotal = 3, kBadCol = 4 };

// An error word holds the complement of the smallest (kind, relation, position) reported, 0 while nothing is.
__device__ __forceinline__ void report(unsigned long long *err, unsigned long long kind, int rel, int64_t at)
{
    atomicMax(err, ~((kind << 56) | (static_cast<unsigned long long>(rel) << 48) | static_cast<unsigned long long>(at)));
}

// Inclusive sum over a wavefront by the vector ALU's data-parallel moves (a shuffle goes through the LDS): steps of 1, 2, 4
// and 8 within a row of 16 lanes, then the last lane of row 0 (2) into row 1 (3), and of row 1 into rows 2 and 3.
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t dpp_or_zero(uint32_t x)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x)
{
    x += dpp_or_zero<0x111, 0xf>(x);
    x += dpp_or_zero<0x112, 0xf>(x);
    x += dpp_or_zero<0x114, 0xf>(x);
    x += dpp_or_zero<0x118, 0xf>(x);
    x += dpp_or_zero<0x142, 0xa>(x);
    return x + dpp_or_zero<0x143, 0xc>(x);
}

// exclusive sums over the workgroup's threads of two values; lds: [2][kWaves]; every thread calls it
__device__ __forceinline__ uint2 block_scan2(uint32_t (*lds)[kWaves], uint32_t a, uint32_t b)
{
    const int w = threadIdx.x >> 6;
    uint32_t x = wave_sum(a), y = wave_sum(b);
    __syncthreads(); // earlier readers of lds
    if ((threadIdx.x & 63) == 63) {
        lds[0][w] = x;
        lds[1][w] = y;
    }
    __syncthreads();
    x -= a;
    y -= b;
    for (int q = 0; q < w; ++q) {
        x += lds[0][q];
        y += lds[1][q];
    }
    return make_uint2(x, y);
}

// Positions of this lane's elements of kRounds consecutive rounds among those of their buckets: the wavefront's counter of
// the bucket, plus the lanes below with the same bucket; advances the counters, whose updates a wavefront's LDS accesses
// take in order.  Whole wavefront.
__device__ __forceinline__ void stable_slots(uint32_t *cnt, const uint32_t (&bucket)[kRounds], const bool (&live)[kRounds], int bits,
                                             uint32_t (&at)[kRounds])
{
    unsigned long long same[kRounds];
    const unsigned long long lower = (1ull << (threadIdx.x & 63)) - 1;
#pragma unroll
    for (int u = 0; u < kRounds; ++u) same[u] = __ballot(live[u]);
    for (int b = 0; b < bits; ++b)
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const bool one = (bucket[u] >> b) & 1u;
            const unsigned long long ones = __ballot(one);
            same[u] &= one ? ones : ~ones;
        }
#pragma unroll
    for (int u = 0; u < kRounds; ++u) {
        at[u] = 0;
        if (live[u] && (same[u] & lower) == 0) at[u] = atomicAdd(&cnt[bucket[u]], static_cast<uint32_t>(__popcll(same[u])));
    }
#pragma unroll
    for (int u = 0; u < kRounds; ++u)
        at[u] = __shfl(at[u], live[u] ? __ffsll(same[u]) - 1 : 0, 64) + static_cast<uint32_t>(__popcll(same[u] & lower));
}

struct HistLds {
    uint32_t rows[kDegHist + 3];
    uint32_t hub_edges, hub_chunks;
};
__device__ __forceinline__ void hist_clear(HistLds &h)
{
    for (int k = threadIdx.x; k < kDegHist; k += kThreads) h.rows[k] = 0;
    if (threadIdx.x == 0) h.hub_edges = h.hub_chunks = 0;
}
__device__ __forceinline__ void hist_add(HistLds &h, uint32_t deg)
{
    atomicAdd(&h.rows[min(deg, static_cast<uint32_t>(kHubMinDeg))], 1u);
    if (deg >= kHubMinDeg) {
        atomicAdd(&h.hub_edges, deg);
        atomicAdd(&h.hub_chunks, (deg + kHubChunk - 1) / kHubChunk);
    }
}
__device__ __forceinline__ void hist_store(const HistLds &h, DegCounts *out)
{
    reinterpret_cast<uint32_t *>(out->rows)[threadIdx.x] = h.rows[2 * threadIdx.x] | (h.rows[2 * threadIdx.x + 1] << 16);
    if (threadIdx.x == 0) {
        out->hub_rows = h.rows[kHubMinDeg];
        out->hub_edges = h.hub_edges;
        out->hub_chunks = h.hub_chunks;
    }
}

// ---- first launch ---------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) blk_prep_kernel(BlockPlan p, BlockArrays a)
{
    __shared__ HistLds hist;
    __shared__ uint32_t buckets[kMaxBuckets];
    __shared__ unsigned long long err;
    __shared__ int first_row, last_row;
    __shared__ int32_t starts[kRowsInLds];
    const int tid = threadIdx.x, row_blocks = p.row_blk[p.n_rel];
    const bool rows = static_cast<int>(blockIdx.x) < row_blocks;
    const int blk = rows ? blockIdx.x : blockIdx.x - row_blocks;
    const int rel = seg_of(rows ? p.row_blk : p.edge_blk, p.n_rel, blk);
    const int n_dst = p.dst_off[rel + 1] - p.dst_off[rel], n_src = p.src_off[rel + 1] - p.src_off[rel], E = p.edge_off[rel + 1] - p.edge_off[rel];
    const int64_t *rp = p.rowptr[rel];
    if (tid == 0) err = 0;
    if (rows) {
        const int lo = (blk - p.row_blk[rel]) * p.rows_per[rel], hi = min(n_dst, lo + p.rows_per[rel]);
        int64_t *ptr = a.csr_ptr + p.dst_off[rel] + rel;
        float *inv_deg = a.inv_deg + p.dst_off[rel];
        hist_clear(hist);
        __syncthreads();
        for (int v = lo + tid; v < hi; v += kThreads) {
            const int64_t r0 = rp[v], r1 = rp[v + 1], deg = r1 - r0;
            if (v == 0 && r0 != 0) report(&err, kBadPtr0, rel, 0);
            if (r1 < r0) report(&err, kBadDecrease, rel, v);
            if (v == n_dst - 1 && r1 != E) report(&err, kBadTotal, rel, 0);
            ptr[v] = r0;
            inv_deg[v] = deg > 0 ? 1.0f / static_cast<float>(deg) : 0.0f;
            hist_add(hist, static_cast<uint32_t>(min(max(deg, static_cast<int64_t>(0)), static_cast<int64_t>(E))));
        }
        if (tid == 0 && hi == n_dst) ptr[n_dst] = E;
        if (tid == 0 && n_dst == 0 && rp[0] != 0) report(&err, kBadPtr0, rel, 0);
        __syncthreads();
        hist_store(hist, a.row_counts + blk);
    } else {
        const int lo = (blk - p.edge_blk[rel]) * p.edges_per[rel], hi = min(E, lo + p.edges_per[rel]), low = p.low[rel];
        const int32_t *col = p.col[rel];
        int32_t *idx = a.csr_idx + p.edge_off[rel];
        uint32_t *row_of = a.row_of + p.edge_off[rel];
        if (tid < kMaxBuckets) buckets[tid] = 0;
        int32_t c[kRounds];
        const auto load = [&](int e0) { // all of a round in flight together
#pragma unroll
            for (int u = 0; u < kRounds; ++u) c[u] = e0 + u * kThreads < hi ? col[e0 + u * kThreads] : 0;
        };
        load(lo + tid);
        if (lo < hi) { // uniform; n_dst > 0
            const int w = tid >> 6;
            if (w < 2) {
                const int r = row_at_wave(rp, 0, n_dst, w == 0 ? lo : hi - 1);
                if ((tid & 63) == 0) (w == 0 ? first_row : last_row) = r;
            }
        }
        __syncthreads();
        const int row0 = first_row, n_rows = lo < hi ? last_row + 1 - row0 : 0;
        const bool in_lds = n_rows <= kRowsInLds; // uniform (malformed offsets: no rows, or some within [0, n_dst))
        if (in_lds) {
            for (int v0 = tid; v0 < n_rows; v0 += kRounds * kThreads) {
                int64_t r[kRounds];
#pragma unroll
                for (int u = 0; u < kRounds; ++u) r[u] = v0 + u * kThreads < n_rows ? rp[row0 + v0 + u * kThreads] : 0;
#pragma unroll
                for (int u = 0; u < kRounds; ++u)
                    if (v0 + u * kThreads < n_rows) starts[v0 + u * kThreads] = static_cast<int32_t>(min(r[u], static_cast<int64_t>(E) + 1));
            }
            __syncthreads();
        }
        for (int e0 = lo + tid; e0 < hi; e0 += kRounds * kThreads) {
            if (e0 != lo + tid) load(e0);
#pragma unroll
            for (int u = 0; u < kRounds; ++u) {
                const int e = e0 + u * kThreads;
                if (e >= hi) continue;
                if (c[u] < 0 || c[u] >= n_src) {
                    report(&err, kBadCol, rel, e);
                    c[u] = 0;
                }
                idx[e] = c[u];
                row_of[e] = static_cast<uint32_t>(in_lds ? row0 + row_at(starts, 0, n_rows, e) : row_at(rp, row0, row0 + n_rows, static_cast<int64_t>(e)));
                atomicAdd(&buckets[c[u] >> low], 1u);
            }
        }
        __syncthreads();
        if (tid < kMaxBuckets) a.bucket_counts[static_cast<int64_t>(blk) * kMaxBuckets + tid] = static_cast<uint16_t>(buckets[tid]);
    }
    if (tid == 0) a.err[blockIdx.x] = err;
}

// Whether the first launch found relation `rel` malformed; `word` (one workgroup's pointer, else null) takes the fault or 0.
__device__ __forceinline__ bool faulty(const BlockPlan &p, const BlockArrays &a, int rel, unsigned long long *word)
{
    const int row_blocks = p.row_blk[p.n_rel], nr = p.row_blk[rel + 1] - p.row_blk[rel], ne = p.edge_blk[rel + 1] - p.edge_blk[rel];
    unsigned long long mine = 0; // nr + ne <= 2 kMaxRowBlocks <= kThreads
    if (static_cast<int>(threadIdx.x) < nr + ne)
        mine = a.err[static_cast<int>(threadIdx.x) < nr ? p.row_blk[rel] + threadIdx.x : row_blocks + p.edge_blk[rel] + threadIdx.x - nr];
    const bool bad = __syncthreads_or(mine != 0);
    if (word && threadIdx.x == 0) {
        unsigned long long all = 0;
        if (bad)
            for (int i = 0; i < nr + ne; ++i) all = max(all, a.err[i < nr ? p.row_blk[rel] + i : row_blocks + p.edge_blk[rel] + i - nr]);
        *word = all;
    }
    return bad;
}

struct PlaceLds {
    uint32_t cnt[kWaves][kDegHist + 3];
    uint32_t rows_ge[kDegHist + 1], edges_ge[kDegHist + 1]; // rows / edges of degree >= k in the relation
    uint32_t delta[kMaxRowsPer]; // schedule position of a row's first edge minus its position by row id
    uint32_t hub_row[kMaxHubs];
    uint32_t scan[2][kWaves];
    uint32_t hub[2][3]; // rows, edges, chunks of hub rows: of the relation, of the workgroups before this one
    uint32_t max_deg;
};

// The rows [lo, hi) of one direction of a relation, placed in its schedule: rows by descending capped degree (stable),
// schedule-ordered offsets and neighbours, hub chunks.  counts: of the relation's nb workgroups, this one is the b-th;
// per: rows per workgroup.  Below the hub degree a row's offset follows from its degree's start and its position.
__device__ __forceinline__ void place_rows(PlaceLds &L, int n, int lo, int hi, int per, int E, const int64_t *ptr, const int32_t *idx,
                                           const uint32_t *row_of, int32_t *perm, int64_t *sptr, int32_t *sidx, int64_t *hub_chunk_ptr,
                                           HubChunk *hub_chunks, const DegCounts *counts, int nb, int b, BlockBack *back)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int share = per / kWaves; // a multiple of 64
    const int wlo = lo + w * share, whi = min(hi, wlo + share);
    uint32_t p0[kRounds], deg[kRounds];
    const auto load_rows = [&](int i0) {
        uint32_t p1[kRounds];
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int v = i0 + 64 * u + lane;
            p0[u] = v < whi ? static_cast<uint32_t>(ptr[v]) : 0;
            p1[u] = v < whi ? static_cast<uint32_t>(ptr[v + 1]) : 0;
        }
#pragma unroll
        for (int u = 0; u < kRounds; ++u) deg[u] = p1[u] - p0[u];
    };
    load_rows(wlo);
    for (int i = tid; i < kWaves * (kDegHist + 3); i += kThreads) (&L.cnt[0][0])[i] = 0;
    if (tid < 6) L.hub[tid / 3][tid % 3] = 0;
    if (tid == 6) L.max_deg = 0;
    // thread t: degrees 2 j and 2 j + 1 with j = 255 - t, over all workgroups and over those before this one
    const int j = kThreads - 1 - tid;
    uint32_t total0 = 0, total1 = 0, before0 = 0, before1 = 0;
    uint32_t rows = 0, edges = 0, chunks = 0;
    if (tid < nb) { // nb <= kThreads
        rows = counts[tid].hub_rows;
        edges = counts[tid].hub_edges;
        chunks = counts[tid].hub_chunks;
    }
    for (int q0 = 0; q0 < nb; q0 += 16) {
        uint32_t c[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) c[i] = q0 + i < nb ? reinterpret_cast<const uint32_t *>(counts[q0 + i].rows)[j] : 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            total0 += c[i] & 0xffffu;
            total1 += c[i] >> 16;
            before0 += q0 + i < b ? c[i] & 0xffffu : 0;
            before1 += q0 + i < b ? c[i] >> 16 : 0;
        }
    }
    __syncthreads();
    if (rows > 0) {
        for (int i = 0; i < (tid < b ? 2 : 1); ++i) {
            atomicAdd(&L.hub[i][0], rows);
            atomicAdd(&L.hub[i][1], edges);
            atomicAdd(&L.hub[i][2], chunks);
        }
    }
    uint32_t most = 0;
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        if (i0 != wlo) load_rows(i0);
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            if (i0 + 64 * u + lane >= whi) continue;
            const uint32_t k = min(deg[u], static_cast<uint32_t>(kHubMinDeg));
            atomicAdd(&L.cnt[w][k], 1u);
            most = max(most, k);
        }
    }
    atomicMax(&L.max_deg, most);
    const uint32_t k0 = 2 * j, k1 = k0 + 1;
    const uint2 above = block_scan2(L.scan, total0 + total1, total0 * k0 + total1 * k1); // its barriers come after the last count
    const uint32_t hub_rows = L.hub[0][0], hub_edges = L.hub[0][1], hubs_before = L.hub[1][0], hub_edges_before = L.hub[1][1], chunks_before = L.hub[1][2];
    const uint32_t rows1 = hub_rows + above.x, edges1 = hub_edges + above.y; // of degrees above k1
    L.rows_ge[k1] = rows1 + total1;
    L.edges_ge[k1] = edges1 + total1 * k1;
    L.rows_ge[k0] = rows1 + total1 + total0;
    L.edges_ge[k0] = edges1 + total1 * k1 + total0 * k0;
    uint32_t run0 = rows1 + total1 + before0, run1 = rows1 + before1;
    for (int q = 0; q < kWaves; ++q) {
        const uint32_t c0 = L.cnt[q][k0], c1 = L.cnt[q][k1];
        L.cnt[q][k0] = run0;
        L.cnt[q][k1] = run1;
        run0 += c0;
        run1 += c1;
    }
    if (tid == 0) {
        L.rows_ge[kHubMinDeg] = hub_rows;
        L.edges_ge[kHubMinDeg] = hub_edges;
        uint32_t run = hubs_before;
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t c = L.cnt[q][kHubMinDeg];
            L.cnt[q][kHubMinDeg] = run;
            run += c;
        }
    }
    if (b == 0) { // uniform
        back->rows[k0] = total0;
        back->rows[k1] = total1;
        if (tid == 0) {
            back->rows[kHubMinDeg] = hub_rows;
            back->hub_edges = hub_edges;
            back->n_chunks = L.hub[0][2];
            hub_chunk_ptr[hub_rows] = L.hub[0][2];
            sptr[n] = E;
        }
    }
    __syncthreads();
    const int bits = 32 - __clz(static_cast<int>(L.max_deg)); // 0 where every row is empty
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        uint32_t k[kRounds], at[kRounds];
        bool live[kRounds];
        if (whi - wlo > 64 * kRounds) load_rows(i0); // else they are still there
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            live[u] = i0 + 64 * u + lane < whi;
            k[u] = live[u] ? min(deg[u], static_cast<uint32_t>(kHubMinDeg)) : 0;
        }
        stable_slots(L.cnt[w], k, live, bits, at);
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            if (!live[u]) continue;
            const int v = i0 + 64 * u + lane;
            perm[at[u]] = v;
            if (k[u] < kHubMinDeg) {
                const uint32_t s = L.edges_ge[k[u] + 1] + (at[u] - L.rows_ge[k[u] + 1]) * k[u];
                sptr[at[u]] = s;
                L.delta[v - lo] = s - p0[u];
            } else {
                L.hub_row[at[u] - hubs_before] = static_cast<uint32_t>(v);
            }
        }
    }
    __syncthreads();
    const int n_hubs = static_cast<int>(counts[b].hub_rows);
    if (n_hubs > 0) { // uniform; two hub rows per thread
        uint32_t v[2] = {0, 0}, hub_deg[2] = {0, 0}, nc[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (2 * tid + i < n_hubs) {
                v[i] = L.hub_row[2 * tid + i];
                hub_deg[i] = static_cast<uint32_t>(ptr[v[i] + 1] - ptr[v[i]]);
            }
            nc[i] = (hub_deg[i] + kHubChunk - 1) / kHubChunk;
        }
        const uint2 first = block_scan2(L.scan, hub_deg[0] + hub_deg[1], nc[0] + nc[1]);
        uint32_t s = hub_edges_before + first.x, c0 = chunks_before + first.y;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (2 * tid + i < n_hubs) {
                const uint32_t q = hubs_before + 2 * tid + i;
                sptr[q] = s;
                hub_chunk_ptr[q] = c0;
                L.delta[v[i] - lo] = s - static_cast<uint32_t>(ptr[v[i]]);
                for (uint32_t c = 0; c < nc[i]; ++c) {
                    HubChunk d;
                    d.e0 = s + c * kHubChunk;
                    d.len = static_cast<int32_t>(min(static_cast<uint32_t>(kHubChunk), hub_deg[i] - c * kHubChunk));
                    d.slot = static_cast<int32_t>(c0 + c);
                    hub_chunks[c0 + c] = d;
                }
            }
            s += hub_deg[i];
            c0 += nc[i];
        }
        __syncthreads();
    }
    if (lo >= hi) return;
    const int e0 = static_cast<int>(ptr[lo]), e1 = static_cast<int>(ptr[hi]);
    for (int i0 = e0 + tid; i0 < e1; i0 += kRounds * kThreads) {
        uint32_t row[kRounds];
        int32_t nbr[kRounds];
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int e = i0 + u * kThreads;
            row[u] = e < e1 ? row_of[e] : 0;
            nbr[u] = e < e1 ? idx[e] : 0;
        }
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int e = i0 + u * kThreads;
            if (e < e1) sidx[e + L.delta[row[u] - lo]] = nbr[u];
        }
    }
}

// ---- second launch --------------------------------------------------------------------------------------------------
// A workgroup's edges moved to their buckets of sources: position = start of the bucket + edges of it in earlier
// workgroups, wavefronts, rounds and lanes.
struct SpreadLds {
    uint32_t cnt[kWaves][kMaxBuckets];
    uint32_t scan[2][kWaves];
};

__device__ __forceinline__ void spread_edges(SpreadLds &L, const BlockPlan &p, const BlockArrays &a, int rel, int b)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int E = p.edge_off[rel + 1] - p.edge_off[rel], n_src = p.src_off[rel + 1] - p.src_off[rel], low = p.low[rel];
    const int nb = p.edge_blk[rel + 1] - p.edge_blk[rel], per = p.edges_per[rel], share = per / kWaves;
    const int lo = b * per, hi = min(E, lo + per), wlo = lo + w * share, whi = min(hi, wlo + share);
    const int32_t *idx = a.csr_idx + p.edge_off[rel];
    const uint32_t *row_of = a.row_of + p.edge_off[rel];
    uint2 *out = a.spread + p.edge_off[rel];
    const uint16_t *counts = a.bucket_counts + static_cast<int64_t>(p.edge_blk[rel]) * kMaxBuckets;
    uint32_t c[kRounds], row[kRounds];
    const auto load = [&](int i0) {
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            const int e = i0 + 64 * u + lane;
            c[u] = e < whi ? static_cast<uint32_t>(idx[e]) : 0;
            row[u] = e < whi ? row_of[e] : 0;
        }
    };
    load(wlo);
    for (int i = tid; i < kWaves * kMaxBuckets; i += kThreads) (&L.cnt[0][0])[i] = 0;
    uint32_t total = 0, before = 0;
    if (tid < kMaxBuckets) {
        for (int q0 = 0; q0 < nb; q0 += 16) {
            uint32_t n[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) n[i] = q0 + i < nb ? counts[(q0 + i) * kMaxBuckets + tid] : 0;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                total += n[i];
                before += q0 + i < b ? n[i] : 0;
            }
        }
    }
    __syncthreads();
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        if (i0 != wlo) load(i0);
#pragma unroll
        for (int u = 0; u < kRounds; ++u)
            if (i0 + 64 * u + lane < whi) atomicAdd(&L.cnt[w][c[u] >> low], 1u);
    }
    const uint32_t start = block_scan2(L.scan, total, 0).x; // its barriers come after the last count
    if (tid < kMaxBuckets) {
        uint32_t run = start + before;
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t c = L.cnt[q][tid];
            L.cnt[q][tid] = run;
            run += c;
        }
        if (b == 0) {
            uint32_t *bs = a.bucket_start + rel * (kMaxBuckets + 1);
            bs[tid] = start;
            if (tid == kMaxBuckets - 1) bs[kMaxBuckets] = E;
        }
    }
    __syncthreads();
    int bits = 0;
    while ((n_src - 1) >> (low + bits) > 0) ++bits;
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        uint32_t bucket[kRounds], at[kRounds];
        bool live[kRounds];
        if (whi - wlo > 64 * kRounds) load(i0); // else they are still there
#pragma unroll
        for (int u = 0; u < kRounds; ++u) {
            live[u] = i0 + 64 * u + lane < whi;
            bucket[u] = c[u] >> low;
        }
        stable_slots(L.cnt[w], bucket, live, bits, at);
#pragma unroll
        for (int u = 0; u < kRounds; ++u)
            if (live[u]) out[at[u]] = make_uint2(c[u], row[u]);
    }
}

__global__ void __launch_bounds__(kThreads) blk_spread_kernel(BlockPlan p, BlockArrays a)
{
    __shared__ union {
        PlaceLds place;
        SpreadLds spread;
    } L;
    const int row_blocks = p.row_blk[p.n_rel];
    const bool rows = static_cast<int>(blockIdx.x) < row_blocks;
    const int blk = rows ? blockIdx.x : blockIdx.x - row_blocks;
    const int rel = seg_of(rows ? p.row_blk : p.edge_blk, p.n_rel, blk);
    const int b = blk - (rows ? p.row_blk : p.edge_blk)[rel];
    if (faulty(p, a, rel, rows && b == 0 ? &a.back[rel].err : nullptr)) return; // uniform
    if (!rows) {
        spread_edges(L.spread, p, a, rel, b);
        return;
    }
    const int n = p.dst_off[rel + 1] - p.dst_off[rel], per = p.rows_per[rel], lo = b * per;
    place_rows(L.place, n, lo, min(n, lo + per), per, p.edge_off[rel + 1] - p.edge_off[rel], a.csr_ptr + p.dst_off[rel] + rel, a.csr_idx + p.edge_off[rel],
               a.row_of + p.edge_off[rel], a.csr_perm + p.dst_off[rel], a.csr_sptr + p.dst_off[rel] + rel, a.csr_sidx + p.edge_off[rel],
               a.hub_chunk_ptr + p.hubptr_off[rel], a.hub_chunks + p.hub_off[rel], a.row_counts + p.row_blk[rel], p.row_blk[rel + 1] - p.row_blk[rel], b,
               a.back + rel);
}

// ---- third launch: one workgroup per bucket of sources -----------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) blk_columns_kernel(BlockPlan p, BlockArrays a)
{
    constexpr int SRC = 1 << kMaxLow, PER = SRC / kThreads;
    __shared__ uint32_t cnt[kWaves][SRC];
    __shared__ uint32_t scan[2][kWaves];
    __shared__ HistLds hist;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int rel = seg_of(p.src_blk, p.n_rel, blockIdx.x), b = blockIdx.x - p.src_blk[rel];
    if (faulty(p, a, rel, nullptr)) return; // uniform
    const int n_src = p.src_off[rel + 1] - p.src_off[rel], low = p.low[rel], u0 = b << low, n = min(n_src - u0, 1 << low);
    const uint32_t *bs = a.bucket_start + rel * (kMaxBuckets + 1);
    const int e0 = static_cast<int>(bs[b]), m = static_cast<int>(bs[b + 1]) - e0;
    const int share = (m + kThreads - 1) / kThreads * 64, wlo = w * share, whi = min(m, wlo + share);
    const uint2 *in = a.spread + p.edge_off[rel] + e0;
    int64_t *ptr = a.csc_ptr + p.src_off[rel] + rel;
    int32_t *idx = a.csc_idx + p.edge_off[rel] + e0;
    uint32_t *src_of = a.src_of + p.edge_off[rel] + e0;
    uint2 pair[kRounds];
    const auto load = [&](int i0) {
#pragma unroll
        for (int r = 0; r < kRounds; ++r) pair[r] = i0 + 64 * r + lane < whi ? in[i0 + 64 * r + lane] : make_uint2(u0, 0);
    };
    load(wlo);
    for (int i = tid; i < kWaves * SRC; i += kThreads) (&cnt[0][0])[i] = 0;
    hist_clear(hist);
    __syncthreads();
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        if (i0 != wlo) load(i0);
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            if (i0 + 64 * r + lane < whi) atomicAdd(&cnt[w][pair[r].x - u0], 1u);
    }
    __syncthreads();
    uint32_t deg[PER], sum = 0; // PER consecutive sources per thread
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int u = tid * PER + k;
        deg[k] = 0;
        for (int q = 0; q < kWaves; ++q) deg[k] += cnt[q][u];
        sum += deg[k];
        if (u < n) hist_add(hist, deg[k]);
    }
    uint32_t at0 = block_scan2(scan, sum, 0).x;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int u = tid * PER + k;
        if (u < n) ptr[u0 + u] = e0 + at0;
        uint32_t run = at0;
        for (int q = 0; q < kWaves; ++q) {
            const uint32_t c = cnt[q][u];
            cnt[q][u] = run;
            run += c;
        }
        at0 = run;
    }
    if (tid == 0 && u0 + n == n_src) ptr[n_src] = p.edge_off[rel + 1] - p.edge_off[rel];
    __syncthreads();
    hist_store(hist, a.src_counts + blockIdx.x);
    for (int i0 = wlo; i0 < whi; i0 += 64 * kRounds) { // uniform per wavefront
        uint32_t u[kRounds], at[kRounds];
        bool live[kRounds];
        if (whi - wlo > 64 * kRounds) load(i0); // else they are still there
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            live[r] = i0 + 64 * r + lane < whi;
            u[r] = pair[r].x - u0;
        }
        stable_slots(cnt[w], u, live, low, at);
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            if (live[r]) {
                idx[at[r]] = static_cast<int32_t>(pair[r].y);
                src_of[at[r]] = pair[r].x;
            }
    }
}

// ---- fourth launch ------------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) blk_place_kernel(BlockPlan p, BlockArrays a)
{
    __shared__ PlaceLds L;
    const int rel = seg_of(p.src_blk, p.n_rel, blockIdx.x), b = blockIdx.x - p.src_blk[rel], sched = p.n_rel + rel;
    if (faulty(p, a, rel, nullptr)) return; // uniform
    const int n = p.src_off[rel + 1] - p.src_off[rel], per = 1 << p.low[rel], lo = b * per;
    place_rows(L, n, lo, min(n, lo + per), per, p.edge_off[rel + 1] - p.edge_off[rel], a.csc_ptr + p.src_off[rel] + rel, a.csc_idx + p.edge_off[rel],
               a.src_of + p.edge_off[rel], a.csc_perm + p.src_off[rel], a.csc_sptr + p.src_off[rel] + rel, a.csc_sidx + p.edge_off[rel],
               a.hub_chunk_ptr + p.hubptr_off[sched], a.hub_chunks + p.hub_off[sched], a.src_counts + p.src_blk[rel],
               p.src_blk[rel + 1] - p.src_blk[rel], b, a.back + sched);
}

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

template <typename T> T *carve(char *&cursor, size_t n)
{
    T *p = reinterpret_cast<T *>(cursor);
    cursor += align_up(std::max<size_t>(n, 1) * sizeof(T), 256);
    return p;
}

template <typename T> size_t carve_size(size_t n) { return align_up(std::max<size_t>(n, 1) * sizeof(T), 256); }

// the message of an error word left by `report`
heta_status malformed(unsigned long long word, const std::vector<Relation *> &rels, const std::vector<std::string> &names)
{
    const unsigned long long bad = ~word, kind = bad >> 56, at = bad & ((1ull << 48) - 1);
    const int which = static_cast<int>((bad >> 48) & 0xff);
    const Relation &r = *rels[which];
    const char *name = names[which].c_str();
    if (kind == kBadPtr0) return fail(HETA_ERR_BAD_CSR, "%s: rowptr[0] is not 0", name);
    if (kind == kBadDecrease) return fail(HETA_ERR_BAD_CSR, "%s: rowptr decreases at row %llu", name, at);
    if (kind == kBadTotal) return fail(HETA_ERR_BAD_CSR, "%s: rowptr[n_dst] differs from num_edges = %lld", name, (long long)r.n_edges);
    return fail(HETA_ERR_BAD_CSR, "%s: col[%llu] outside [0, %lld)", name, at, (long long)r.n_src);
}

} // namespace

int block_ingest_max_relations() { return kMaxBlockRels; }

// Builds the listed relations (registered already in their graphs: types, sizes; no arrays yet) from their CSRs;
// `names` says how an error message calls each.
// rowptr / col: DEVICE arrays per listed relation.  On success the relations' schedules point into *arena_out
// (one pool block, to be released with scratch_free when the graph goes) and carry their host-side histograms.
// Synchronous.
heta_status build_block_on_device(const std::vector<Relation *> &rels, const std::vector<std::string> &names,
                                  const int64_t *const *rowptr, const int32_t *const *col, void **arena_out, hipStream_t st)
{
    *arena_out = nullptr;
    const int n_rel = static_cast<int>(rels.size());
    if (n_rel == 0) return HETA_OK;
    if (n_rel > kMaxBlockRels) return fail(HETA_ERR_UNSUPPORTED, "block ingest takes at most %d relations at once", kMaxBlockRels);
    BlockPlan p{};
    p.n_rel = n_rel;
    for (int i = 0; i < n_rel; ++i) { // what needs no look at the arrays is rejected before anything is launched
        const Relation &r = *rels[i];
        if (r.n_edges > 0 && r.n_dst == 0)
            return fail(HETA_ERR_BAD_CSR, "%s: rowptr[n_dst] differs from num_edges = %lld", names[i].c_str(), (long long)r.n_edges);
        if (r.n_edges > 0 && r.n_src == 0) return fail(HETA_ERR_BAD_CSR, "%s: col[0] outside [0, 0)", names[i].c_str());
        if (r.n_edges + r.n_dst + r.n_src >= kMaxElems) return fail(HETA_ERR_UNSUPPORTED, "%s: too large for the block ingest", names[i].c_str());
        p.dst_off[i + 1] = p.dst_off[i] + static_cast<int32_t>(r.n_dst);
        p.src_off[i + 1] = p.src_off[i] + static_cast<int32_t>(r.n_src);
        p.edge_off[i + 1] = p.edge_off[i] + static_cast<int32_t>(r.n_edges);
        // one workgroup at least on every side: it writes what a relation without rows has, too
        const auto per = [](int64_t n, int64_t least) { return static_cast<int32_t>(std::max<int64_t>(least, ((n + kMaxRowBlocks - 1) / kMaxRowBlocks + 255) / 256 * 256)); };
        const auto blocks = [](int64_t n, int64_t each) { return static_cast<int32_t>(std::max<int64_t>(1, (n + each - 1) / each)); };
        p.rows_per[i] = per(r.n_dst, 256);
        p.edges_per[i] = per(r.n_edges, 1024);
        p.low[i] = r.n_src <= (int64_t(kMaxBuckets) << 9) ? 10 : kMaxLow;
        p.row_blk[i + 1] = p.row_blk[i] + blocks(r.n_dst, p.rows_per[i]);
        p.edge_blk[i + 1] = p.edge_blk[i] + blocks(r.n_edges, p.edges_per[i]);
        p.src_blk[i + 1] = p.src_blk[i] + blocks(r.n_src, int64_t(1) << p.low[i]);
        p.rowptr[i] = rowptr[i];
        p.col[i] = col[i];
    }
    for (int s = 0; s < 2 * n_rel; ++s) { // chunk descriptors / chunk ranges per schedule: the same bounds as the host path's
        const int32_t E = static_cast<int32_t>(rels[s % n_rel]->n_edges);
        p.hub_off[s + 1] = p.hub_off[s] + E / kHubChunk + E / kHubMinDeg + 1;
        p.hubptr_off[s + 1] = p.hubptr_off[s] + E / kHubMinDeg + 2;
    }
    const int64_t nR = p.dst_off[n_rel], nS = p.src_off[n_rel], nE = p.edge_off[n_rel];

    // ---- the arena: everything the relations keep ------------------------------------------------------
    const size_t n_hub = p.hub_off[2 * n_rel], n_hubptr = p.hubptr_off[2 * n_rel];
    const size_t arena_bytes = 2 * carve_size<int64_t>(nR + n_rel) + 2 * carve_size<int64_t>(nS + n_rel) + carve_size<int64_t>(n_hubptr) +
                               carve_size<HubChunk>(n_hub) + 4 * carve_size<int32_t>(nE) + carve_size<int32_t>(nR) +
                               carve_size<int32_t>(nS) + carve_size<float>(nR);
    void *arena = nullptr;
    HETA_HIP(scratch_alloc(&arena, arena_bytes));
    BlockArrays a{};
    char *cur = static_cast<char *>(arena);
    a.csr_ptr = carve<int64_t>(cur, nR + n_rel);
    a.csr_sptr = carve<int64_t>(cur, nR + n_rel);
    a.csc_ptr = carve<int64_t>(cur, nS + n_rel);
    a.csc_sptr = carve<int64_t>(cur, nS + n_rel);
    a.hub_chunk_ptr = carve<int64_t>(cur, n_hubptr);
    a.hub_chunks = carve<HubChunk>(cur, n_hub);
    a.csr_idx = carve<int32_t>(cur, nE);
    a.csr_sidx = carve<int32_t>(cur, nE);
    a.csc_idx = carve<int32_t>(cur, nE);
    a.csc_sidx = carve<int32_t>(cur, nE);
    a.csr_perm = carve<int32_t>(cur, nR);
    a.csc_perm = carve<int32_t>(cur, nS);
    a.inv_deg = carve<float>(cur, nR);

    // ---- scratch: one pool block, and the page-locked results of this thread (written by the kernels: no copy) ----
    const size_t row_blocks = p.row_blk[n_rel], edge_blocks = p.edge_blk[n_rel], src_blocks = p.src_blk[n_rel];
    const size_t scratch_bytes = carve_size<DegCounts>(row_blocks) + carve_size<DegCounts>(src_blocks) +
                                 carve_size<uint16_t>(edge_blocks * kMaxBuckets) + carve_size<uint32_t>(n_rel * (kMaxBuckets + 1)) +
                                 carve_size<unsigned long long>(row_blocks + edge_blocks) + 2 * carve_size<uint32_t>(nE) + carve_size<uint2>(nE);
    static thread_local BlockBack *t_back = nullptr; // never freed: it lives as long as the thread builds graphs
    void *scratch = nullptr, *back = nullptr;
    hipError_t e = t_back ? hipSuccess : hipHostMalloc(&back, 2 * kMaxBlockRels * sizeof(BlockBack), hipHostMallocPortable | hipHostMallocMapped);
    if (back) t_back = static_cast<BlockBack *>(back);
    if (e == hipSuccess) e = scratch_alloc(&scratch, scratch_bytes);
    if (e != hipSuccess) {
        scratch_free(arena);
        return fail(e == hipErrorOutOfMemory ? HETA_ERR_OOM : HETA_ERR_DEVICE, "block ingest: %s", hipGetErrorString(e));
    }
    cur = static_cast<char *>(scratch);
    a.row_counts = carve<DegCounts>(cur, row_blocks);
    a.src_counts = carve<DegCounts>(cur, src_blocks);
    a.bucket_counts = carve<uint16_t>(cur, edge_blocks * kMaxBuckets);
    a.bucket_start = carve<uint32_t>(cur, n_rel * (kMaxBuckets + 1));
    a.err = carve<unsigned long long>(cur, row_blocks + edge_blocks);
    a.row_of = carve<uint32_t>(cur, nE);
    a.src_of = carve<uint32_t>(cur, nE);
    a.spread = carve<uint2>(cur, nE);
    a.back = t_back;

    const char *name = "blk_prep_kernel";
    hipLaunchKernelGGL(blk_prep_kernel, dim3(row_blocks + edge_blocks), dim3(kThreads), 0, st, p, a);
    if ((e = hipGetLastError()) == hipSuccess) {
        name = "blk_spread_kernel";
        hipLaunchKernelGGL(blk_spread_kernel, dim3(row_blocks + edge_blocks), dim3(kThreads), 0, st, p, a);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        name = "blk_columns_kernel";
        hipLaunchKernelGGL(blk_columns_kernel, dim3(src_blocks), dim3(kThreads), 0, st, p, a);
        e = hipGetLastError();
    }
    if (e == hipSuccess) {
        name = "blk_place_kernel";
        hipLaunchKernelGGL(blk_place_kernel, dim3(src_blocks), dim3(kThreads), 0, st, p, a);
        e = hipGetLastError();
    }
    const hipError_t done = hipStreamSynchronize(st);
    scratch_free(scratch); // idle
    heta_status status = HETA_OK;
    if (e != hipSuccess) status = fail(HETA_ERR_DEVICE, "launch of %s failed: %s", name, hipGetErrorString(e));
    else if (done != hipSuccess) status = fail(HETA_ERR_DEVICE, "block ingest: %s", hipGetErrorString(done));
    else {
        unsigned long long err = 0; // complements: the largest is the first fault
        for (int i = 0; i < n_rel; ++i) err = std::max(err, t_back[i].err);
        if (err) status = malformed(err, rels, names);
    }
    if (status != HETA_OK) {
        scratch_free(arena);
        return status;
    }
    for (int i = 0; i < n_rel; ++i) {
        Relation &r = *rels[i];
        for (int side = 0; side < 2; ++side) {
            Schedule &s = side ? r.csc : r.csr;
            const int sched = side ? n_rel + i : i;
            const int32_t row0 = side ? p.src_off[i] : p.dst_off[i];
            s.d_ptr = (side ? a.csc_ptr : a.csr_ptr) + row0 + i;
            s.d_sptr = (side ? a.csc_sptr : a.csr_sptr) + row0 + i;
            s.d_idx = (side ? a.csc_idx : a.csr_idx) + p.edge_off[i];
            s.d_sidx = (side ? a.csc_sidx : a.csr_sidx) + p.edge_off[i];
            s.d_perm = (side ? a.csc_perm : a.csr_perm) + row0;
            s.d_hub_chunks = a.hub_chunks + p.hub_off[sched];
            s.d_hub_chunk_ptr = a.hub_chunk_ptr + p.hubptr_off[sched];
            const BlockBack &h = t_back[sched];
            int64_t rows = 0, edges = 0;
            for (int k = kHubMinDeg; k >= 0; --k) {
                rows += h.rows[k];
                edges += k == kHubMinDeg ? static_cast<int64_t>(h.hub_edges) : static_cast<int64_t>(h.rows[k]) * k;
                s.rows_with_deg_ge[k] = rows;
                s.edges_with_deg_ge[k] = edges;
            }
            s.n_hub_rows = s.rows_with_deg_ge[kHubMinDeg];
            s.n_hub_chunks = h.n_chunks;
        }
        r.d_inv_deg = a.inv_deg + p.dst_off[i];
        r.host_built = true; // its arrays are slices of an arena of the graph, not allocations of its own
    }
    *arena_out = arena;
    return HETA_OK;
}

} // namespace heta
