// k-hop neighbour sampling on the device (Section 2.2 of the paper and the sampling step of
// Algorithm 1: every iteration samples a fixed number of neighbours per relation for the nodes of the
// mini-batch, hop by hop; fan-outs such as {25, 20}, Section 8.1).
//
// Rule per (destination, relation): all in-edges if the in-degree is at most the fan-out, otherwise
// `fanout` distinct edge slots uniformly without replacement, by Floyd's subset algorithm (Bentley &
// Floyd, CACM 1987) driven by a counter-based generator, SplitMix64 (Steele, Lea, Flood, OOPSLA 2014):
// destination v draws from the stream keyed mix(seed ^ mix(v)), its j-th number is mix(key + j), and a
// number is mapped below n by the high half of (its high 32 bits) * n.  The result therefore depends
// on (seed, v) only - not on the launch shape or on which other destinations are sampled.
//
// One wavefront per destination: lane i draws the i-th number and holds the i-th chosen slot, membership is one ballot,
// and the ascending order of the output is each lane's rank among the chosen slots.  The unique source ids of a node type
// and the local ids of the sampled edges come from a bitmap of the type's ids, or one radix sort of all sampled ids.  A
// whole hop is five launches and one synchronisation (heta_sample_hop).
#include <algorithm>
#include <vector>

#include <new>

#include "heta_internal.h"

namespace heta {

namespace {

constexpr int kMaxFanout = 64;
constexpr unsigned long long kGamma = 0x9E3779B97F4A7C15ull;

__host__ __device__ inline unsigned long long mix(unsigned long long x)
{
    unsigned long long z = x + kGamma;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ bool id_ok(int64_t v, int64_t n_rows) { return v >= 0 && v < n_rows; }

// ---- sampling: up to 32 relations of a hop in two launches --------------------------------------------------------
// The first counts (destinations in chunks of 256), the second adds up what lies before its 16 destinations, writes their
// row offsets and samples them, one wavefront per destination.  A launch of a few us costs as much again in submission and
// gap, so the sum over the chunks before is taken by every workgroup itself while they are at most kChunksAdded; beyond
// that by a scan (10 M destinations: the workgroups would read 50 GB of sums).  Counts, scan, row offsets and samples in a
// launch each, with two fills and two copies, took 72 to 93 us a hop where this takes 77 to 116 with the source sets, which
// had taken another 59 to 68 (64 / 1,024 seeds of a graph of 21 M edges, seven relations).
constexpr int kFusedItems = 32;
constexpr int kChunk = 256, kFillPer = 16, kFillSubs = kChunk / kFillPer;
constexpr int64_t kChunksAdded = 4096;
struct FusedSample { // passed by value
    int n, fanout;
    const int64_t *ptr[kFusedItems];
    const int32_t *idx[kFusedItems];
    int64_t n_rows[kFusedItems];
    const int64_t *dst[kFusedItems];
    int64_t n_dst[kFusedItems];
    int32_t chunk0[kFusedItems + 1]; // first chunk of each item, one at least
    unsigned long long seed[kFusedItems];
    int64_t *rowptr[kFusedItems];
    int64_t *out[kFusedItems];
};
__device__ __forceinline__ int item_of(const FusedSample &f, int chunk)
{
    int r = 0;
    while (chunk >= f.chunk0[r + 1]) ++r; // uniform; chunk < chunk0[n]
    return r;
}

// Results of one call, in page-locked host memory that the kernels write: no copies to wait for.
struct SampleBack {
    int64_t count[kFusedItems];
    int32_t bad[kFusedItems]; // set where a destination id is out of range; cleared by the host
};

// The workgroups past the last chunk clear n_zero pieces of 16 bytes (the bitmap of the same hop's source sets).
__global__ void __launch_bounds__(kChunk) sample_count_kernel(FusedSample f, uint8_t *cnt, int64_t *chunk_sum, SampleBack *back, uint4 *zero,
                                                              int64_t n_zero)
{
    const int chunk = blockIdx.x;
    if (chunk >= f.chunk0[f.n]) {
        const int64_t i = static_cast<int64_t>(chunk - f.chunk0[f.n]) * kChunk + threadIdx.x;
        if (i < n_zero) zero[i] = make_uint4(0u, 0u, 0u, 0u);
        return;
    }
    __shared__ int total;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    const int r = item_of(f, chunk);
    const int64_t i = static_cast<int64_t>(chunk - f.chunk0[r]) * kChunk + threadIdx.x;
    int c = 0;
    if (i < f.n_dst[r]) {
        const int64_t v = f.dst[r][i];
        if (!id_ok(v, f.n_rows[r])) back->bad[r] = 1; // every writer stores the same value
        else c = static_cast<int>(min(f.ptr[r][v + 1] - f.ptr[r][v], static_cast<int64_t>(f.fanout)));
    }
    cnt[static_cast<int64_t>(chunk) * kChunk + threadIdx.x] = static_cast<uint8_t>(c); // at most kMaxFanout
    atomicAdd(&total, c);
    __syncthreads();
    if (threadIdx.x == 0) chunk_sum[chunk] = total;
}

__device__ __forceinline__ int64_t readlane64(int64_t x, int lane)
{
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(x), lane), hi = __builtin_amdgcn_readlane(static_cast<int>(x >> 32), lane);
    return static_cast<int64_t>((static_cast<unsigned long long>(hi) << 32) | lo);
}

// one wavefront: the sampled in-edges of destination v, whose `deg` edges start at `start`, ascending edge slot, at out[0 ...]
__device__ __forceinline__ void fill_one(const int32_t *idx, int64_t v, int64_t start, int64_t deg, int fanout, unsigned long long seed,
                                         int64_t *out, int lane)
{
    if (deg <= fanout) {
        if (lane < deg) out[lane] = idx[start + lane];
        return;
    }
    // lane c draws the c-th number and holds the c-th chosen slot
    const unsigned long long key = mix(seed ^ mix(static_cast<unsigned long long>(v)));
    const int64_t j = deg - fanout + lane;
    const int64_t drawn = static_cast<int64_t>(((mix(key + static_cast<unsigned long long>(lane)) >> 32) * static_cast<unsigned long long>(j + 1)) >> 32);
    int64_t mine = -1;
    for (int step = 0; step < fanout; ++step) {
        const int64_t t = readlane64(drawn, step);
        const bool present = __ballot(mine == t) != 0ull;
        if (lane == step) mine = present ? j : t;
    }
    int rank = 0;
    for (int c = 0; c < fanout; ++c) rank += readlane64(mine, c) < mine ? 1 : 0;
    if (lane < fanout) out[rank] = idx[start + mine];
}

// SCANNED: chunk_sum holds the exclusive sums over all chunks; first_blk: see launch_pieces
template <bool SCANNED>
__global__ void __launch_bounds__(256) sample_fill_kernel(FusedSample f, int64_t first_blk, const uint8_t *cnt, const int64_t *chunk_sum, SampleBack *back)
{
    __shared__ unsigned long long before_s;
    __shared__ int64_t at[kFillPer], node[kFillPer], first[kFillPer], degree[kFillPer];
    __shared__ int own[kFillPer];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t blk = first_blk + blockIdx.x;
    const int chunk = static_cast<int>(blk / kFillSubs), sub = static_cast<int>(blk % kFillSubs), r = item_of(f, chunk), chunk0 = f.chunk0[r];
    const int64_t n = f.n_dst[r], i0 = static_cast<int64_t>(chunk - chunk0) * kChunk + sub * kFillPer;
    if (i0 >= n) { // uniform
        if (i0 == 0 && tid == 0) {
            f.rowptr[r][0] = 0;
            back->count[r] = 0;
        }
        return;
    }
    if (tid == 0) before_s = 0;
    if (tid < kFillPer && i0 + tid < n) {
        const int64_t v = f.dst[r][i0 + tid];
        node[tid] = v;
        if (id_ok(v, f.n_rows[r])) {
            first[tid] = f.ptr[r][v];
            degree[tid] = f.ptr[r][v + 1] - first[tid];
        } else {
            degree[tid] = 0;
        }
    }
    unsigned long long before = 0;
    if (SCANNED) {
        if (tid == 0) before = static_cast<unsigned long long>(chunk_sum[chunk] - chunk_sum[chunk0]);
    } else {
#pragma unroll 4
        for (int q = chunk0 + tid; q < chunk; q += 256) before += static_cast<unsigned long long>(chunk_sum[q]);
    }
    const int c = cnt[static_cast<int64_t>(chunk) * kChunk + tid];
    if (tid < sub * kFillPer) before += static_cast<unsigned long long>(c);
    else if (tid < (sub + 1) * kFillPer) own[tid - sub * kFillPer] = c;
    __syncthreads();
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
    if (lane == 0 && before) atomicAdd(&before_s, before);
    __syncthreads();
    if (tid < kFillPer && i0 + tid < n) {
        int64_t p = static_cast<int64_t>(before_s);
        for (int q = 0; q < tid; ++q) p += own[q];
        at[tid] = p;
        f.rowptr[r][i0 + tid] = p;
        if (i0 + tid == n - 1) {
            f.rowptr[r][n] = p + own[tid];
            back->count[r] = p + own[tid];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kFillPer / 4; ++q) {
        const int t = wave + 4 * q;
        if (i0 + t < n) fill_one(f.idx[r], node[t], first[t], degree[t], f.fanout, f.seed[r], f.out[r] + at[t], lane);
    }
}

// ---- unique + relabel ----------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) gather_keys_kernel(const int64_t *ids, int64_t n, int64_t offset, int64_t limit,
                                                          uint32_t *keys, uint32_t *vals, int *bad)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t v = ids[i];
    if (v < 0 || v >= limit) *bad = 1;
    keys[offset + i] = static_cast<uint32_t>(v);
    vals[offset + i] = static_cast<uint32_t>(offset + i);
}

__global__ void __launch_bounds__(256) head_flag_kernel(const uint32_t *keys, int64_t n, int64_t *head)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    head[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1 : 0;
}

// before[i] = number of heads before i; the element's unique index is before[i] + head[i] - 1
__global__ void __launch_bounds__(256) unique_scatter_kernel(const uint32_t *keys, const uint32_t *vals, const int64_t *head,
                                                             const int64_t *before, int64_t n, int64_t *unique_ids,
                                                             int32_t *local_all)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const int64_t u = before[i] + head[i] - 1;
    if (head[i]) unique_ids[u] = keys[i];
    local_all[vals[i]] = static_cast<int32_t>(u);
}

// ---- several id sets per launch: the set's index rides in the key's high bits ---------------------------------
constexpr int kFusedLists = 64;
struct FusedLists { // passed by value
    int n_lists, shift; // shift: bits of the id part of a key
    const int64_t *ids[kFusedLists];
    int64_t len[kFusedLists];
    int64_t off[kFusedLists]; // position of the list's first id in the concatenation of all sets
    int64_t limit[kFusedLists];
    uint32_t group[kFusedLists];
};
struct FusedGroups { // passed by value
    int n, shift;
    int64_t base[kFusedItems + 1]; // set g occupies [base[g], base[g+1]) of the sorted array
    int64_t *uniq[kFusedItems];
};

__global__ void __launch_bounds__(256) gather_keys_multi_kernel(FusedLists f, uint32_t *keys, uint32_t *vals, int *bad)
{
    const int l = blockIdx.y;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= f.len[l]) return;
    const int64_t v = f.ids[l][i];
    const bool ok = v >= 0 && v < f.limit[l];
    if (!ok) bad[f.group[l]] = 1;
    // an id out of range must not reach another set's key range (the sets' sizes in the sorted array are relied on)
    keys[f.off[l] + i] = (f.group[l] << f.shift) | (ok ? static_cast<uint32_t>(v) : 0u);
    vals[f.off[l] + i] = static_cast<uint32_t>(f.off[l] + i);
}

__global__ void __launch_bounds__(256) unique_scatter_multi_kernel(FusedGroups f, const uint32_t *keys, const uint32_t *vals,
                                                                   const int64_t *head, const int64_t *before, int64_t n,
                                                                   int32_t *local_all)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t key = keys[i];
    const int g = static_cast<int>(key >> f.shift);
    const int64_t u = before[i] + head[i] - 1 - before[f.base[g]];
    if (head[i]) f.uniq[g][u] = static_cast<int64_t>(key & ((1u << f.shift) - 1u));
    local_all[vals[i]] = static_cast<int32_t>(u);
}

__global__ void __launch_bounds__(64) group_counts_kernel(FusedGroups f, const int64_t *before, int64_t *counts)
{
    const int g = threadIdx.x;
    if (g < f.n) counts[g] = before[f.base[g + 1]] - before[f.base[g]];
}

// ---- unique + relabel through a bitmap of the id ranges ---------------------------------------------------------
// One bit per possible id: mark, count the bits of each tile of 256 64-bit words, emit the set bits in order (which is
// the ascending unique list) with the number of set bits before every word, look every id up.  Five short launches
// whose bytes are the bitmap's; a radix sort of the ids is three launches per eight key bits, each as long as all of
// this (1.9 M possible ids, 120,000 sampled: 95 us of kernels by the sort, 22 us here).
constexpr int kBitTile = 256 * 64;             // ids per tile
constexpr int64_t kBitTilesMax = 4096;         // 8 MB of bits; a tile adds up the counts of those before it in its set
struct BitSets { // passed by value
    int n_sets;
    const int64_t *ids[kFusedLists];
    int32_t *local[kFusedLists];
    int64_t len[kFusedLists];
    const int64_t *len_at[kFusedLists]; // where the length stands on the device, if the host does not know it
    uint8_t set_of[kFusedLists];
    int64_t limit[kFusedItems];
    int64_t *uniq[kFusedItems];
    int32_t tile0[kFusedItems + 1]; // first tile of each set
};

__device__ __forceinline__ int64_t list_len(const BitSets &f, int l) { return f.len_at[l] ? *f.len_at[l] : f.len[l]; }

__global__ void __launch_bounds__(256) bit_zero_kernel(uint4 *bits, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) bits[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Sets the bits `m` of a word unless all of them are set already.
__device__ __forceinline__ void mark_word(unsigned long long *w, unsigned long long m)
{
    if (m & ~__hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(w, m);
}

// A hub is sampled thousands of times and a small range has few words, but updates of one word, and of the words beside
// it, are served one after the other (0.6 to 5 ns each; every wavefront in flight still finds the bit clear).  So a
// workgroup gathers bits in LDS and updates each word once: sets of up to kMarkDirect words in a copy of the whole set,
// at most kMarkGroups workgroups per list; others, 512 ids at a time, in a table of words, where a word that finds no slot
// within kMarkProbes is updated directly; lists of up to kMarkPlain ids past the LDS.  Whole calls with one update per id /
// like this / by the sort, 1 M ids: half of them one of 1.1 M possible ids 2,597 / 117 / 234 us; 64 possible ids
// 2,983 / 48 / 173; 9,000 possible 349 / 50 / 215; spread over 1.1 M 167 / 153 / 240.  300,000 ids spread over 700,000:
// 65 / 80 / 174.
constexpr int kMarkItems = 2, kMarkIds = 256 * kMarkItems, kMarkGroups = 128, kMarkDirect = 4096, kMarkSlots = 1024, kMarkProbes = 4,
              kMarkPlain = 4096;
__global__ void __launch_bounds__(256) bit_mark_kernel(BitSets f, unsigned long long *bits, int *bad)
{
    constexpr unsigned EMPTY = ~0u; // word indices stay below kBitTilesMax * 256
    __shared__ unsigned long long set[kMarkDirect];
    __shared__ unsigned key[kMarkSlots];
    const int l = blockIdx.y, g = f.set_of[l];
    const int64_t n = list_len(f, l), limit = f.limit[g], *ids = f.ids[l];
    const unsigned n_words = static_cast<unsigned>((limit + 63) / 64);
    const bool direct = n_words <= kMarkDirect && n >= 4 * static_cast<int64_t>(n_words); // uniform
    const int64_t rounds = direct ? (n + kMarkGroups * kMarkIds - 1) / (kMarkGroups * kMarkIds) : 1;
    const int64_t start = blockIdx.x * rounds * kMarkIds;
    if (start >= n) return; // uniform
    unsigned long long *words = bits + static_cast<int64_t>(f.tile0[g]) * 256;
    bool outside = false; // an id outside the set's range
    if (direct) {
        for (unsigned s = threadIdx.x; s < n_words; s += 256) set[s] = 0;
        __syncthreads();
        const int64_t end = min(n, start + rounds * kMarkIds);
#pragma unroll 4
        for (int64_t i = start + threadIdx.x; i < end; i += 256) {
            const int64_t v = ids[i];
            if (v < 0 || v >= limit) outside = true;
            else atomicOr(&set[v >> 6], 1ull << (v & 63));
        }
        __syncthreads();
        for (unsigned s = threadIdx.x; s < n_words; s += 256)
            if (set[s]) mark_word(words + s, set[s]);
        if (outside) bad[g] = 1;
        return;
    }
    int64_t v[kMarkItems];
#pragma unroll
    for (int j = 0; j < kMarkItems; ++j) v[j] = start + 256 * j + threadIdx.x < n ? ids[start + 256 * j + threadIdx.x] : -1;
    if (n <= kMarkPlain) { // too few to queue up for long: past the LDS
#pragma unroll
        for (int j = 0; j < kMarkItems; ++j) {
            if (start + 256 * j + threadIdx.x >= n) continue;
            if (v[j] < 0 || v[j] >= limit) bad[g] = 1; // every writer stores the same value
            else mark_word(words + (v[j] >> 6), 1ull << (v[j] & 63));
        }
        return;
    }
#pragma unroll
    for (int s = 0; s < kMarkSlots; s += 256) {
        set[s + threadIdx.x] = 0;
        key[s + threadIdx.x] = EMPTY;
    }
    __syncthreads();
    int slot[kMarkItems]; // of the words that this thread updates: it entered them
#pragma unroll
    for (int j = 0; j < kMarkItems; ++j) {
        slot[j] = -1;
        if (v[j] < 0 || v[j] >= limit) {
            outside |= start + 256 * j + threadIdx.x < n;
            continue;
        }
        const unsigned w = static_cast<unsigned>(v[j] >> 6);
        const unsigned long long bit = 1ull << (v[j] & 63);
        unsigned h = (w * 2654435761u) >> 22; // multiplicative hashing: the upper 10 bits
        bool placed = false;
        for (int q = 0; q < kMarkProbes && !placed; ++q) {
            unsigned k = __hip_atomic_load(&key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (k == EMPTY) {
                k = atomicCAS(&key[h], EMPTY, w);
                if (k == EMPTY) slot[j] = h;
            }
            placed = k == EMPTY || k == w;
            if (placed) atomicOr(&set[h], bit);
            h = (h + 1) % kMarkSlots;
        }
        if (!placed) mark_word(words + w, bit);
    }
    __syncthreads();
    unsigned long long now[kMarkItems]; // all loads before the first update, for which a later load would wait
#pragma unroll
    for (int j = 0; j < kMarkItems; ++j)
        now[j] = slot[j] >= 0 ? __hip_atomic_load(words + (v[j] >> 6), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0ull;
#pragma unroll
    for (int j = 0; j < kMarkItems; ++j)
        if (slot[j] >= 0 && (set[slot[j]] & ~now[j])) atomicOr(words + (v[j] >> 6), set[slot[j]]);
    if (outside) bad[g] = 1;
}

// sum over the workgroup's 256 threads, in every thread
__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *lds)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    __syncthreads(); // earlier readers of lds
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    return lds[0] + lds[1] + lds[2] + lds[3];
}

__global__ void __launch_bounds__(256) bit_count_kernel(const unsigned long long *bits, uint32_t *tile_count)
{
    __shared__ uint32_t lds[4];
    const uint32_t n = block_sum(__popcll(bits[static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x]), lds);
    if (threadIdx.x == 0) tile_count[blockIdx.x] = n;
}

// tile_count null: the bits of the tiles before are counted here.  Up to kBitTilesCounted tiles that is shorter than the
// launch of bit_count_kernel.
// (115 tiles: 7 us; with the other launch 2 + 4 us and the gap between them.)
constexpr int kBitTilesCounted = 256;
__global__ void __launch_bounds__(256) bit_emit_kernel(BitSets f, const unsigned long long *bits, const uint32_t *tile_count,
                                                       uint32_t *word_rank, int64_t *counts)
{
    __shared__ uint32_t lds[4];
    const int tile = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int g = 0;
    while (tile >= f.tile0[g + 1]) ++g; // uniform; tile < tile0[n_sets]
    uint32_t before = 0;
    if (tile_count) {
        for (int t = f.tile0[g] + threadIdx.x; t < tile; t += 256) before += tile_count[t];
    } else {
        const ulonglong2 *pairs = reinterpret_cast<const ulonglong2 *>(bits);
#pragma unroll 8
        for (int64_t i = static_cast<int64_t>(f.tile0[g]) * 128 + threadIdx.x; i < static_cast<int64_t>(tile) * 128; i += 256)
            before += __popcll(pairs[i].x) + __popcll(pairs[i].y);
    }
    before = block_sum(before, lds);
    const int64_t at = static_cast<int64_t>(tile) * 256 + threadIdx.x;
    unsigned long long w = bits[at];
    const uint32_t mine = __popcll(w);
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
    }
    __syncthreads();
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    uint32_t rank = before + incl - mine;
    for (int q = 0; q < wave; ++q) rank += lds[q];
    word_rank[at] = rank;
    const int64_t id0 = (static_cast<int64_t>(tile - f.tile0[g]) * 256 + threadIdx.x) * 64;
    int64_t *uniq = f.uniq[g];
    while (w) {
        uniq[rank++] = id0 + __ffsll(w) - 1;
        w &= w - 1;
    }
    if (threadIdx.x == 255 && tile + 1 == f.tile0[g + 1]) counts[g] = rank;
}

__global__ void __launch_bounds__(256) bit_local_kernel(BitSets f, const unsigned long long *bits, const uint32_t *word_rank)
{
    const int l = blockIdx.y;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= list_len(f, l)) return;
    const int g = f.set_of[l];
    const int64_t v = f.ids[l][i];
    if (v < 0 || v >= f.limit[g]) return; // reported after the synchronisation
    const int64_t at = static_cast<int64_t>(f.tile0[g]) * 256 + (v >> 6);
    f.local[l][i] = static_cast<int32_t>(word_rank[at] + __popcll(bits[at] & ((1ull << (v & 63)) - 1)));
}

// Whether no output (unique lists, local ids) shares memory with an input list.  The bitmap reads the lists once more after
// the unique lists are written, and its threads write local ids beside lists that others still read; the sort copies the
// ids out of the lists before it writes anything.
static bool outputs_apart(int32_t n_groups, const int32_t *group_ptr, const int64_t *const *lists, const int64_t *lens,
                          const std::vector<int64_t> &totals, int64_t *const *unique_ids, int32_t *const *local)
{
    const auto apart = [&](const void *out, int64_t bytes) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(out);
        for (int32_t l = 0; l < group_ptr[n_groups]; ++l) {
            const uintptr_t b = reinterpret_cast<uintptr_t>(lists[l]);
            if (bytes > 0 && lens[l] > 0 && a < b + static_cast<uintptr_t>(lens[l]) * 8 && b < a + static_cast<uintptr_t>(bytes)) return false;
        }
        return true;
    };
    for (int32_t g = 0; g < n_groups; ++g)
        if (!apart(unique_ids[g], totals[g] * 8)) return false;
    for (int32_t l = 0; l < group_ptr[n_groups]; ++l)
        if (!apart(local[l], lens[l] * 4)) return false;
    return true;
}

// scratch of one call, from the recycling pool (released idle: every entry point below synchronises its
// stream before it returns, and the destructor waits for the device in case an error path did not)
struct Scratch {
    char *p = nullptr;
    size_t cursor = 0;
    bool idle = false; // the entry point has synchronised its stream after the last use
    ~Scratch()
    {
        if (!p) return;
        if (!idle) (void)hipDeviceSynchronize(); // error paths
        scratch_free(p);
    }
    static size_t padded(size_t bytes) { return (std::max<size_t>(bytes, 1) + 255) / 256 * 256; }
    heta_status alloc(size_t bytes)
    {
        hipError_t e = scratch_alloc(reinterpret_cast<void **>(&p), std::max<size_t>(bytes, 256));
        if (e != hipSuccess)
            return fail(e == hipErrorOutOfMemory ? HETA_ERR_OOM : HETA_ERR_DEVICE, "allocation of sampler scratch failed: %s",
                        hipGetErrorString(e));
        return HETA_OK;
    }
    template <typename T> T *take(size_t n) // slices were sized with padded() before alloc()
    {
        T *q = reinterpret_cast<T *>(p + cursor);
        cursor += padded(n * sizeof(T));
        return q;
    }
};

// Counts and error flags come back through page-locked slots, so that the copies are asynchronous and a
// whole batch is awaited once (a copy into pageable memory blocks the host until it has landed).
struct Slot {
    int64_t count;
    int32_t bad;
    int32_t pad;
};
struct PinnedSlots {
    Slot *p = nullptr;
    size_t cap = 0;
};
static thread_local PinnedSlots t_slots; // never freed: it lives as long as the thread samples

static heta_status slots_reserve(size_t n)
{
    if (n <= t_slots.cap) return HETA_OK;
    const size_t cap = std::max<size_t>(n, 64);
    void *q = nullptr;
    if (hipHostMalloc(&q, cap * sizeof(Slot), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess)
        return fail(HETA_ERR_OOM, "page-locked host allocation of %zu result slots failed", cap);
    if (t_slots.p) (void)hipHostFree(t_slots.p);
    t_slots.p = static_cast<Slot *>(q);
    t_slots.cap = cap;
    return HETA_OK;
}

// Fills in the items' arguments.
static void sample_plan(FusedSample &f, const heta_graph *g, int32_t n, const int32_t *rels, const int64_t *const *dst_ids, const int64_t *n_dst,
                           int32_t fanout, const uint64_t *seeds, int64_t *const *rowptr, int64_t *const *src_ids)
{
    f.n = n;
    f.fanout = fanout;
    int64_t chunks = 0; // at most kFusedItems + 2^31 / kChunk: the callers bound the destinations
    for (int32_t i = 0; i < n; ++i) {
        const Relation &r = g->rels[rels[i]];
        f.ptr[i] = r.csr.d_ptr;
        f.idx[i] = r.csr.d_idx;
        f.n_rows[i] = r.n_dst;
        f.dst[i] = dst_ids[i];
        f.n_dst[i] = n_dst[i];
        f.seed[i] = seeds[i];
        f.rowptr[i] = rowptr[i];
        f.out[i] = src_ids[i];
        f.chunk0[i] = static_cast<int32_t>(chunks);
        chunks += std::max<int64_t>(1, (n_dst[i] + kChunk - 1) / kChunk);
    }
    f.chunk0[n] = static_cast<int32_t>(chunks);
}
static size_t sample_scratch_bytes(int64_t chunks)
{
    const size_t c = static_cast<size_t>(chunks);
    return Scratch::padded(c * kChunk) + 2 * Scratch::padded((c + 1) * sizeof(int64_t)) +
           Scratch::padded(static_cast<size_t>(scan_scratch_elems(chunks + 1)) * sizeof(int64_t));
}
static heta_status sample_launch(const FusedSample &f, Scratch &scratch, SampleBack *back, uint4 *zero, int64_t n_zero, hipStream_t st)
{
    const int64_t chunks = f.chunk0[f.n];
    uint8_t *cnt = scratch.take<uint8_t>(static_cast<size_t>(chunks) * kChunk);
    int64_t *sums = scratch.take<int64_t>(static_cast<size_t>(chunks) + 1), *scanned = scratch.take<int64_t>(static_cast<size_t>(chunks) + 1);
    int64_t *tsum = scratch.take<int64_t>(static_cast<size_t>(scan_scratch_elems(chunks + 1)));
    for (int r = 0; r < f.n; ++r) back->bad[r] = 0;
    hipLaunchKernelGGL(sample_count_kernel, dim3((unsigned)(chunks + (n_zero + kChunk - 1) / kChunk)), dim3(kChunk), 0, st, f, cnt, sums, back, zero, n_zero);
    HETA_LAUNCH_CHECK("sample_count_kernel");
    if (chunks > kChunksAdded) {
        heta_status e = device_exclusive_scan_i64_async(sums, chunks, scanned, chunks + 1, tsum, st);
        if (e != HETA_OK) return e;
    }
    launch_pieces(chunks * kFillSubs, 256, [&](int64_t first, unsigned blocks) {
        if (chunks > kChunksAdded)
            hipLaunchKernelGGL(sample_fill_kernel<true>, dim3(blocks), dim3(256), 0, st, f, first, cnt, scanned, back);
        else
            hipLaunchKernelGGL(sample_fill_kernel<false>, dim3(blocks), dim3(256), 0, st, f, first, cnt, sums, back);
    });
    HETA_LAUNCH_CHECK("sample_fill_kernel");
    return HETA_OK;
}
// after the synchronisation: the counts, or the fault
static heta_status sample_results(const heta_graph *g, const SampleBack *back, int32_t n, const int32_t *rels, int64_t *n_sampled)
{
    for (int32_t i = 0; i < n; ++i)
        if (back->bad[i])
            return fail(HETA_ERR_INVALID_ARG, "heta_sample_neighbors: a destination id of relation %d lies outside [0, %lld)", rels[i],
                        (long long)g->rels[rels[i]].n_dst);
    for (int32_t i = 0; i < n; ++i) n_sampled[i] = back->count[i];
    return HETA_OK;
}
constexpr size_t kBackSlots = (sizeof(SampleBack) + sizeof(Slot) - 1) / sizeof(Slot);

// The bitmap form of unique + relabel from the mark on, for sets whose bits are clear; counts and bad (cleared) may be
// page-locked host memory.  cap: the longest list's length or a bound of it.
static heta_status bits_launch(const BitSets &f, int32_t n_lists, int64_t cap, unsigned long long *bits, uint32_t *word_rank, uint32_t *tile_count,
                               int64_t *counts, int *bad, hipStream_t st)
{
    const int tiles = f.tile0[f.n_sets];
    if (cap == 0) return HETA_OK;
    const dim3 mark_grid((unsigned)((cap + kMarkIds - 1) / kMarkIds), (unsigned)n_lists);
    hipLaunchKernelGGL(bit_mark_kernel, mark_grid, dim3(256), 0, st, f, bits, bad);
    HETA_LAUNCH_CHECK("bit_mark_kernel");
    if (tiles > kBitTilesCounted) {
        hipLaunchKernelGGL(bit_count_kernel, dim3((unsigned)tiles), dim3(256), 0, st, bits, tile_count);
        HETA_LAUNCH_CHECK("bit_count_kernel");
    }
    hipLaunchKernelGGL(bit_emit_kernel, dim3((unsigned)tiles), dim3(256), 0, st, f, bits, tiles > kBitTilesCounted ? tile_count : (uint32_t *)nullptr,
                       word_rank, counts);
    HETA_LAUNCH_CHECK("bit_emit_kernel");
    hipLaunchKernelGGL(bit_local_kernel, dim3((unsigned)((cap + 255) / 256), (unsigned)n_lists), dim3(256), 0, st, f, bits, word_rank);
    HETA_LAUNCH_CHECK("bit_local_kernel");
    return HETA_OK;
}

} // namespace

} // namespace heta

using namespace heta;

extern "C" {

heta_status heta_sample_neighbors_batch(const heta_graph *g, int32_t n, const int32_t *rels, const int64_t *const *dst_ids,
                                        const int64_t *n_dst, int32_t fanout, const uint64_t *seeds, int64_t *const *rowptr,
                                        int64_t *const *src_ids, int64_t *n_sampled, void *hip_stream)
{
    if (!g || n < 0 || (n > 0 && (!rels || !dst_ids || !n_dst || !seeds || !rowptr || !src_ids || !n_sampled)))
        return fail(HETA_ERR_INVALID_ARG, "heta_sample_neighbors: null argument");
    if (fanout < 1 || fanout > kMaxFanout)
        return fail(HETA_ERR_SHAPE, "heta_sample_neighbors: need 1 <= fanout <= %d", kMaxFanout);
    int64_t all_dst = 0;
    for (int32_t i = 0; i < n; ++i) {
        if (rels[i] < 0 || rels[i] >= (int32_t)g->rels.size())
            return fail(HETA_ERR_INVALID_ARG, "heta_sample_neighbors: relation %d out of range", rels[i]);
        if (n_dst[i] < 0) return fail(HETA_ERR_SHAPE, "heta_sample_neighbors: need n_dst >= 0");
        if (!rowptr[i] || (n_dst[i] > 0 && (!dst_ids[i] || !src_ids[i])))
            return fail(HETA_ERR_INVALID_ARG, "heta_sample_neighbors: null argument");
        n_sampled[i] = 0;
        if (n_dst[i] >= (int64_t(1) << 31)) return fail(HETA_ERR_UNSUPPORTED, "heta_sample_neighbors: more than 2^31 destinations");
        all_dst += n_dst[i];
    }
    if (n == 0) return HETA_OK;
    hipStream_t st = as_stream(hip_stream);
    heta_status e;
    if (n <= kFusedItems && all_dst >= (int64_t(1) << 31)) return fail(HETA_ERR_UNSUPPORTED, "heta_sample_neighbors: more than 2^31 destinations");
    // Up to kFusedItems items of fewer than 2^31 destinations together share their launches; one synchronisation for all.
    const auto group_end = [&](int32_t i) {
        int64_t total = n_dst[i];
        int32_t j = i + 1;
        while (j < n && j - i < kFusedItems && total + n_dst[j] < (int64_t(1) << 31)) total += n_dst[j++];
        return j;
    };
    size_t bytes = 0, groups = 0;
    for (int32_t i = 0; i < n; ++i) bytes += sample_scratch_bytes(std::max<int64_t>(1, (n_dst[i] + kChunk - 1) / kChunk));
    for (int32_t i = 0; i < n; i = group_end(i)) ++groups;
    Scratch scratch;
    if ((e = scratch.alloc(bytes)) != HETA_OK || (e = slots_reserve(kBackSlots * groups)) != HETA_OK) return e;
    Slot *slot = t_slots.p;
    for (int32_t i = 0, j; i < n; i = j, slot += kBackSlots) {
        j = group_end(i);
        FusedSample f{};
        sample_plan(f, g, j - i, rels + i, dst_ids + i, n_dst + i, fanout, seeds + i, rowptr + i, src_ids + i);
        if ((e = sample_launch(f, scratch, reinterpret_cast<SampleBack *>(slot), nullptr, 0, st)) != HETA_OK) return e;
    }
    HETA_HIP(hipStreamSynchronize(st));
    scratch.idle = true;
    slot = t_slots.p;
    for (int32_t i = 0, j; i < n; i = j, slot += kBackSlots) {
        j = group_end(i);
        if ((e = sample_results(g, reinterpret_cast<const SampleBack *>(slot), j - i, rels + i, n_sampled + i)) != HETA_OK) {
            std::fill(n_sampled, n_sampled + n, int64_t(0));
            return e;
        }
    }
    return HETA_OK;
}

heta_status heta_sample_neighbors(const heta_graph *g, int32_t rel, const int64_t *dst_ids, int64_t n_dst, int32_t fanout,
                                  uint64_t seed, int64_t *rowptr, int64_t *src_ids, int64_t *n_sampled, void *hip_stream)
{
    if (!n_sampled) return fail(HETA_ERR_INVALID_ARG, "heta_sample_neighbors: null argument");
    return heta_sample_neighbors_batch(g, 1, &rel, &dst_ids, &n_dst, fanout, &seed, &rowptr, &src_ids, n_sampled, hip_stream);
}

static heta_status heta_unique_relabel_batch_impl(int32_t n_groups, const int32_t *group_ptr, const int64_t *const *lists,
                                      const int64_t *lens, const int64_t *id_limit, int64_t *const *unique_ids,
                                      int64_t *n_unique, int32_t *const *local, void *hip_stream)
{
    if (n_groups < 0 || (n_groups > 0 && (!group_ptr || !id_limit || !unique_ids || !n_unique)))
        return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: null argument");
    if (n_groups == 0) return HETA_OK;
    if (group_ptr[0] != 0) return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: group_ptr[0] must be 0");
    std::vector<int64_t> totals(n_groups, 0);
    size_t bytes = Scratch::padded(static_cast<size_t>(n_groups) * sizeof(int));
    for (int32_t gidx = 0; gidx < n_groups; ++gidx) {
        if (group_ptr[gidx + 1] < group_ptr[gidx]) return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: group_ptr decreases");
        if (group_ptr[gidx + 1] > group_ptr[gidx] && (!lists || !lens || !local))
            return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: null argument");
        if (id_limit[gidx] < 0 || id_limit[gidx] > (int64_t(1) << 31))
            return fail(HETA_ERR_SHAPE, "heta_unique_relabel: id_limit outside [0, 2^31]");
        for (int32_t l = group_ptr[gidx]; l < group_ptr[gidx + 1]; ++l) {
            if (lens[l] < 0 || (lens[l] > 0 && (!lists[l] || !local[l])))
                return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: list %d is null or has a negative length", l);
            totals[gidx] += lens[l];
        }
        n_unique[gidx] = 0;
        const int64_t total = totals[gidx];
        if (total == 0) continue;
        if (total >= (int64_t(1) << 31)) return fail(HETA_ERR_UNSUPPORTED, "heta_unique_relabel: more than 2^31 ids");
        if (!unique_ids[gidx]) return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: null unique_ids");
        const size_t N = static_cast<size_t>(total), n_hist = static_cast<size_t>(sort_hist_elems(total));
        bytes += 4 * Scratch::padded(N * sizeof(uint32_t)) + 2 * Scratch::padded(n_hist * sizeof(uint32_t)) +
                 Scratch::padded(static_cast<size_t>(scan_scratch_elems(static_cast<int64_t>(n_hist))) * sizeof(uint32_t)) +
                 Scratch::padded(N * sizeof(int64_t)) + Scratch::padded((N + 1) * sizeof(int64_t)) +
                 Scratch::padded(static_cast<size_t>(scan_scratch_elems(total + 1)) * sizeof(int64_t)) +
                 Scratch::padded(N * sizeof(int32_t));
    }
    if (std::all_of(totals.begin(), totals.end(), [](int64_t t) { return t == 0; })) return HETA_OK; // nothing for the device
    hipStream_t st = as_stream(hip_stream);
    Scratch scratch;
    heta_status e;
    if (n_groups <= kFusedItems && group_ptr[n_groups] <= kFusedLists && outputs_apart(n_groups, group_ptr, lists, lens, totals, unique_ids, local)) {
        // Id ranges of up to 67 M ids together: by bitmap, whatever the number of ids.  The bound keeps the scratch at 12 MB, which
        // the recycling pool still takes, and the counts that a tile adds up at 4,096; the sort is not yet faster there (67 M
        // possible ids, 300 / 50,000 / 5 M given: 50 / 56 / 388 us, by the sort 96 / 133 / 867), but for many ids of few words
        // (400,000 of the lowest 67,000: 161 us, by the sort 145).
        BitSets f{};
        f.n_sets = n_groups;
        int64_t tiles = 0, len_max = 0;
        for (int32_t gidx = 0; gidx < n_groups; ++gidx) {
            f.tile0[gidx] = static_cast<int32_t>(std::min<int64_t>(tiles, kBitTilesMax + 1));
            if (totals[gidx] > 0) tiles += std::max<int64_t>(1, (id_limit[gidx] + kBitTile - 1) / kBitTile);
            f.limit[gidx] = id_limit[gidx];
            f.uniq[gidx] = unique_ids[gidx];
            for (int32_t l = group_ptr[gidx]; l < group_ptr[gidx + 1]; ++l) {
                f.ids[l] = lists[l];
                f.local[l] = local[l];
                f.len[l] = lens[l];
                f.set_of[l] = static_cast<uint8_t>(gidx);
                len_max = std::max(len_max, lens[l]);
            }
        }
        if (tiles <= kBitTilesMax) {
            f.tile0[n_groups] = static_cast<int32_t>(tiles);
            const size_t words = static_cast<size_t>(tiles) * 256, ns = static_cast<size_t>(n_groups);
            if ((e = scratch.alloc(Scratch::padded(words * 8) + Scratch::padded(words * 4) + Scratch::padded(static_cast<size_t>(tiles) * 4))) != HETA_OK ||
                (e = slots_reserve(ns)) != HETA_OK) // a slot holds a count and a flag
                return e;
            int64_t *h_counts = reinterpret_cast<int64_t *>(t_slots.p); // written by the kernels
            int *h_bad = reinterpret_cast<int *>(h_counts + n_groups);
            for (int32_t gidx = 0; gidx < n_groups; ++gidx) h_bad[gidx] = 0;
            unsigned long long *bits = scratch.take<unsigned long long>(words);
            uint32_t *word_rank = scratch.take<uint32_t>(words), *tile_count = scratch.take<uint32_t>(static_cast<size_t>(tiles));
            hipLaunchKernelGGL(bit_zero_kernel, dim3((unsigned)((words / 2 + 255) / 256)), dim3(256), 0, st, reinterpret_cast<uint4 *>(bits),
                               static_cast<int64_t>(words / 2));
            HETA_LAUNCH_CHECK("bit_zero_kernel");
            if ((e = bits_launch(f, group_ptr[n_groups], len_max, bits, word_rank, tile_count, h_counts, h_bad, st)) != HETA_OK) return e;
            HETA_HIP(hipStreamSynchronize(st));
            scratch.idle = true;
            for (int32_t gidx = 0; gidx < n_groups; ++gidx)
                if (h_bad[gidx])
                    return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: an id lies outside [0, %lld)", (long long)id_limit[gidx]);
            for (int32_t gidx = 0; gidx < n_groups; ++gidx) n_unique[gidx] = totals[gidx] > 0 ? h_counts[gidx] : 0;
            return HETA_OK;
        }
    }
    {
        // All sets in one sort when the set index fits above the ids in a 32-bit key: set g's ids then occupy
        // exactly [base[g], base[g+1]) of the sorted array, and one pass of every stage serves all sets.
        int id_bits = 1, set_bits = 0;
        int64_t N = 0;
        for (int32_t gidx = 0; gidx < n_groups; ++gidx) {
            while ((int64_t(1) << id_bits) < id_limit[gidx]) ++id_bits;
            N += totals[gidx];
        }
        while ((1 << set_bits) < n_groups) ++set_bits;
        const int32_t n_lists = group_ptr[n_groups];
        if (n_groups <= kFusedItems && n_lists <= kFusedLists && id_bits + set_bits <= 32 && id_bits <= 31 && N < (int64_t(1) << 31)) {
            FusedLists fl{};
            FusedGroups fg{};
            fl.n_lists = n_lists;
            fl.shift = fg.shift = id_bits;
            fg.n = n_groups;
            int64_t off = 0, len_max = 0;
            int32_t *local_first = nullptr;
            bool contiguous = true; // the lists' local arrays laid end to end in the same order: written in place
            for (int32_t gidx = 0; gidx < n_groups; ++gidx) {
                fg.base[gidx] = off;
                fg.uniq[gidx] = unique_ids[gidx];
                for (int32_t l = group_ptr[gidx]; l < group_ptr[gidx + 1]; ++l) {
                    fl.ids[l] = lists[l];
                    fl.len[l] = lens[l];
                    fl.off[l] = off;
                    fl.limit[l] = id_limit[gidx];
                    fl.group[l] = static_cast<uint32_t>(gidx);
                    if (lens[l] > 0) {
                        if (!local_first) local_first = local[l];
                        contiguous = contiguous && local[l] == local_first + off;
                    }
                    off += lens[l];
                    len_max = std::max(len_max, lens[l]);
                }
            }
            fg.base[n_groups] = off;
            const size_t Ns = static_cast<size_t>(N), n_hist = static_cast<size_t>(sort_hist_elems(N));
            const size_t fused_bytes =
                Scratch::padded(static_cast<size_t>(n_groups) * sizeof(int)) + 4 * Scratch::padded(Ns * sizeof(uint32_t)) +
                2 * Scratch::padded(n_hist * sizeof(uint32_t)) +
                Scratch::padded(static_cast<size_t>(scan_scratch_elems(static_cast<int64_t>(n_hist))) * sizeof(uint32_t)) +
                Scratch::padded(Ns * sizeof(int64_t)) + Scratch::padded((Ns + 1) * sizeof(int64_t)) +
                Scratch::padded(static_cast<size_t>(scan_scratch_elems(N + 1)) * sizeof(int64_t)) + Scratch::padded(Ns * sizeof(int32_t)) +
                Scratch::padded(static_cast<size_t>(n_groups) * sizeof(int64_t));
            if ((e = scratch.alloc(fused_bytes)) != HETA_OK || (e = slots_reserve(2 * static_cast<size_t>(n_groups))) != HETA_OK) return e;
            int *bad = scratch.take<int>(static_cast<size_t>(n_groups));
            uint32_t *k0 = scratch.take<uint32_t>(Ns), *v0 = scratch.take<uint32_t>(Ns), *k1 = scratch.take<uint32_t>(Ns),
                     *v1 = scratch.take<uint32_t>(Ns), *hist = scratch.take<uint32_t>(n_hist), *offs = scratch.take<uint32_t>(n_hist);
            uint32_t *tsum32 = scratch.take<uint32_t>(static_cast<size_t>(scan_scratch_elems(static_cast<int64_t>(n_hist))));
            int64_t *head = scratch.take<int64_t>(Ns), *before = scratch.take<int64_t>(Ns + 1);
            int64_t *tsum64 = scratch.take<int64_t>(static_cast<size_t>(scan_scratch_elems(N + 1)));
            int32_t *local_scratch = scratch.take<int32_t>(Ns);
            int64_t *counts = scratch.take<int64_t>(static_cast<size_t>(n_groups));
            int32_t *local_all = contiguous ? local_first : local_scratch;
            HETA_HIP(hipMemsetAsync(bad, 0, static_cast<size_t>(n_groups) * sizeof(int), st));
            hipLaunchKernelGGL(gather_keys_multi_kernel, dim3((unsigned)((len_max + 255) / 256), (unsigned)n_lists), dim3(256), 0, st, fl,
                               k0, v0, bad);
            HETA_LAUNCH_CHECK("gather_keys_multi_kernel");
            uint32_t *ks = nullptr, *vs = nullptr;
            const int64_t key_limit = static_cast<int64_t>(n_groups) << id_bits;
            if ((e = device_sort_pairs_u32_async(k0, v0, k1, v1, N, key_limit, &ks, &vs, hist, offs, tsum32, st)) != HETA_OK) return e;
            const unsigned blocks = (unsigned)((N + 255) / 256);
            hipLaunchKernelGGL(head_flag_kernel, dim3(blocks), dim3(256), 0, st, ks, N, head);
            HETA_LAUNCH_CHECK("head_flag_kernel");
            if ((e = device_exclusive_scan_i64_async(head, N, before, N + 1, tsum64, st)) != HETA_OK) return e;
            hipLaunchKernelGGL(unique_scatter_multi_kernel, dim3(blocks), dim3(256), 0, st, fg, ks, vs, head, before, N, local_all);
            HETA_LAUNCH_CHECK("unique_scatter_multi_kernel");
            hipLaunchKernelGGL(group_counts_kernel, dim3(1), dim3(64), 0, st, fg, before, counts);
            HETA_LAUNCH_CHECK("group_counts_kernel");
            if (!contiguous)
                for (int32_t l = 0; l < n_lists; ++l)
                    if (lens[l] > 0)
                        HETA_HIP(hipMemcpyAsync(local[l], local_all + fl.off[l], static_cast<size_t>(lens[l]) * sizeof(int32_t),
                                                hipMemcpyDeviceToDevice, st));
            int64_t *h_counts = reinterpret_cast<int64_t *>(t_slots.p);
            int *h_bad = reinterpret_cast<int *>(t_slots.p + n_groups);
            HETA_HIP(hipMemcpyAsync(h_counts, counts, static_cast<size_t>(n_groups) * sizeof(int64_t), hipMemcpyDeviceToHost, st));
            HETA_HIP(hipMemcpyAsync(h_bad, bad, static_cast<size_t>(n_groups) * sizeof(int), hipMemcpyDeviceToHost, st));
            HETA_HIP(hipStreamSynchronize(st));
            for (int32_t gidx = 0; gidx < n_groups; ++gidx)
                if (h_bad[gidx])
                    return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: an id lies outside [0, %lld)", (long long)id_limit[gidx]);
            for (int32_t gidx = 0; gidx < n_groups; ++gidx) n_unique[gidx] = h_counts[gidx];
            return HETA_OK;
        }
    }
    if ((e = scratch.alloc(bytes)) != HETA_OK || (e = slots_reserve(static_cast<size_t>(n_groups))) != HETA_OK) return e;
    int *bad = scratch.take<int>(static_cast<size_t>(n_groups));
    HETA_HIP(hipMemsetAsync(bad, 0, static_cast<size_t>(n_groups) * sizeof(int), st));
    // per group gather -> sort -> head flags -> scan -> scatter -> copies, all asynchronous; one synchronisation for the batch
    for (int32_t gidx = 0; gidx < n_groups; ++gidx) {
        t_slots.p[gidx].count = 0;
        t_slots.p[gidx].bad = 0;
        const int64_t total = totals[gidx];
        if (total == 0) continue;
        const size_t N = static_cast<size_t>(total), n_hist = static_cast<size_t>(sort_hist_elems(total));
        uint32_t *k0 = scratch.take<uint32_t>(N), *v0 = scratch.take<uint32_t>(N), *k1 = scratch.take<uint32_t>(N),
                 *v1 = scratch.take<uint32_t>(N), *hist = scratch.take<uint32_t>(n_hist), *offs = scratch.take<uint32_t>(n_hist);
        uint32_t *tsum32 = scratch.take<uint32_t>(static_cast<size_t>(scan_scratch_elems(static_cast<int64_t>(n_hist))));
        int64_t *head = scratch.take<int64_t>(N), *before = scratch.take<int64_t>(N + 1);
        int64_t *tsum64 = scratch.take<int64_t>(static_cast<size_t>(scan_scratch_elems(total + 1)));
        int32_t *local_all = scratch.take<int32_t>(N);
        int64_t off = 0;
        for (int32_t l = group_ptr[gidx]; l < group_ptr[gidx + 1]; ++l) {
            if (lens[l] == 0) continue;
            hipLaunchKernelGGL(gather_keys_kernel, dim3((unsigned)((lens[l] + 255) / 256)), dim3(256), 0, st, lists[l], lens[l], off,
                               id_limit[gidx], k0, v0, bad + gidx);
            HETA_LAUNCH_CHECK("gather_keys_kernel");
            off += lens[l];
        }
        // an id outside the range is reported after the synchronisation; until then it is only a key like any other
        uint32_t *ks = nullptr, *vs = nullptr;
        if ((e = device_sort_pairs_u32_async(k0, v0, k1, v1, total, id_limit[gidx], &ks, &vs, hist, offs, tsum32, st)) != HETA_OK)
            return e;
        const unsigned blocks = (unsigned)((total + 255) / 256);
        hipLaunchKernelGGL(head_flag_kernel, dim3(blocks), dim3(256), 0, st, ks, total, head);
        HETA_LAUNCH_CHECK("head_flag_kernel");
        if ((e = device_exclusive_scan_i64_async(head, total, before, total + 1, tsum64, st)) != HETA_OK) return e;
        hipLaunchKernelGGL(unique_scatter_kernel, dim3(blocks), dim3(256), 0, st, ks, vs, head, before, total, unique_ids[gidx],
                           local_all);
        HETA_LAUNCH_CHECK("unique_scatter_kernel");
        off = 0;
        for (int32_t l = group_ptr[gidx]; l < group_ptr[gidx + 1]; ++l) {
            if (lens[l] == 0) continue;
            HETA_HIP(hipMemcpyAsync(local[l], local_all + off, static_cast<size_t>(lens[l]) * sizeof(int32_t),
                                    hipMemcpyDeviceToDevice, st));
            off += lens[l];
        }
        HETA_HIP(hipMemcpyAsync(&t_slots.p[gidx].bad, bad + gidx, sizeof(int), hipMemcpyDeviceToHost, st));
        HETA_HIP(hipMemcpyAsync(&t_slots.p[gidx].count, before + total, sizeof(int64_t), hipMemcpyDeviceToHost, st));
    }
    HETA_HIP(hipStreamSynchronize(st));
    for (int32_t gidx = 0; gidx < n_groups; ++gidx)
        if (t_slots.p[gidx].bad)
            return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: an id lies outside [0, %lld)", (long long)id_limit[gidx]);
    for (int32_t gidx = 0; gidx < n_groups; ++gidx) n_unique[gidx] = t_slots.p[gidx].count;
    return HETA_OK;
}

// No exception crosses the boundary: host containers may throw std::bad_alloc.
heta_status heta_unique_relabel_batch(int32_t n_groups, const int32_t *group_ptr, const int64_t *const *lists,
                                      const int64_t *lens, const int64_t *id_limit, int64_t *const *unique_ids,
                                      int64_t *n_unique, int32_t *const *local, void *hip_stream)
{
    try {
        return heta_unique_relabel_batch_impl(n_groups, group_ptr, lists, lens, id_limit, unique_ids, n_unique, local, hip_stream);
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_unique_relabel_batch: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_unique_relabel_batch: unexpected exception");
    }
}

static heta_status heta_sample_hop_impl(const heta_graph *g, int32_t n, const int32_t *rels, const int64_t *const *dst_ids, const int64_t *n_dst,
                                        int32_t fanout, const uint64_t *seeds, int64_t *const *rowptr, int64_t *const *src_ids,
                                        int32_t *const *local, int64_t *n_sampled, int64_t *const *unique_ids, int64_t *n_unique, void *hip_stream)
{
    if (!g || n < 0 || (n > 0 && (!rels || !dst_ids || !n_dst || !seeds || !rowptr || !src_ids || !local || !n_sampled || !unique_ids || !n_unique)))
        return fail(HETA_ERR_INVALID_ARG, "heta_sample_hop: null argument");
    if (fanout < 1 || fanout > kMaxFanout) return fail(HETA_ERR_SHAPE, "heta_sample_hop: need 1 <= fanout <= %d", kMaxFanout);
    const int32_t n_types = static_cast<int32_t>(g->ntypes.size());
    std::vector<int64_t> cap(n_types, 0); // sampled edges per source type, at most
    int64_t all_dst = 0, cap_max = 0;
    for (int32_t i = 0; i < n; ++i) {
        if (rels[i] < 0 || rels[i] >= (int32_t)g->rels.size()) return fail(HETA_ERR_INVALID_ARG, "heta_sample_hop: relation %d out of range", rels[i]);
        if (n_dst[i] < 0) return fail(HETA_ERR_SHAPE, "heta_sample_hop: need n_dst >= 0");
        if (!rowptr[i] || (n_dst[i] > 0 && (!dst_ids[i] || !src_ids[i] || !local[i]))) return fail(HETA_ERR_INVALID_ARG, "heta_sample_hop: null argument");
        if (n_dst[i] >= (int64_t(1) << 31)) return fail(HETA_ERR_UNSUPPORTED, "heta_sample_hop: more than 2^31 destinations");
        all_dst += n_dst[i];
        cap[g->rels[rels[i]].src_type] += n_dst[i] * fanout;
        cap_max = std::max(cap_max, n_dst[i] * fanout);
    }
    if (n == 0) return HETA_OK;
    int64_t tiles = 0;
    for (int32_t t = 0; t < n_types; ++t) {
        if (cap[t] > 0 && !unique_ids[t]) return fail(HETA_ERR_INVALID_ARG, "heta_sample_hop: null unique_ids");
        if (cap[t] > 0) tiles += std::max<int64_t>(1, (g->ntypes[t].num_nodes + kBitTile - 1) / kBitTile);
        n_unique[t] = 0;
    }
    for (int32_t i = 0; i < n; ++i) n_sampled[i] = 0;
    heta_status e;
    if (n > kFusedItems || n_types > kFusedItems || tiles > kBitTilesMax || all_dst >= (int64_t(1) << 31) / kMaxFanout) {
        // as the two calls that this one stands for
        if ((e = heta_sample_neighbors_batch(g, n, rels, dst_ids, n_dst, fanout, seeds, rowptr, src_ids, n_sampled, hip_stream)) != HETA_OK) return e;
        std::vector<int32_t> first(1, 0);
        std::vector<const int64_t *> lists;
        std::vector<int64_t> lens, limit;
        std::vector<int32_t *> loc;
        for (int32_t t = 0; t < n_types; ++t) {
            for (int32_t i = 0; i < n; ++i)
                if (g->rels[rels[i]].src_type == t) {
                    lists.push_back(src_ids[i]);
                    lens.push_back(n_sampled[i]);
                    loc.push_back(local[i]);
                }
            first.push_back(static_cast<int32_t>(lists.size()));
            limit.push_back(g->ntypes[t].num_nodes);
        }
        return heta_unique_relabel_batch_impl(n_types, first.data(), lists.data(), lens.data(), limit.data(), unique_ids, n_unique, loc.data(), hip_stream);
    }
    hipStream_t st = as_stream(hip_stream);
    FusedSample f{};
    sample_plan(f, g, n, rels, dst_ids, n_dst, fanout, seeds, rowptr, src_ids);
    const size_t words = static_cast<size_t>(tiles) * 256;
    Scratch scratch;
    if ((e = scratch.alloc(sample_scratch_bytes(f.chunk0[n]) + Scratch::padded(words * 8) + Scratch::padded(words * 4) +
                           Scratch::padded(static_cast<size_t>(tiles) * 4))) != HETA_OK ||
        (e = slots_reserve(kBackSlots + static_cast<size_t>(n_types))) != HETA_OK)
        return e;
    unsigned long long *bits = scratch.take<unsigned long long>(words);
    uint32_t *word_rank = scratch.take<uint32_t>(words), *tile_count = scratch.take<uint32_t>(static_cast<size_t>(tiles));
    SampleBack *back = reinterpret_cast<SampleBack *>(t_slots.p);
    int64_t *h_counts = reinterpret_cast<int64_t *>(t_slots.p + kBackSlots);
    int *h_bad = reinterpret_cast<int *>(h_counts + n_types); // the ids are the graph's own, in range
    BitSets b{};
    b.n_sets = n_types;
    tiles = 0;
    for (int32_t t = 0; t < n_types; ++t) {
        h_bad[t] = 0;
        b.tile0[t] = static_cast<int32_t>(tiles);
        if (cap[t] > 0) tiles += std::max<int64_t>(1, (g->ntypes[t].num_nodes + kBitTile - 1) / kBitTile);
        b.limit[t] = g->ntypes[t].num_nodes;
        b.uniq[t] = unique_ids[t];
    }
    b.tile0[n_types] = static_cast<int32_t>(tiles);
    for (int32_t i = 0; i < n; ++i) {
        b.ids[i] = src_ids[i];
        b.local[i] = local[i];
        b.len_at[i] = rowptr[i] + n_dst[i];
        b.set_of[i] = static_cast<uint8_t>(g->rels[rels[i]].src_type);
    }
    if ((e = sample_launch(f, scratch, back, reinterpret_cast<uint4 *>(bits), static_cast<int64_t>(words / 2), st)) != HETA_OK) return e;
    if ((e = bits_launch(b, n, cap_max, bits, word_rank, tile_count, h_counts, h_bad, st)) != HETA_OK) return e;
    HETA_HIP(hipStreamSynchronize(st));
    scratch.idle = true;
    if ((e = sample_results(g, back, n, rels, n_sampled)) != HETA_OK) return e;
    for (int32_t t = 0; t < n_types; ++t) n_unique[t] = cap[t] > 0 ? h_counts[t] : 0;
    return HETA_OK;
}

heta_status heta_sample_hop(const heta_graph *g, int32_t n, const int32_t *rels, const int64_t *const *dst_ids, const int64_t *n_dst, int32_t fanout,
                            const uint64_t *seeds, int64_t *const *rowptr, int64_t *const *src_ids, int32_t *const *local, int64_t *n_sampled,
                            int64_t *const *unique_ids, int64_t *n_unique, void *hip_stream)
{
    try {
        return heta_sample_hop_impl(g, n, rels, dst_ids, n_dst, fanout, seeds, rowptr, src_ids, local, n_sampled, unique_ids, n_unique, hip_stream);
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_sample_hop: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_sample_hop: unexpected exception");
    }
}

heta_status heta_unique_relabel(int32_t n_lists, const int64_t *const *lists, const int64_t *lens, int64_t id_limit,
                                int64_t *unique_ids, int64_t *n_unique, int32_t *const *local, void *hip_stream)
{
    if (n_lists < 0 || !n_unique) return fail(HETA_ERR_INVALID_ARG, "heta_unique_relabel: null argument");
    const int32_t group_ptr[2] = {0, n_lists};
    return heta_unique_relabel_batch(1, group_ptr, lists, lens, &id_limit, &unique_ids, n_unique, local, hip_stream);
}

} // extern "C"
