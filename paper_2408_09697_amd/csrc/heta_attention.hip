// Graph attention as the relation-specific aggregation (R-GAT, Section 2.1 of the paper: one GAT
// module per mono-relation subgraph, outputs summed over the relations and activated by ReLU).
// The module is the attention layer of the GAT paper (Velickovic et al. 2018, Eqs. 1-4, multi-head
// concatenation) on a bipartite relation with K heads of width F:
//
//     s_e[k]     = LeakyReLU(el[u_e, k] + er[v_e, k])
//     alpha_e[k] = exp(s_e[k]) / sum_{e' into v_e} exp(s_e'[k])
//     o[v, kF+f] = sum_{e into v} alpha_e[k] z[u_e, kF+f]
//
// el = <z_u[k,:], a[k,:]> and er = <h_v, q[k,:]> are row scores computed by attn_score_kernel.
//
// Split of the work: everything that touches only scalars per edge (logits, softmax statistics, the
// weights alpha, their LeakyReLU-gated form) runs in "row sweep" kernels over the schedule-ordered
// adjacency and leaves one weight per (edge slot, head) in a workspace; everything that moves feature
// rows is then the ordinary segmented gather-reduce with those weights (aggregate_slot_weighted), so
// the hub-chunk / long-row / equal-degree-batch scheduling is shared with the R-GCN aggregation.
//
// Backward, for upstream gradient g = dL/do, with dot[v,k] = <g[v,k,:], o[v,k,:]>:
//     dz[u]     = sum_{e out of u} alpha_e g[v_e]                           (CSC gather, weights alpha)
//     gate_e    = alpha_e * LeakyReLU'(el + er)
//     der[v,k]  = sum_{e into v} gate_e (<g[v], z[u_e]>_k - dot[v,k])
//               = <g[v], sum_e gate_e z[u_e]>_k - dot[v,k] sum_e gate_e      (CSR gather, weights gate)
//     del[u,k]  = <z[u], sum_{e out of u} gate_e g[v_e]>_k - sum_e gate_e dot[v_e,k]   (CSC gather, weights gate)
// i.e. the per-edge dot products of the softmax backward collapse, by linearity, into weighted
// aggregations followed by one per-row, per-head dot product.  No atomics anywhere.
#include <algorithm>
#include <new>
#include <vector>

#include "heta_internal.h"

namespace heta {

namespace {

using bf16_t = uint16_t;
constexpr int kMaxHeads = 16;
constexpr int kShortDegAttn = 32; // same split as the aggregation: from here on, a wavefront per row
constexpr int kThreadDegAttn = 4; // up to here, one thread per row

__device__ __forceinline__ float lrelu(float x, float slope) { return x > 0.f ? x : slope * x; }

// ---- row sweeps ------------------------------------------------------------------------------------------
// One sweep touches only scalars: per edge slot of a schedule the neighbour's id, KT consecutive heads of its
// score (one vector load), and the per-slot weights it writes.  A sweep is bound by the latency of its gathers, so
// a row gets as many lanes as bring it down to a few loads per lane, all in flight together:
//   rows of up to 4 edges: one thread per row; 5..31: eight lanes per row; 32..511: one wavefront per row;
//   hub rows (>= 512 edges): one wavefront per 256-edge chunk writes partial statistics, a second kernel
//   combines a row's chunks in chunk order, and (forward only) a third writes the weights.
// The first three and the hub chunks share one launch.  The forward keeps a row's logits in registers from the
// gather to the weights.  (One thread per row below 32 edges, one gather per phase and a launch per row class:
// 0.4 M edges into 70,000 rows of a power-law relation, 8 heads: forward 106 us, now 35 us; all sweeps of a 4-head
// layer over 21 M edges 2.7 ms, now 1.75 ms.)
enum SweepOp { SWEEP_FWD = 0, SWEEP_BWD_CSR = 1, SWEEP_BWD_CSC = 2 };
enum Phase { PH_ALPHA = 0, PH_BWD_DST = 1 };

struct SweepParams {
    const int64_t *sptr;
    const int32_t *sidx;
    const int32_t *perm;
    const HubChunk *hub_chunks;
    const int64_t *hub_chunk_ptr;
    int64_t n_hub_rows, n_hub_chunks;
    // schedule positions [0, q_wave) are hub rows, then one wavefront per row, from q_mid on eight lanes, from
    // q_short on one thread; first workgroup of each class in the shared launch (hub chunks first)
    int64_t q_wave, q_mid, q_short, n_rows;
    unsigned b_wave, b_mid, b_short;
    unsigned b_first;     // first workgroup of this launch
    int K;
    float slope;
    const float *row_a;   // [rows][K]  score half of the row side (er for the CSR, el for the CSC)
    const float *nbr_a;   // [nbrs][K]  score half of the neighbour side
    float *smax, *sinv;   // [dst][K]   softmax shift and 1/denominator: written by FWD (nullable), read by the others
    const float *dot;     // [dst][K]   <g, o> per head (backward)
    float *alpha;         // [E][K] by edge slot (FWD, BWD_CSC)
    int sign;             // FWD: alpha's sign bit is set where the logit is not positive.  BWD_CSC always sets it.  Weights
                          // restricted to positive logits, or times LeakyReLU', are then read off the one array
    float *gate;          // [E][K] by edge slot: alpha * LeakyReLU' (BWD_CSR, if non-null)
    float dot_shift;      // BWD_CSR: corr = dot * (sum of gates - dot_shift)
    float *corr;          // [rows][K]  the scalar term subtracted from the row's score gradient (BWD_*)
    const float *nbr_pack; // BWD_CSC: [dst][K][4] = er, smax, sinv, dot of the destination's head (one cache line per
                          // neighbour instead of four gathers, one 16-byte load per head)
    float *apos;          // [dst][K]   sum of alpha over the edges with a positive logit (FWD, nullable)
    float *part;          // hub chunks: [n_hub_chunks][K][3] partial statistics
    float *hub_stat;      // hub rows (FWD): [n_hub_rows][K][2] = shift, 1/denominator
};

template <int KT> __device__ __forceinline__ void loadk(const float *p, float *v);
template <> __device__ __forceinline__ void loadk<1>(const float *p, float *v) { v[0] = *p; }
template <> __device__ __forceinline__ void loadk<2>(const float *p, float *v)
{
    const float2 t = *reinterpret_cast<const float2 *>(p);
    v[0] = t.x; v[1] = t.y;
}
template <> __device__ __forceinline__ void loadk<4>(const float *p, float *v)
{
    const float4 t = *reinterpret_cast<const float4 *>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
template <> __device__ __forceinline__ void loadk<8>(const float *p, float *v)
{
    loadk<4>(p, v);
    loadk<4>(p + 4, v + 4);
}
template <int KT> __device__ __forceinline__ void storek(float *p, const float *v);
template <> __device__ __forceinline__ void storek<1>(float *p, const float *v) { *p = v[0]; }
template <> __device__ __forceinline__ void storek<2>(float *p, const float *v) { *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]); }
template <> __device__ __forceinline__ void storek<4>(float *p, const float *v)
{
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
}

template <> __device__ __forceinline__ void storek<8>(float *p, const float *v)
{
    storek<4>(p, v);
    storek<4>(p + 4, v + 4);
}

// a weight (>= 0 or NaN) whose sign bit says that its logit is not positive
__device__ __forceinline__ float signed_weight(float a, bool up) { return __uint_as_float((__float_as_uint(a) & 0x7fffffffu) | (up ? 0u : 0x80000000u)); }

// One edge slot e, heads k0 .. k0+KT-1.  ar: the row's score half; m, inv: shift and 1/denominator of the
// row; acc: running sum.
template <int KT, int PH>
__device__ __forceinline__ void visit(const SweepParams &p, int64_t e, int k0, const float *ar, const float *m,
                                      const float *inv, float *acc)
{
    const int64_t id = p.sidx[e];
    float x[KT];
    loadk<KT>(p.nbr_a + id * p.K + k0, x);
    float a[KT], gt[KT];
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        x[k] += ar[k];
        const float sc = lrelu(x[k], p.slope);
        if (PH == PH_ALPHA) {
            a[k] = expf(sc - m[k]) * inv[k];
            if (p.sign) a[k] = signed_weight(a[k], x[k] > 0.f);
        } else {
            gt[k] = expf(sc - m[k]) * inv[k] * (x[k] > 0.f ? 1.f : p.slope);
            acc[k] += gt[k];
        }
    }
    if (PH == PH_ALPHA) storek<KT>(p.alpha + e * p.K + k0, a);
    if (PH == PH_BWD_DST && p.gate) storek<KT>(p.gate + e * p.K + k0, gt);
}

// the slots e0 + lane, e0 + lane + W, ...
template <int W, int KT, int PH>
__device__ __forceinline__ void sweep_range(const SweepParams &p, int64_t e0, int64_t e1, int lane, int k0, const float *ar,
                                            const float *m, const float *inv, float *acc)
{
#pragma unroll KT >= 8 ? 2 : 4
    for (int64_t e = e0 + lane; e < e1; e += W) visit<KT, PH>(p, e, k0, ar, m, inv, acc);
}

// over the W lanes of a row's group
template <int W, int KT> __device__ __forceinline__ void group_sum(float *v)
{
#pragma unroll
    for (int k = 0; k < KT; ++k)
#pragma unroll
        for (int off = W / 2; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
}
template <int W, int KT> __device__ __forceinline__ void group_max(float *v)
{
#pragma unroll
    for (int k = 0; k < KT; ++k)
#pragma unroll
        for (int off = W / 2; off > 0; off >>= 1) v[k] = fmaxf(v[k], __shfl_xor(v[k], off, 64));
}

// Forward statistics of up to W NPL edges from slot e0, W lanes, NPL slots per lane: every id and score is loaded
// once.  Left in x: exp(LeakyReLU(logit) - m), its sign bit set where the logit itself is not positive (the activation
// keeps the sign only for a positive slope; a bit, not a product with -1, so that a NaN keeps it as well); m: the largest
// activated logit (-inf without edges), den and pos: the sums of all exps and of those of positive logits, in every
// lane of the group.
template <int W, int KT, int NPL>
__device__ __forceinline__ void fwd_stats(const SweepParams &p, int64_t e0, int n, int lane, int k0, const float *ar, float (&x)[NPL][KT],
                                          float *m, float *den, float *pos)
{
    int64_t id[NPL];
#pragma unroll
    for (int j = 0; j < NPL; ++j) id[j] = lane + j * W < n ? p.sidx[e0 + lane + j * W] : -1;
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
#pragma unroll
        for (int k = 0; k < KT; ++k) x[j][k] = 0.f;
        if (id[j] >= 0) loadk<KT>(p.nbr_a + id[j] * p.K + k0, x[j]);
    }
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        m[k] = -INFINITY;
        den[k] = pos[k] = 0.f;
    }
#pragma unroll
    for (int j = 0; j < NPL; ++j)
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            x[j][k] += ar[k];
            if (id[j] >= 0) m[k] = fmaxf(m[k], lrelu(x[j][k], p.slope));
        }
    group_max<W, KT>(m);
#pragma unroll
    for (int j = 0; j < NPL; ++j)
#pragma unroll
        for (int k = 0; k < KT; ++k) {
            const bool up = x[j][k] > 0.f;
            const float e = id[j] >= 0 ? expf(lrelu(x[j][k], p.slope) - m[k]) : 0.f;
            den[k] += e;
            pos[k] += up ? e : 0.f;
            x[j][k] = signed_weight(e, up);
        }
    group_sum<W, KT>(den);
    group_sum<W, KT>(pos);
}

// Forward of one row: W lanes, at most W NPL edges.
template <int W, int KT, int NPL>
__device__ __forceinline__ void fwd_row(const SweepParams &p, int64_t row, int64_t e0, int n, bool live, int lane, int k0, const float *ar)
{
    float x[NPL][KT], m[KT], inv[KT], den[KT], pos[KT];
    fwd_stats<W, KT, NPL>(p, e0, n, lane, k0, ar, x, m, den, pos);
    const bool empty = n == 0;
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        inv[k] = empty ? 0.f : 1.f / den[k];
        if (empty) m[k] = 0.f;
        pos[k] = empty ? 0.f : pos[k] * inv[k];
    }
#pragma unroll
    for (int j = 0; j < NPL; ++j) {
        if (lane + j * W < n) {
            float a[KT];
#pragma unroll
            for (int k = 0; k < KT; ++k) a[k] = signed_weight(fabsf(x[j][k]) * inv[k], !p.sign || __float_as_uint(x[j][k]) >> 31 == 0);
            storek<KT>(p.alpha + (e0 + lane + j * W) * p.K + k0, a);
        }
    }
    if (live && lane == 0 && p.smax) {
        storek<KT>(p.smax + row * p.K + k0, m);
        storek<KT>(p.sinv + row * p.K + k0, inv);
    }
    if (live && lane == 0 && p.apos) storek<KT>(p.apos + row * p.K + k0, pos);
}

// Source side of the backward: a lane has one head of a slot, so that a neighbour's terms arrive as one piece of 16 KT bytes.
// A load instruction costs the cache lines that it touches, and a lane that loads all heads of its slot touches its line KT
// times: this sweep over 2.1 M edges of seven relations, 8 heads, 97 -> 68 us (76 with five wavefronts per SIMD instead
// of six); over 21 M edges, 4 heads, 495 -> 489, and 514 with the short rows one at a time.
// U slots (j, j + step, ..) of each of R rows of n slots from e0 on, all loads in flight together; acc: the head's sums.
template <int R, int U>
__device__ __forceinline__ void bwd_src_slots(const SweepParams &p, const int64_t (&e0)[R], const int (&n)[R], int j, int step, int k, const float (&ar)[R],
                                              float (&acc)[R])
{
    const float4 *pk = reinterpret_cast<const float4 *>(p.nbr_pack);
    int32_t id[R][U];
    float4 t[R][U];
    float term[U];
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (n[r] > 0) { // slots past the end repeat the last one
#pragma unroll
            for (int u = 0; u < U; ++u) id[r][u] = p.sidx[e0[r] + min(j + u * step, n[r] - 1)];
        }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (n[r] > 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) t[r][u] = pk[static_cast<int64_t>(id[r][u]) * p.K + k];
        }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float x = t[r][u].x + ar[r], a = expf(lrelu(x, p.slope) - t[r][u].y) * t[r][u].z;
            const bool given = j + u * step < n[r];
            term[u] = given ? a * (x > 0.f ? 1.f : p.slope) * t[r][u].w : 0.f;
            if (given) p.alpha[(e0[r] + j + u * step) * p.K + k] = signed_weight(a, x > 0.f);
        }
#pragma unroll
        for (int w = U / 2; w > 0; w /= 2)
#pragma unroll
            for (int u = 0; u < w; ++u) term[u] += term[u + w];
        acc[r] += term[0];
    }
}

// n slots from e0 on, G lanes; returns the head's sum in all of them
template <int G, int KT, int U> __device__ __forceinline__ float bwd_src_edges(const SweepParams &p, int64_t e0, int n, int lane, int k, float ar)
{
    constexpr int EP = G / KT;
    const int64_t e[1] = {e0};
    const int nn[1] = {n};
    const float arr[1] = {ar};
    float acc[1] = {0.f};
    for (int j = lane / KT; j < n; j += EP * U) bwd_src_slots<1, U>(p, e, nn, j, EP, k, arr, acc);
#pragma unroll
    for (int off = G / 2; off >= KT; off >>= 1) acc[0] += __shfl_xor(acc[0], off, 64);
    return acc[0];
}

// One row of it, G lanes.
template <int G, int KT, int U> __device__ __forceinline__ void bwd_src_row(const SweepParams &p, int64_t q, bool live, int lane, int k0)
{
    const int64_t row = live ? p.perm[q] : 0, e0 = live ? p.sptr[q] : 0, e1 = live ? p.sptr[q + 1] : 0;
    const int k = k0 + lane % KT;
    const float sum = bwd_src_edges<G, KT, U>(p, e0, static_cast<int>(e1 - e0), lane, k, p.row_a[row * p.K + k]);
    if (live && lane < KT) p.corr[row * p.K + k] = sum;
}

// Rows of up to four edges: KT lanes per row, KT rows each (q + 256 / KT i), R of them at a time.
template <int KT> __device__ __forceinline__ void bwd_src_short(const SweepParams &p, int64_t q0, int k)
{
    constexpr int R = KT < 2 ? 1 : 2;
    for (int i = 0; i < KT; i += R) {
        int64_t row[R], e0[R];
        int n[R];
        float ar[R], acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t q = q0 + (i + r) * (256 / KT), qc = min(q, p.n_rows - 1);
            row[r] = p.perm[qc];
            e0[r] = p.sptr[qc];
            n[r] = q < p.n_rows ? static_cast<int>(p.sptr[qc + 1] - e0[r]) : -1;
            acc[r] = 0.f;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) ar[r] = p.row_a[row[r] * p.K + k];
        bwd_src_slots<R, 4>(p, e0, n, 0, 1, k, ar, acc);
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (n[r] >= 0) p.corr[row[r] * p.K + k] = acc[r];
    }
}

// One row: W lanes, at most W NPL edges.
template <int W, int KT, int NPL, int OP>
__device__ __forceinline__ void sweep_row(const SweepParams &p, int64_t q, bool live, int lane, int k0)
{
    const int64_t row = live ? p.perm[q] : 0;
    const int64_t e0 = live ? p.sptr[q] : 0, e1 = live ? p.sptr[q + 1] : 0;
    float ar[KT], acc[KT], m[KT], inv[KT];
    loadk<KT>(p.row_a + row * p.K + k0, ar);
    if (OP == SWEEP_FWD) {
        // Only as many slots per lane as the row needs (uniform per wavefront), the same bits whichever runs: an empty slot
        // costs its exponentials all the same (whole forwards of 20,000 rows of 40 edges, 8 heads 103 -> 69 us, 16 heads
        // 200 -> 136; 100,000 rows of one edge, 8 heads 23.0 -> 21.0).
        const int n = static_cast<int>(e1 - e0);
        if (W == 64 && n <= 64) fwd_row<W, KT, 1>(p, row, e0, n, live, lane, k0, ar);
        else if (W == 64 && n <= 128) fwd_row<W, KT, 2>(p, row, e0, n, live, lane, k0, ar);
        else if (W == 64 && n <= 256) fwd_row<W, KT, 4>(p, row, e0, n, live, lane, k0, ar);
        else if (W == 1 && !__any(n > 1)) fwd_row<W, KT, 1>(p, row, e0, n, live, lane, k0, ar);
        else fwd_row<W, KT, NPL>(p, row, e0, n, live, lane, k0, ar);
    } else {
#pragma unroll
        for (int k = 0; k < KT; ++k) acc[k] = 0.f;
        loadk<KT>(p.smax + row * p.K + k0, m);
        loadk<KT>(p.sinv + row * p.K + k0, inv);
        sweep_range<W, KT, PH_BWD_DST>(p, e0, e1, lane, k0, ar, m, inv, acc);
        group_sum<W, KT>(acc);
        if (live && lane == 0) {
            float d[KT];
            loadk<KT>(p.dot + row * p.K + k0, d);
#pragma unroll
            for (int k = 0; k < KT; ++k) acc[k] = (acc[k] - p.dot_shift) * d[k];
            storek<KT>(p.corr + row * p.K + k0, acc);
        }
    }
}

// hub row of chunk w: the h with hub_chunk_ptr[h] <= w < hub_chunk_ptr[h + 1]
__device__ __forceinline__ int64_t hub_of_chunk(const SweepParams &p, int64_t w)
{
    int64_t lo = 0, hi = p.n_hub_rows; // invariant: ptr[lo] <= w < ptr[hi]
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if (p.hub_chunk_ptr[mid] <= w) lo = mid;
        else hi = mid;
    }
    return lo;
}

// hub chunks, first kernel: partial statistics of one chunk (and the backward's weights)
template <int KT, int OP> __device__ __forceinline__ void sweep_hub_chunk(const SweepParams &p, int64_t w, int lane, int k0)
{
    static_assert(kHubChunk == 256, "four slots per lane");
    const HubChunk c = p.hub_chunks[w];
    const int64_t row = p.perm[hub_of_chunk(p, w)];
    const int64_t e0 = c.e0, e1 = c.e0 + c.len;
    float ar[KT], acc[KT], m[KT], inv[KT];
    float *out = p.part + (w * p.K + k0) * 3;
    if constexpr (OP == SWEEP_BWD_CSC) {
        const int k = k0 + lane % KT;
        const float sum = bwd_src_edges<64, KT, KT >= 4 ? 8 : 4>(p, e0, c.len, lane, k, p.row_a[row * p.K + k]);
        if (lane < KT) out[3 * lane] = sum;
        return;
    }
    loadk<KT>(p.row_a + row * p.K + k0, ar);
    if (OP == SWEEP_FWD) {
        float x[4][KT], pos[KT];
        fwd_stats<64, KT, 4>(p, e0, static_cast<int>(e1 - e0), lane, k0, ar, x, m, acc, pos);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < KT; ++k) {
                out[3 * k] = m[k];
                out[3 * k + 1] = acc[k];
                out[3 * k + 2] = pos[k];
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < KT; ++k) acc[k] = 0.f;
        loadk<KT>(p.smax + row * p.K + k0, m);
        loadk<KT>(p.sinv + row * p.K + k0, inv);
        sweep_range<64, KT, PH_BWD_DST>(p, e0, e1, lane, k0, ar, m, inv, acc);
        group_sum<64, KT>(acc);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < KT; ++k) out[3 * k] = acc[k];
        }
    }
}

// Up to N relations of one call; first: the first workgroup of each in a launch over all of them.
constexpr int kSweepMulti = 8;
template <int N> struct SweepMulti {
    SweepParams p[N];
    unsigned first[N];
};
static_assert(sizeof(SweepMulti<kSweepMulti>) <= 3840, "kernel arguments are limited to 4 KB");

// All row classes of all schedules in one launch: relation and class follow from the workgroup's index (uniform).  Six wavefronts per
// SIMD on the source side: with seven its gathers spill.
template <int KT, int OP, int N>
__global__ void __launch_bounds__(256, OP == SWEEP_BWD_CSC ? 6 : 1) attn_rows_kernel(SweepMulti<N> m)
{
    int i = 0;
#pragma unroll
    for (int j = 1; j < N; ++j) i += blockIdx.x >= m.first[j] ? 1 : 0;
    const SweepParams &p = m.p[i];
    const int lane = threadIdx.x & 63;
    const int k0 = blockIdx.y * KT;
    const unsigned b = p.b_first + (blockIdx.x - m.first[i]);
    if (b < p.b_wave) {
        const int64_t w = static_cast<int64_t>(b) * 4 + (threadIdx.x >> 6);
        if (w < p.n_hub_chunks) sweep_hub_chunk<KT, OP>(p, w, lane, k0); // uniform per wavefront
    } else if (b < p.b_mid) {
        const int64_t q = p.q_wave + static_cast<int64_t>(b - p.b_wave) * 4 + (threadIdx.x >> 6);
        if (q < p.q_mid) {
            if constexpr (OP == SWEEP_BWD_CSC) bwd_src_row<64, KT, KT >= 4 ? 8 : 4>(p, q, true, lane, k0);
            else sweep_row<64, KT, 8, OP>(p, q, true, lane, k0);
        }
    } else if (b < p.b_short) {
        const int64_t q = p.q_mid + static_cast<int64_t>(b - p.b_mid) * 32 + (threadIdx.x >> 3);
        // every lane of the wavefront takes part in the sums
        if constexpr (OP == SWEEP_BWD_CSC) bwd_src_row<8, KT, KT >= 4 ? 8 : 4>(p, q, q < p.q_short, threadIdx.x & 7, k0);
        else sweep_row<8, KT, 4, OP>(p, q, q < p.q_short, threadIdx.x & 7, k0);
    } else if constexpr (OP == SWEEP_BWD_CSC) {
        bwd_src_short<KT>(p, p.q_short + static_cast<int64_t>(b - p.b_short) * 256 + threadIdx.x / KT, k0 + threadIdx.x % KT);
    } else {
        const int64_t q = p.q_short + static_cast<int64_t>(b - p.b_short) * 256 + threadIdx.x;
        if (q < p.n_rows) sweep_row<1, KT, 4, OP>(p, q, true, 0, k0);
    }
}

// hub rows, second kernel: one wavefront per (hub row, head) combines the row's chunks in chunk order
// (blockIdx.z: the relation)
template <int OP, int N>
__global__ void __launch_bounds__(256) attn_hub_combine_kernel(SweepMulti<N> m)
{
    const SweepParams &p = m.p[blockIdx.z];
    const int lane = threadIdx.x & 63;
    const int64_t h = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (h >= p.n_hub_rows) return;
    const int k = blockIdx.y;
    const int64_t row = p.perm[h];
    const int64_t s0 = p.hub_chunk_ptr[h], s1 = p.hub_chunk_ptr[h + 1];
    if (OP == SWEEP_FWD) {
        float m = -INFINITY;
        for (int64_t s = s0 + lane; s < s1; s += 64) m = fmaxf(m, p.part[(s * p.K + k) * 3]);
        group_max<64, 1>(&m);
        float den = 0.f, pos = 0.f;
        for (int64_t s = s0 + lane; s < s1; s += 64) {
            const float *t = p.part + (s * p.K + k) * 3;
            const float e = expf(t[0] - m);
            den += t[1] * e;
            pos += t[2] * e;
        }
        group_sum<64, 1>(&den);
        group_sum<64, 1>(&pos);
        if (lane == 0) {
            const float inv = 1.f / den; // a hub row has edges
            p.hub_stat[(h * p.K + k) * 2] = m;
            p.hub_stat[(h * p.K + k) * 2 + 1] = inv;
            if (p.smax) {
                p.smax[row * p.K + k] = m;
                p.sinv[row * p.K + k] = inv;
            }
            if (p.apos) p.apos[row * p.K + k] = pos * inv;
        }
    } else {
        float a = 0.f;
        for (int64_t s = s0 + lane; s < s1; s += 64) a += p.part[(s * p.K + k) * 3];
        group_sum<64, 1>(&a);
        if (lane == 0) p.corr[row * p.K + k] = OP == SWEEP_BWD_CSR ? (a - p.dot_shift) * p.dot[row * p.K + k] : a;
    }
}

// hub chunks, third kernel (forward): the weights, from the combined statistics
template <int KT, int N>
__global__ void __launch_bounds__(256) attn_hub_alpha_kernel(SweepMulti<N> all)
{
    const SweepParams &p = all.p[blockIdx.z];
    const int lane = threadIdx.x & 63;
    const int64_t w = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (w >= p.n_hub_chunks) return;
    const int k0 = blockIdx.y * KT;
    const HubChunk c = p.hub_chunks[w];
    const int64_t h = hub_of_chunk(p, w);
    const int64_t row = p.perm[h];
    float ar[KT], m[KT], inv[KT];
    loadk<KT>(p.row_a + row * p.K + k0, ar);
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        m[k] = p.hub_stat[(h * p.K + k0 + k) * 2];
        inv[k] = p.hub_stat[(h * p.K + k0 + k) * 2 + 1];
    }
    sweep_range<64, KT, PH_ALPHA>(p, c.e0, c.e0 + c.len, lane, k0, ar, m, inv, nullptr);
}

// pack[v][k] = er, smax, sinv, dot of (v, k)
__global__ void __launch_bounds__(256) attn_pack_kernel(const float *er, const float *smax, const float *sinv, const float *dot, int64_t total,
                                                        float4 *pack)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (t < total) pack[t] = make_float4(er[t], smax[t], sinv[t], dot[t]);
}

inline size_t hub_scratch_bytes(const Schedule &s, int K)
{
    return static_cast<size_t>(s.n_hub_chunks * 3 + s.n_hub_rows * 2) * K * sizeof(float);
}

// One sweep of a call: the schedule, its parameters, and hub_scratch_bytes of device memory for the hub rows' statistics.
struct Sweep {
    const Schedule *s;
    SweepParams p;
    float *hub_scratch;
    int64_t blocks; // filled in below
};

template <int KT, int OP, int N>
heta_status launch_sweeps_n(const Sweep *sw, int n, hipStream_t st)
{
    SweepMulti<N> m{};
    int64_t total = 0, hub_rows = 0, hub_blocks = 0;
    for (int i = 0; i < N; ++i) {
        m.first[i] = static_cast<unsigned>(total);
        if (i >= n) {
            m.first[i] = 0xffffffffu; // no workgroup reaches it
            continue;
        }
        m.p[i] = sw[i].p;
        total += sw[i].blocks;
        hub_rows = std::max(hub_rows, sw[i].s->n_hub_rows);
        hub_blocks = std::max(hub_blocks, (sw[i].s->n_hub_chunks + 3) / 4);
    }
    const unsigned K = sw[0].p.K, gy = K / KT;
    if (N == 1) {
        // (eight lanes per row: 2^29 rows of 5 to 31 edges are more threads than a grid takes)
        launch_pieces(total, 256, [&](unsigned first, unsigned count) {
            m.p[0].b_first = first;
            hipLaunchKernelGGL((attn_rows_kernel<KT, OP, N>), dim3(count, gy), dim3(256), 0, st, m);
        });
    } else {
        hipLaunchKernelGGL((attn_rows_kernel<KT, OP, N>), dim3((unsigned)total, gy), dim3(256), 0, st, m);
    }
    HETA_LAUNCH_CHECK("attn_rows_kernel");
    if (hub_rows > 0) {
        hipLaunchKernelGGL((attn_hub_combine_kernel<OP, N>), dim3((unsigned)((hub_rows + 3) / 4), K, n), dim3(256), 0, st, m);
        HETA_LAUNCH_CHECK("attn_hub_combine_kernel");
        if (OP == SWEEP_FWD) {
            hipLaunchKernelGGL((attn_hub_alpha_kernel<KT, N>), dim3((unsigned)hub_blocks, gy, n), dim3(256), 0, st, m);
            HETA_LAUNCH_CHECK("attn_hub_alpha_kernel");
        }
    }
    return HETA_OK;
}

template <int KT, int OP>
heta_status launch_sweeps_kt(Sweep *sw, int n, hipStream_t st)
{
    int64_t total = 0;
    for (int i = 0; i < n; ++i) {
        const Schedule &s = *sw[i].s;
        SweepParams &p = sw[i].p;
        p.q_wave = s.n_hub_rows;
        p.q_mid = s.rows_with_deg_ge[kShortDegAttn];
        p.q_short = s.rows_with_deg_ge[kThreadDegAttn + 1];
        p.n_rows = s.n_rows;
        const int64_t cb = (s.n_hub_chunks + 3) / 4;
        const int64_t wb = (p.q_mid - p.q_wave + 3) / 4, mb = (p.q_short - p.q_mid + 31) / 32, sb = (p.n_rows - p.q_short + 255) / 256;
        if (cb + wb + mb + sb > 0x7fffffff) return fail(HETA_ERR_UNSUPPORTED, "attention: too many rows");
        p.b_wave = (unsigned)cb;
        p.b_mid = (unsigned)(cb + wb);
        p.b_short = (unsigned)(cb + wb + mb);
        p.b_first = 0;
        sw[i].blocks = cb + wb + mb + sb;
        total += sw[i].blocks;
    }
    if (n > 1 && n <= kSweepMulti && total <= max_blocks(256)) return launch_sweeps_n<KT, OP, kSweepMulti>(sw, n, st);
    for (int i = 0; i < n; ++i) {
        const heta_status e = launch_sweeps_n<KT, OP, 1>(sw + i, 1, st);
        if (e != HETA_OK) return e;
    }
    return HETA_OK;
}

// One kind of sweep over several relations of one head count.
template <int OP>
heta_status launch_sweeps(std::vector<Sweep> &sw, hipStream_t st, const char *name)
{
    sw.erase(std::remove_if(sw.begin(), sw.end(), [](const Sweep &x) { return x.s->n_rows == 0; }), sw.end());
    if (sw.empty()) return HETA_OK;
    const int K = sw[0].p.K;
    double bytes = 0;
    uintptr_t all = 0;
    for (Sweep &x : sw) {
        const Schedule &s = *x.s;
        SweepParams &p = x.p;
        p.sptr = s.d_sptr;
        p.sidx = s.d_sidx;
        p.perm = s.d_perm;
        p.hub_chunks = s.d_hub_chunks;
        p.hub_chunk_ptr = s.d_hub_chunk_ptr;
        p.n_hub_rows = s.n_hub_rows;
        p.n_hub_chunks = s.n_hub_chunks;
        p.part = x.hub_scratch;
        p.hub_stat = x.hub_scratch + s.n_hub_chunks * p.K * 3;
        // Algorithmic bytes: per edge one 4-byte id, per edge and head the neighbour's 4-byte terms and the
        // 4-byte weight written; per row its offsets and per-head terms.
        const double per_edge = 4.0 + K * (OP == SWEEP_BWD_CSC ? 20.0 : 8.0);
        bytes += per_edge * static_cast<double>(s.n_edges) + static_cast<double>(s.n_rows) * (12.0 + 12.0 * K);
        // KT consecutive heads per thread need 4*KT-byte aligned score rows
        all |= reinterpret_cast<uintptr_t>(p.row_a) | reinterpret_cast<uintptr_t>(p.nbr_a) | reinterpret_cast<uintptr_t>(p.smax) |
               reinterpret_cast<uintptr_t>(p.sinv) | reinterpret_cast<uintptr_t>(p.dot) | reinterpret_cast<uintptr_t>(p.nbr_pack) |
               reinterpret_cast<uintptr_t>(p.alpha) | reinterpret_cast<uintptr_t>(p.gate) | reinterpret_cast<uintptr_t>(p.corr) |
               reinterpret_cast<uintptr_t>(p.apos);
    }
    ProfScope prof(name, st, bytes, 0);
    const int n = static_cast<int>(sw.size());
    if (K % 8 == 0 && all % 16 == 0) return launch_sweeps_kt<8, OP>(sw.data(), n, st);
    if (K % 4 == 0 && all % 16 == 0) return launch_sweeps_kt<4, OP>(sw.data(), n, st);
    if (K % 2 == 0 && all % 8 == 0) return launch_sweeps_kt<2, OP>(sw.data(), n, st);
    return launch_sweeps_kt<1, OP>(sw.data(), n, st);
}

// ---- per-row, per-head dot products -------------------------------------------------------------------
// out[i, k] = sum_j x[i, j] y_k[j] - corr[i, k], one wavefront per row.
//   per_head = 1: j runs over head k's columns [kF, (k+1)F); y is a second matrix (ld_y > 0) or one
//                 row shared by every i (ld_y = 0: the attention vector a, laid out [K][F] = [d]).
//   per_head = 0: j runs over all d columns and y_k = y + k*d (a [K][d] matrix shared by every row).
struct DotParams {
    unsigned first; // first workgroup of this launch
    const void *x;
    int64_t ld_x;
    const void *y;
    int64_t ld_y;
    int64_t n;
    int d, K, F, per_head;
    float scale;          // out = scale * <x, y> - corr
    const float *corr;
    float *out;
    // optional second operand with rows of its own (per_head only): out2 = scale2 * <x, y2>, in the same pass over x
    const void *y2;
    float scale2;
    float *out2;
};

template <typename T> __device__ __forceinline__ float ld1(const T *p);
template <> __device__ __forceinline__ float ld1<float>(const float *p) { return *p; }
template <> __device__ __forceinline__ float ld1<bf16_t>(const bf16_t *p) { return __uint_as_float(static_cast<uint32_t>(*p) << 16); }

template <typename T, int EPC> __device__ __forceinline__ void ldv(const T *p, float *f);
template <> __device__ __forceinline__ void ldv<float, 4>(const float *p, float *f)
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}
template <> __device__ __forceinline__ void ldv<float, 1>(const float *p, float *f) { f[0] = *p; }
template <> __device__ __forceinline__ void ldv<bf16_t, 4>(const bf16_t *p, float *f)
{
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
}
template <> __device__ __forceinline__ void ldv<bf16_t, 1>(const bf16_t *p, float *f) { f[0] = ld1(p); }

template <typename TX, typename TY, int EPC>
__global__ void __launch_bounds__(256) attn_rowdot_kernel(DotParams p)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = (static_cast<int64_t>(p.first) + blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (i >= p.n) return; // uniform per wavefront
    const TX *x = static_cast<const TX *>(p.x) + i * p.ld_x;
    const TY *y = static_cast<const TY *>(p.y) + i * p.ld_y;
    float res = 0.f;
    for (int k = 0; k < p.K; ++k) {
        const int j0 = p.per_head ? k * p.F : 0, j1 = p.per_head ? (k + 1) * p.F : p.d;
        const TY *yk = p.per_head ? y : y + static_cast<int64_t>(k) * p.d;
        float part = 0.f;
        for (int j = j0 + lane * EPC; j < j1; j += 64 * EPC) {
            float a[EPC], b[EPC];
            ldv<TX, EPC>(x + j, a);
            ldv<TY, EPC>(yk + j, b);
#pragma unroll
            for (int t = 0; t < EPC; ++t) part = fmaf(a[t], b[t], part);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
        if (lane == k) res = part;
    }
    if (lane < p.K) p.out[i * p.K + lane] = p.scale * res - (p.corr ? p.corr[i * p.K + lane] : 0.f);
}

// Fast path: a row's 16-byte chunks are spread over a group of L lanes (L a power of two, T chunks per
// lane), 64 / L rows per wavefront, every chunk loaded once; the per-head sums are segmented cross-lane
// reductions.  Needs 4-element chunks that do not straddle heads and, per head, a power-of-two number of
// chunks (cph); a head then lies inside one t (cph <= L) or covers whole t's (cph a multiple of L).
template <typename TX, typename TY, int T, int R>
__global__ void __launch_bounds__(256) attn_rowdot_fast_kernel(DotParams p, int L, int cph)
{
    const int lane = threadIdx.x & 63;
    const int G = 64 / L, g = lane / L, l = lane % L;
    const int64_t first = ((static_cast<int64_t>(p.first) + blockIdx.x) * 4 + (threadIdx.x >> 6)) * R * G + g; // rows first, first + G, ...
    const int n_chunks = p.d / 4;
    float xv[R][T][4];
    bool live[R];
    // every load of the wavefront's R row groups is issued before the first use
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = first + static_cast<int64_t>(r) * G;
        live[r] = i < p.n;
        const TX *x = static_cast<const TX *>(p.x) + (live[r] ? i : 0) * p.ld_x;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int c = l + L * t;
            if (live[r] && c < n_chunks) ldv<TX, 4>(x + 4 * c, xv[r][t]);
            else xv[r][t][0] = xv[r][t][1] = xv[r][t][2] = xv[r][t][3] = 0.f;
        }
    }
    if (p.per_head) {
      for (int pass = 0; pass < (p.y2 ? 2 : 1); ++pass) { // uniform: the second operand's rows against the same x registers
        const void *yp = pass ? p.y2 : p.y;
        float *outp = pass ? p.out2 : p.out;
        const float scl = pass ? p.scale2 : p.scale;
        const float *corrp = pass ? nullptr : p.corr;
        float part[R][T];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = first + static_cast<int64_t>(r) * G;
            const TY *y = static_cast<const TY *>(yp) + (live[r] ? i : 0) * p.ld_y;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int c = l + L * t;
                float yv[4] = {0.f, 0.f, 0.f, 0.f};
                if (live[r] && c < n_chunks) ldv<TY, 4>(y + 4 * c, yv);
                part[r][t] = xv[r][t][0] * yv[0] + xv[r][t][1] * yv[1] + xv[r][t][2] * yv[2] + xv[r][t][3] * yv[3];
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = first + static_cast<int64_t>(r) * G;
            if (cph <= L) {
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    for (int off = cph >> 1; off > 0; off >>= 1) part[r][t] += __shfl_xor(part[r][t], off, 64);
                    const int c = l + L * t;
                    if (live[r] && c < n_chunks && (l & (cph - 1)) == 0) {
                        const int k = c / cph;
                        outp[i * p.K + k] = scl * part[r][t] - (corrp ? corrp[i * p.K + k] : 0.f);
                    }
                }
            } else {
                const int m = cph / L; // t's per head
                float acc = 0.f;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    acc += part[r][t];
                    if ((t + 1) % m == 0) {
                        for (int off = L >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
                        const int k = t / m;
                        if (live[r] && l == 0 && k < p.K) outp[i * p.K + k] = scl * acc - (corrp ? corrp[i * p.K + k] : 0.f);
                        acc = 0.f;
                    }
                }
            }
        }
      }
    } else {
        // y_k = p.y + k d is shared by every row (ld_y = 0): one load per k serves the R rows
        for (int k = 0; k < p.K; ++k) {
            const TY *yk = static_cast<const TY *>(p.y) + static_cast<int64_t>(k) * p.d;
            float yv[T][4];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int c = l + L * t;
                if (c < n_chunks) ldv<TY, 4>(yk + 4 * c, yv[t]);
                else yv[t][0] = yv[t][1] = yv[t][2] = yv[t][3] = 0.f;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t i = first + static_cast<int64_t>(r) * G;
                float acc = 0.f;
#pragma unroll
                for (int t = 0; t < T; ++t)
                    acc += xv[r][t][0] * yv[t][0] + xv[r][t][1] * yv[t][1] + xv[r][t][2] * yv[t][2] + xv[r][t][3] * yv[t][3];
                for (int off = L >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
                if (live[r] && l == 0) p.out[i * p.K + k] = p.scale * acc - (p.corr ? p.corr[i * p.K + k] : 0.f);
            }
        }
    }
}

// a[i] -= b[i]
__global__ void __launch_bounds__(256) attn_sub_kernel(float *a, const float *b, int64_t n)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < n) a[i] -= b[i];
}

// ---- the destination side of the backward -------------------------------------------------------------------
// Per destination type, one pass over its rows: the activation's backward (grad = act'(h) g, written when there is
// an activation) and, for each relation into the type, dot = <grad, o>, der = (1 - slope) (<grad, o_pos> - apos dot)
// per head, and the terms that the source side gathers, side by side in one line per destination: er, smax, sinv, dot.
// With sum_e alpha_e = 1 and gate_e = alpha_e (slope + (1 - slope) [logit_e > 0]) this der is
// sum_e gate_e (<grad, z_e> - dot); no edge is visited.  Streaming, bound by its bytes: grad rows are read once for
// all relations.  (As four launches per relation and one for the activation, with a sweep over the edges for the
// sums of gates: 4.1 ms for 7 relations into 1.87 M rows of 256, now 2.9 ms = 5.1 TB/s.)  Rows of up to 1,024 columns
// stay in registers for all relations (200,000 rows, 3 relations: 256 columns 363 us, 512 in 8 heads 748, 1,024 in 4
// heads 1,454 = 5.1 to 5.3 TB/s; served row by row with 4-byte loads, 512 columns took 1,597 us and 1,024 took 2,193).
// Past that, and where a long row's heads are no power of two of chunks, row by row and head by head: 600 columns in 6
// heads 1,375 us, with 4-byte loads 1,802.
constexpr int kDstRels = 8;
struct DstItem {
    const float *o, *opos, *er, *smax, *sinv, *apos;
    float *der, *pack;
    int64_t ld_o;
};
struct DstParams {
    const float *g, *h; // h: null without an activation
    float *ga;
    int64_t ld_g, ld_h, ld_ga, n;
    int64_t first; // its first workgroup
    int d, K, F, n_rels;
    float slope;
    DstItem it[kDstRels];
};
// Several destination types in one launch, their workgroups end to end: by itself a type of a few thousand rows takes the
// 4 to 5 us that any launch takes.
constexpr int kDstTypes = 4;
struct DstTypes { // passed by value
    DstParams t[kDstTypes];
    int64_t first; // first workgroup of this launch
    int n;
};
// the type that this workgroup serves, and the workgroup's number within it
__device__ __forceinline__ const DstParams &dst_type_of(const DstTypes &m, int64_t &wg)
{
    wg = m.first + blockIdx.x;
    int c = 0;
    while (c + 1 < m.n && wg >= m.t[c + 1].first) ++c; // uniform
    wg -= m.t[c].first;
    return m.t[c];
}

__device__ __forceinline__ void dst_store(const DstParams &p, const DstItem &t, int64_t i, int k, float dot, float dpos)
{
    const int64_t at = i * p.K + k;
    t.der[at] = (1.f - p.slope) * (dpos - t.apos[at] * dot);
    reinterpret_cast<float4 *>(t.pack)[at] = make_float4(t.er[at], t.smax[at], t.sinv[at], dot);
}

// Rows of 16-byte chunks, T chunks per lane, L lanes per row (L a power of two; 64 if T > 1), R rows per lane group; heads
// of whole chunks, for T > 1 a power of two of them.
template <int R, int T>
__global__ void __launch_bounds__(256) attn_dst_kernel(DstTypes m, int L)
{
    int64_t wg;
    const DstParams &p = dst_type_of(m, wg);
    const int lane = threadIdx.x & 63;
    const int G = 64 / L, grp = lane / L, l = lane % L;
    const int64_t first = (wg * 4 + (threadIdx.x >> 6)) * R * G + grp;
    const int n_chunks = p.d / 4, cph = p.F / 4;
    const bool pow2 = (cph & (cph - 1)) == 0;
    float4 gv[R][T];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int64_t i = first + static_cast<int64_t>(r) * G;
            const int c = l + L * t;
            float4 &v = gv[r][t];
            v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i < p.n && c < n_chunks) {
                v = *reinterpret_cast<const float4 *>(p.g + i * p.ld_g + 4 * c);
                if (p.h) {
                    const float4 x = *reinterpret_cast<const float4 *>(p.h + i * p.ld_h + 4 * c);
                    v.x = x.x > 0.f ? v.x : 0.f; v.y = x.y > 0.f ? v.y : 0.f;
                    v.z = x.z > 0.f ? v.z : 0.f; v.w = x.w > 0.f ? v.w : 0.f;
                }
            }
        }
    for (int q = 0; q < p.n_rels; ++q) {
        const DstItem &t = p.it[q];
        float a[R][T], b[R][T];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int s = 0; s < T; ++s) {
                const int64_t i = first + static_cast<int64_t>(r) * G;
                const int c = l + L * s;
                const float4 v = gv[r][s];
                a[r][s] = b[r][s] = 0.f;
                if (i < p.n && c < n_chunks) {
                    const float4 o = *reinterpret_cast<const float4 *>(t.o + i * t.ld_o + 4 * c);
                    const float4 u = *reinterpret_cast<const float4 *>(t.opos + i * t.ld_o + 4 * c);
                    a[r][s] = v.x * o.x + v.y * o.y + v.z * o.z + v.w * o.w;
                    b[r][s] = v.x * u.x + v.y * u.y + v.z * u.z + v.w * u.w;
                }
            }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int64_t i = first + static_cast<int64_t>(r) * G;
            if (T > 1 && cph > 64) { // a head is whole steps of 64 chunks (uniform)
                float sa = 0.f, sb = 0.f;
#pragma unroll
                for (int s = 0; s < T; ++s) {
                    sa += a[r][s];
                    sb += b[r][s];
                    if ((64 * (s + 1)) % cph == 0) {
                        group_sum<64, 1>(&sa);
                        group_sum<64, 1>(&sb);
                        const int k = (64 * (s + 1)) / cph - 1;
                        if (i < p.n && l == 0 && k < p.K) dst_store(p, t, i, k, sa, sb);
                        sa = sb = 0.f;
                    }
                }
                continue;
            }
#pragma unroll
            for (int s = 0; s < T; ++s) {
                const int c = l + L * s;
                if (T > 1 || pow2) { // uniform
                    for (int off = cph >> 1; off > 0; off >>= 1) {
                        a[r][s] += __shfl_xor(a[r][s], off, 64);
                        b[r][s] += __shfl_xor(b[r][s], off, 64);
                    }
                } else { // a head's chunks lie in consecutive lanes: its first lane adds the others' in order
                    const float a0 = a[r][s], b0 = b[r][s];
                    for (int j = 1; j < cph; ++j) {
                        a[r][s] += __shfl(a0, (lane + j) & 63, 64);
                        b[r][s] += __shfl(b0, (lane + j) & 63, 64);
                    }
                }
                if (i < p.n && c < n_chunks && c % cph == 0) dst_store(p, t, i, c / cph, a[r][s], b[r][s]);
            }
        }
    }
    if (p.ga) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int64_t i = first + static_cast<int64_t>(r) * G;
                const int c = l + L * t;
                if (i < p.n && c < n_chunks) *reinterpret_cast<float4 *>(p.ga + i * p.ld_ga + 4 * c) = gv[r][t];
            }
    }
}

// any other shape: one wavefront per row, head by head; EPC = 4: 16-byte loads, heads of whole chunks
template <int EPC>
__global__ void __launch_bounds__(256) attn_dst_any_kernel(DstTypes m)
{
    int64_t wg;
    const DstParams &p = dst_type_of(m, wg);
    const int lane = threadIdx.x & 63;
    const int64_t i = wg * 4 + (threadIdx.x >> 6);
    if (i >= p.n) return; // uniform per wavefront
    const float *g = p.g + i * p.ld_g, *h = p.h ? p.h + i * p.ld_h : nullptr;
    const auto grad = [&](int j, float (&v)[EPC]) { // the gradient behind the activation, columns j ..
        ldv<float, EPC>(g + j, v);
        if (h) {
            float x[EPC];
            ldv<float, EPC>(h + j, x);
#pragma unroll
            for (int e = 0; e < EPC; ++e) v[e] = x[e] > 0.f ? v[e] : 0.f;
        }
    };
    for (int q = 0; q < p.n_rels; ++q) {
        const DstItem &t = p.it[q];
        for (int k = 0; k < p.K; ++k) {
            float a = 0.f, b = 0.f;
            for (int j = k * p.F + lane * EPC; j < (k + 1) * p.F; j += 64 * EPC) {
                float v[EPC], o[EPC], u[EPC];
                grad(j, v);
                ldv<float, EPC>(t.o + i * t.ld_o + j, o);
                ldv<float, EPC>(t.opos + i * t.ld_o + j, u);
#pragma unroll
                for (int e = 0; e < EPC; ++e) {
                    a = fmaf(v[e], o[e], a);
                    b = fmaf(v[e], u[e], b);
                }
            }
            group_sum<64, 1>(&a);
            group_sum<64, 1>(&b);
            if (lane == 0) dst_store(p, t, i, k, a, b);
        }
    }
    if (p.ga)
        for (int j = lane * EPC; j < p.d; j += 64 * EPC) {
            float v[EPC];
            grad(j, v);
#pragma unroll
            for (int e = 0; e < EPC; ++e) p.ga[i * p.ld_ga + j + e] = v[e];
        }
}

template <typename TX, typename TY>
heta_status launch_rowdot_t(const DotParams &p, hipStream_t st)
{
    if (p.n == 0) return HETA_OK;
    const size_t sx = sizeof(TX), sy = sizeof(TY);
    if (p.y2) { // only the one-pass kernel takes a second operand: anything else runs as two launches
        const int nc = p.d / 4, cph2 = p.F / 4;
        int L2 = 1;
        while (L2 < nc && L2 < 64) L2 <<= 1;
        const int T2 = (nc + L2 - 1) / L2;
        const bool one_pass = p.per_head && p.ld_y && (reinterpret_cast<uintptr_t>(p.x) % (4 * sx) == 0) && (p.ld_x % 4 == 0) &&
                              (reinterpret_cast<uintptr_t>(p.y) % (4 * sy) == 0) && (reinterpret_cast<uintptr_t>(p.y2) % (4 * sy) == 0) &&
                              (p.ld_y % 4 == 0) && (p.d % 4 == 0) && (p.F % 4 == 0) && T2 <= 4 && cph2 > 0 &&
                              (cph2 & (cph2 - 1)) == 0 && (cph2 <= L2 || T2 % (cph2 / L2) == 0);
        if (!one_pass) {
            DotParams a = p, b = p;
            a.y2 = nullptr;
            b.y = p.y2;
            b.y2 = nullptr;
            b.scale = p.scale2;
            b.corr = nullptr;
            b.out = p.out2;
            heta_status e = launch_rowdot_t<TX, TY>(a, st);
            return e != HETA_OK ? e : launch_rowdot_t<TX, TY>(b, st);
        }
    }
    const bool vec = (reinterpret_cast<uintptr_t>(p.x) % (4 * sx) == 0) && (p.ld_x % 4 == 0) &&
                     (reinterpret_cast<uintptr_t>(p.y) % (4 * sy) == 0) && (p.ld_y % 4 == 0) && (p.d % 4 == 0) &&
                     (p.F % 4 == 0);
    const double bytes = static_cast<double>(p.n) * (p.d * (sx + (p.ld_y ? sy : 0) + (p.y2 ? sy : 0)) + 4.0 * p.K * ((p.corr ? 2 : 1) + (p.y2 ? 1 : 0)));
    ProfScope prof("attn_rowdot_kernel", st, bytes, 0);
    const int n_chunks = p.d / 4, cph = p.F / 4;
    int L = 1;
    while (L < n_chunks && L < 64) L <<= 1;
    const int T = (n_chunks + L - 1) / L;
    const bool fast = vec && T <= 4 && (!p.per_head || ((cph & (cph - 1)) == 0 && (cph <= L || T % (cph / L) == 0)));
    const int R = !fast || T > 2 ? 1 : (T == 1 ? 4 : 2); // row groups per wavefront, all loads in flight together
    const int64_t rows_per_block = fast ? static_cast<int64_t>(4) * R * (64 / L) : 4;
    launch_pieces((p.n + rows_per_block - 1) / rows_per_block, 256, [&](unsigned first, unsigned count) {
        DotParams q = p;
        q.first = first;
        if (!vec) hipLaunchKernelGGL((attn_rowdot_kernel<TX, TY, 1>), dim3(count), dim3(256), 0, st, q);
        else if (!fast) hipLaunchKernelGGL((attn_rowdot_kernel<TX, TY, 4>), dim3(count), dim3(256), 0, st, q);
        else if (T == 1) hipLaunchKernelGGL((attn_rowdot_fast_kernel<TX, TY, 1, 4>), dim3(count), dim3(256), 0, st, q, L, cph);
        else if (T == 2) hipLaunchKernelGGL((attn_rowdot_fast_kernel<TX, TY, 2, 2>), dim3(count), dim3(256), 0, st, q, L, cph);
        else if (T == 3) hipLaunchKernelGGL((attn_rowdot_fast_kernel<TX, TY, 3, 1>), dim3(count), dim3(256), 0, st, q, L, cph);
        else hipLaunchKernelGGL((attn_rowdot_fast_kernel<TX, TY, 4, 1>), dim3(count), dim3(256), 0, st, q, L, cph);
    });
    HETA_LAUNCH_CHECK("attn_rowdot_kernel");
    return HETA_OK;
}

heta_status launch_rowdot(const DotParams &p, heta_dtype x_dt, heta_dtype y_dt, hipStream_t st)
{
    if (x_dt == HETA_F32) return y_dt == HETA_F32 ? launch_rowdot_t<float, float>(p, st) : launch_rowdot_t<float, bf16_t>(p, st);
    return y_dt == HETA_F32 ? launch_rowdot_t<bf16_t, float>(p, st) : launch_rowdot_t<bf16_t, bf16_t>(p, st);
}

// ---- backward of the scores -------------------------------------------------------------------------
// dx[i, j] = beta dx[i, j] + sum_k ds[i, k] y_k[j]   (per_head: only k = j / F, y_k[j] = vec[j])
__global__ void __launch_bounds__(256) attn_score_bwd_input_kernel(const float *ds, const float *vec, int64_t n, int d,
                                                                   int K, int F, int per_head, float *dx, int64_t ld_dx,
                                                                   float beta)
{
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t i = t / d;
    const int j = static_cast<int>(t % d);
    if (i >= n) return;
    float v = 0.f;
    if (per_head) {
        v = ds[i * K + j / F] * vec[j];
    } else {
        for (int k = 0; k < K; ++k) v = fmaf(ds[i * K + k], vec[static_cast<int64_t>(k) * d + j], v);
    }
    float *o = dx + i * ld_dx + j;
    *o = beta != 0.f ? *o + v : v;
}

// the same, four columns per thread (rows 16-byte aligned, heads a multiple of four columns wide)
__global__ void __launch_bounds__(256) attn_score_bwd_input_vec_kernel(const float *ds, const float *vec, int64_t n, int d,
                                                                       int K, int F, int per_head, float *dx,
                                                                       int64_t ld_dx, float beta)
{
    const int d4 = d / 4;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t i = t / d4;
    const int j = static_cast<int>(t - i * d4) * 4;
    if (i >= n) return;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (per_head) {
        const float s = ds[i * K + j / F];
        const float4 w = *reinterpret_cast<const float4 *>(vec + j);
        v = make_float4(s * w.x, s * w.y, s * w.z, s * w.w);
    } else {
        for (int k = 0; k < K; ++k) {
            const float s = ds[i * K + k];
            const float4 w = *reinterpret_cast<const float4 *>(vec + static_cast<int64_t>(k) * d + j);
            v.x = fmaf(s, w.x, v.x); v.y = fmaf(s, w.y, v.y); v.z = fmaf(s, w.z, v.z); v.w = fmaf(s, w.w, v.w);
        }
    }
    float4 *o = reinterpret_cast<float4 *>(dx + i * ld_dx + j);
    if (beta != 0.f) {
        const float4 old = *o;
        v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
    }
    *o = v;
}

// dvec_k[j] = sum_i ds[i, k] x[i, j]: stage 1, one workgroup per (slab of rows, 256 columns), partial sums
// to part[slab][k][j] (per_head: part[slab][j], only k = j / F); stage 2 adds the slabs in order.
constexpr int kSlabRows = 512;
template <typename T>
__global__ void __launch_bounds__(256) attn_score_bwd_param_kernel(const T *x, int64_t ld_x, const float *ds, int64_t n,
                                                                   int d, int K, int F, int per_head, float *part)
{
    const int j = blockIdx.y * 256 + threadIdx.x;
    const int64_t slab = blockIdx.x;
    const int64_t i0 = slab * kSlabRows, i1 = min(n, i0 + kSlabRows);
    if (j >= d) return;
    const int nk = per_head ? 1 : K;
    float acc[kMaxHeads];
#pragma unroll
    for (int k = 0; k < kMaxHeads; ++k) acc[k] = 0.f;
    const int kh = per_head ? j / F : 0;
    for (int64_t i = i0; i < i1; ++i) {
        const float xv = ld1(x + i * ld_x + j);
        if (per_head) {
            acc[0] = fmaf(ds[i * K + kh], xv, acc[0]);
        } else {
#pragma unroll
            for (int k = 0; k < kMaxHeads; ++k)
                if (k < K) acc[k] = fmaf(ds[i * K + k], xv, acc[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < kMaxHeads; ++k)
        if (k < nk) part[(slab * nk + k) * d + j] = acc[k];
}

// the same, four columns per lane and four row groups per workgroup (rows 16 / 8-byte aligned, heads a
// multiple of four columns wide); the row groups are added in order through LDS
// KH = 0: per head (one accumulator per column); KH > 0: every head uses the whole row, K <= KH accumulators per column
template <typename T, int KH>
__global__ void __launch_bounds__(256) attn_score_bwd_param_vec_kernel(const T *x, int64_t ld_x, const float *ds, int64_t n,
                                                                       int d, int K, int F, float *part)
{
    constexpr int NA = KH == 0 ? 1 : KH;
    __shared__ float4 red[4][64];
    const int lane = threadIdx.x & 63, rg = threadIdx.x >> 6;
    const int j = (blockIdx.y * 64 + lane) * 4;
    const int64_t slab = blockIdx.x;
    const int64_t i0 = slab * kSlabRows, i1 = min(n, i0 + kSlabRows);
    const bool live = j < d;
    const int nk = KH == 0 ? 1 : K;
    const int kh = KH == 0 && live ? j / F : 0;
    float acc[NA][4];
#pragma unroll
    for (int k = 0; k < NA; ++k) acc[k][0] = acc[k][1] = acc[k][2] = acc[k][3] = 0.f;
    if (live) {
        constexpr int U = KH > 4 ? 4 : 8; // rows in flight per row group
        for (int64_t ib = i0 + rg; ib < i1; ib += 4 * U) {
            float xv[U][4], sv[U][NA];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = ib + 4 * u;
                if (i < i1) {
                    ldv<T, 4>(x + i * ld_x + j, xv[u]);
                    if (KH == 0) {
                        sv[u][0] = ds[i * K + kh];
                    } else {
#pragma unroll
                        for (int k = 0; k < NA; ++k) sv[u][k] = k < K ? ds[i * K + k] : 0.f;
                    }
                } else {
                    xv[u][0] = xv[u][1] = xv[u][2] = xv[u][3] = 0.f;
#pragma unroll
                    for (int k = 0; k < NA; ++k) sv[u][k] = 0.f;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int k = 0; k < NA; ++k)
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[k][c] = fmaf(sv[u][k], xv[u][c], acc[k][c]);
        }
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        if (k < nk) { // uniform
            red[rg][lane] = make_float4(acc[k][0], acc[k][1], acc[k][2], acc[k][3]);
            __syncthreads();
            if (rg == 0 && live) {
                float4 a = red[0][lane];
#pragma unroll
                for (int r = 1; r < 4; ++r) {
                    const float4 b = red[r][lane];
                    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
                }
                *reinterpret_cast<float4 *>(part + (slab * nk + k) * d + j) = a;
            }
            __syncthreads();
        }
    }
}

// stage 2: out[t] = sum over slabs of part[slab][t].  One workgroup of 16 wavefronts per 64 elements:
// wavefront w adds slabs w, w + 16, ... (coalesced 256-byte reads), the sixteen partial sums are added in
// wavefront order through LDS.
__global__ void __launch_bounds__(1024) attn_slab_sum_kernel(const float *part, int64_t n_slabs, int64_t elems, float *out)
{
    __shared__ float red[16][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 64 + lane;
    float a = 0.f;
    if (t < elems) {
#pragma unroll 4
        for (int64_t s = w; s < n_slabs; s += 16) a += part[s * elems + t];
    }
    red[w][lane] = a;
    __syncthreads();
    if (w == 0 && t < elems) {
        float r = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) r += red[i][lane];
        out[t] = r;
    }
}


// ---- scores of several vector sets of one table ---------------------------------------------------------
// A node type is the source of some relations and the destination of others, and every one of them takes
// a row score <x_i, vec_k> of the same table with vectors of its own (el with W_r a_r, er with q_r).  One
// launch serves them all, reading the table once per 32 vectors: scores, dx[i, :] = sum_v dscore_v[i] vec_v and
// dvec_v = sum_i dscore_v[i] x[i, :] are thin contractions (at most 128 columns, 32 vectors
// at a time) and run on the fp32 matrix instruction, whose
// products and sums are the fp32 FMAs of the vector ALU: what bounds them is the pass over the table.  Measured
// over the four tables of an academic graph (1.87 M fp32 rows of 128, 16 and 24 vectors), against lane shuffles and
// per-lane FMAs: scores 547 -> 271 us, input gradient 472 -> 224 us; 187,000 bf16 rows with up to 56 vectors (set by set
// before, above 32): 274 -> 63 and 209 -> 81 us.
constexpr int kMultiSets = 8, kMultiCols = 128;
constexpr int kScoreTiles = 4; // tiles of 16 vectors that a workgroup of the forward keeps in LDS
constexpr int kMultiVecs = 120; // the input gradient keeps all vectors in LDS: 120 * (512 + 8) bytes stay below 64 KB
struct ScoreMulti {
    const float *vec[kMultiSets]; // [K][d] each
    float *score[kMultiSets];     // [n][K] each: written by the forward, read (dscore) by the backward
    float *dvec[kMultiSets];      // [K][d] each, or null
    int n_sets, K, NV;            // NV = n_sets * K
};

// Several tables in one launch, their workgroups end to end (by itself a table of a few thousand rows takes the 4 to 5 us
// that any launch takes, its input gradient 10: the vectors are brought into LDS first).  With the weights' folds, the
// destination side and the sums over relations laid end to end as well, 69 launches of an attention layer of 64 columns, 4
// node types and 7 relations (2.1 M edges) become 26: forward and backward 1,206 -> 988 us; 21 M edges of 256 columns, where
// the small launches are 1 % of the time, 21,355 -> 21,190.
constexpr int kMultiTables = 8;
struct ScoreTable {
    const void *x;
    float *dx, *part;
    int64_t ld_x, ld_dx, n, slab_rows, n_slabs;
    int d, nb, nvc; // nb: workgroups along the rows; nvc: tiles of vectors per workgroup (forward), vectors in whole tiles (backward)
    float beta;
    unsigned first; // its first workgroup
    ScoreMulti m;
};
struct ScoreTables { // passed by value
    ScoreTable t[kMultiTables];
    int n;
};
// the table that this workgroup serves, and the workgroup's number within it
__device__ __forceinline__ const ScoreTable &score_table_of(const ScoreTables &q, unsigned &wg)
{
    int c = 0;
    while (c + 1 < q.n && blockIdx.x >= q.t[c + 1].first) ++c; // uniform
    wg = blockIdx.x - q.t[c].first;
    return q.t[c];
}

using f32x16 = __attribute__((ext_vector_type(16))) float;
using f32x4 = __attribute__((ext_vector_type(4))) float;
// pointers kept in LDS: the address space says that they point to global memory
using gf32 = __attribute__((address_space(1))) float;
using gf32x4 = __attribute__((address_space(1))) f32x4;

// element (v / K) of a table of kMultiSets pointers for a lane-dependent v (a select chain: indexing the kernel
// arguments by a vector register would move them to scratch memory)
template <typename P> __device__ __forceinline__ P pick(P const (&tab)[kMultiSets], int j)
{
    P p = tab[0];
#pragma unroll
    for (int q = 1; q < kMultiSets; ++q) p = j == q ? tab[q] : p;
    return p;
}

template <typename T> __device__ __forceinline__ void load4(const T *p, float f[4]);
template <> __device__ __forceinline__ void load4<float>(const float *p, float f[4])
{
    const float4 v = *reinterpret_cast<const float4 *>(p);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
}

// the same in two steps: the load, and its four columns
template <typename T> struct Raw4;
template <> struct Raw4<float> {
    float4 v;
    __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
    __device__ __forceinline__ void get(float f[4]) const { f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w; }
};
template <> struct Raw4<bf16_t> {
    uint2 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint2 *>(p); }
    __device__ __forceinline__ void get(float f[4]) const
    {
        f[0] = __uint_as_float(v.x << 16); f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16); f[3] = __uint_as_float(v.y & 0xffff0000u);
    }
};

// Scores of up to 16 kScoreTiles vectors and 16 rows per tile: the vectors are the first operand, so a
// lane ends with one row's scores of four consecutive vectors - one 16-byte store where a set has a multiple of
// four heads (VEC).  A lane holds the columns 16 c + 4 h .. + 3 of its vector and of its row (h: its quarter of the
// wavefront): which k a step multiplies is free as long as both operands agree.  Sums of eight products
// (two instructions) are added pairwise, which keeps the rounding error of a 128-term score where a
// tree over the columns has it; one running accumulator shows in the layer's output.  NC = chunks of 16 columns.
template <int NC> __device__ __forceinline__ f32x4 score_sum(const float (&a)[NC][4], const float (&x)[NC][4])
{
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 level[4]; // level[i]: the sum of the last 2^i chunks that is not part of a larger one yet
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        f32x4 p = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][0], x[c][0], zero, 0, 0, 0);
        f32x4 q = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][2], x[c][2], zero, 0, 0, 0);
        p = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][1], x[c][1], p, 0, 0, 0);
        q = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][3], x[c][3], q, 0, 0, 0);
        f32x4 s = p + q;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (((c + 1) >> i & 1) != 0) {
                level[i] = s;
                break;
            }
            s = level[i] + s;
        }
    }
    return level[NC == 8 ? 3 : NC == 4 ? 2 : 1]; // NC is 2, 4 or 8
}

// Half of the time of a table of 100,000 rows was the start of each wavefront (its vectors into registers, for two tiles of rows)
// and the wait for each tile's rows.  So the vectors lie in LDS as the lanes hold them, brought there once per workgroup, up to
// 64 for one pass over the rows, and the rows of the next tile are on their way while this one's are multiplied.  Four bf16
// tables of 187,000 rows together with 32 vectors in registers, two workgroups per CU: 50 + 7 us in two launches, now 32 in one;
// fp32 tables of 1.87 M rows, whose wavefronts had many tiles: 167 + 110 us, now 271.  Four workgroups per CU spill at 128 columns
// (45 and 501 us).
template <typename T, int NC, bool VEC>
__global__ void __launch_bounds__(256, NC == 8 ? 3 : 4) attn_score_multi_kernel(ScoreTables q)
{
    extern __shared__ __align__(16) float4 svec[]; // [tile][NC][lane], then the pointers
    unsigned wg;
    const ScoreTable &tab = score_table_of(q, wg);
    const ScoreMulti &m = tab.m;
    const T *x = static_cast<const T *>(tab.x);
    const int64_t ld_x = tab.ld_x, n = tab.n;
    const int d = tab.d, nb = tab.nb;
    const int lane = threadIdx.x & 63, l = lane & 15, h = lane >> 4;
    const int t0 = static_cast<int>(wg / nb) * tab.nvc, nt = min(tab.nvc, (m.NV + 15) / 16 - t0), v0 = 16 * t0;
    wg %= nb;
    const int64_t step = static_cast<int64_t>(nb) * 4 * 16;
    int64_t r0 = (static_cast<int64_t>(wg) * 4 + (threadIdx.x >> 6)) * 16;
    Raw4<T> next[NC];
    const auto load = [&](int64_t row0) { // rows past the end repeat the last one and are not stored, columns past it count as zero
        const T *xr = x + min(row0 + l, n - 1) * ld_x;
#pragma unroll
        for (int c = 0; c < NC; ++c) next[c].load(xr + (16 * c + 4 * h < d ? 16 * c + 4 * h : 0));
    };
    load(r0);
    gf32 **sptr = reinterpret_cast<gf32 **>(svec + nt * NC * 64);
    for (int i0 = threadIdx.x; i0 < nt * NC * 64; i0 += 1024) { // four loads in flight
        float4 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 256 * u, v = min(v0 + i / (NC * 64) * 16 + l, m.NV - 1), set = v / m.K, col = i / 64 % NC * 16 + 4 * h;
            t[u] = *reinterpret_cast<const float4 *>(pick(m.vec, set) + static_cast<int64_t>(v - set * m.K) * d + (col < d ? col : 0));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + 256 * u;
            if (i >= nt * NC * 64) continue;
            const bool given = v0 + i / (NC * 64) * 16 + l < m.NV && i / 64 % NC * 16 + 4 * h < d;
            svec[i] = given ? t[u] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
    if (static_cast<int>(threadIdx.x) < 16 * nt) {
        const int v = v0 + threadIdx.x;
        sptr[threadIdx.x] = v < m.NV ? (gf32 *)(pick(m.score, v / m.K) + v % m.K) : nullptr;
    }
    __syncthreads();
    for (; r0 < n; r0 += step) { // uniform per wavefront
        const int64_t r = r0 + l;
        float xv[NC][4];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            next[c].get(xv[c]);
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[c][j] = 16 * c + 4 * h < d ? xv[c][j] : 0.f;
        }
        if (r0 + step < n) load(r0 + step);
        for (int t = 0; t < nt; ++t) {
            float a[NC][4];
#pragma unroll
            for (int c = 0; c < NC; ++c) load4<float>(reinterpret_cast<const float *>(svec + (t * NC + c) * 64 + lane), a[c]);
            const f32x4 s = score_sum<NC>(a, xv);
            if (r < n) {
                if (VEC) {
                    gf32 *o = sptr[16 * t + 4 * h];
                    if (o) *(gf32x4 *)(o + r * m.K) = s;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        gf32 *o = sptr[16 * t + 4 * h + j];
                        if (o) o[r * m.K] = s[j];
                    }
                }
            }
        }
    }
}

// dx[i, :] (+)= sum_v dscore_v[i] vec_v: 32 rows per tile are the first operand, the four columns 4 l .. 4 l + 3 of
// lane l the second one of four products, so that a row leaves as 16-byte stores of whole cache lines.  The vectors
// sit in LDS, zero beyond d and up to a multiple of eight vectors; step (c, j) multiplies vector 8 c + 4 h + j.
// (Brought there element by element, each lane working out its vector, that was half of the time where a table of 100,000
// rows has 56 vectors: four tables of 187,000 rows together 59 us, now 44.)
template <bool VEC>
__global__ void __launch_bounds__(256, 3) attn_score_bwd_multi_input_kernel(ScoreTables q)
{
    extern __shared__ __align__(16) float vecs[]; // [8 nc][128], then the pointers
    unsigned wg;
    const ScoreTable &tab = score_table_of(q, wg);
    const ScoreMulti &m = tab.m;
    const int64_t n = tab.n, ld_dx = tab.ld_dx;
    const int d = tab.d;
    float *const dx = tab.dx;
    const float beta = tab.beta;
    const int lane = threadIdx.x & 63, l = lane & 31, h = lane >> 5;
    const int nc = (m.NV + 7) / 8;
    const gf32 **sptr = reinterpret_cast<const gf32 **>(vecs + 8 * nc * kMultiCols);
    // one vector per wavefront and load, two columns per lane (d is a multiple of four): which set it belongs to is uniform
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int v0 = w; v0 < 8 * nc; v0 += 16) {
        float2 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = min(v0 + 4 * u, m.NV - 1), set = v / m.K;
            t[u] = *reinterpret_cast<const float2 *>(m.vec[set] + static_cast<int64_t>(v - set * m.K) * d + (2 * lane < d ? 2 * lane : 0));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + 4 * u;
            if (v >= 8 * nc) continue;
            const bool given = v < m.NV && 2 * lane < d;
            *reinterpret_cast<float2 *>(vecs + v * kMultiCols + 2 * lane) = given ? t[u] : make_float2(0.f, 0.f);
        }
    }
    for (int v = threadIdx.x; v < 8 * nc; v += 256) sptr[v] = v < m.NV ? (const gf32 *)(pick(m.score, v / m.K) + v % m.K) : nullptr;
    __syncthreads();
    const int64_t wave = static_cast<int64_t>(wg) * 4 + (threadIdx.x >> 6), n_waves = static_cast<int64_t>(tab.nb) * 4;
    for (int64_t r0 = wave * 32; r0 < n; r0 += n_waves * 32) { // uniform per wavefront
        const int64_t r = min(r0 + l, n - 1);
        f32x16 acc[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
        for (int c0 = 0; c0 < nc; c0 += 4) { // 32 vectors: all their loads before the first product
            float ds[4][4];
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                ds[cc][0] = ds[cc][1] = ds[cc][2] = ds[cc][3] = 0.f;
                if (c0 + cc < nc) {
                    const int v = 8 * (c0 + cc) + 4 * h;
                    if (VEC) {
                        const gf32 *p = sptr[v];
                        if (p) {
                            const f32x4 t = *(const gf32x4 *)(p + r * m.K);
                            ds[cc][0] = t.x; ds[cc][1] = t.y; ds[cc][2] = t.z; ds[cc][3] = t.w;
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const gf32 *p = sptr[v + j];
                            if (p) ds[cc][j] = p[r * m.K];
                        }
                    }
                }
            }
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                if (c0 + cc < nc) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float4 b = *reinterpret_cast<const float4 *>(vecs + (8 * (c0 + cc) + 4 * h + j) * kMultiCols + 4 * l);
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(ds[cc][j], b.x, acc[0], 0, 0, 0);
                        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(ds[cc][j], b.y, acc[1], 0, 0, 0);
                        acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(ds[cc][j], b.z, acc[2], 0, 0, 0);
                        acc[3] = __builtin_amdgcn_mfma_f32_32x32x2f32(ds[cc][j], b.w, acc[3], 0, 0, 0);
                    }
                }
            }
        }
        if (4 * l < d) {
#pragma unroll
            for (int i0 = 0; i0 < 16; i0 += 8) { // eight rows' loads before their stores
                float4 old[8];
                if (beta != 0.f) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int64_t row = r0 + 8 * ((i0 + i) / 4) + 4 * h + i % 4;
                        old[i] = *reinterpret_cast<const float4 *>(dx + min(row, n - 1) * ld_dx + 4 * l);
                    }
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int64_t row = r0 + 8 * ((i0 + i) / 4) + 4 * h + i % 4;
                    float4 w4 = make_float4(acc[0][i0 + i], acc[1][i0 + i], acc[2][i0 + i], acc[3][i0 + i]);
                    if (beta != 0.f) {
                        w4.x += old[i].x; w4.y += old[i].y; w4.z += old[i].z; w4.w += old[i].w;
                    }
                    if (row < n) *reinterpret_cast<float4 *>(dx + row * ld_dx + 4 * l) = w4;
                }
            }
        }
    }
}

// part[slab][v][128]: the slab's sum over its rows of dscore_v[i] x[i, :].  The contraction runs over the rows, four per
// step (one per quarter h of the wavefront); a lane's first operand is its vector's dscore, its second the four columns
// 64 c + 4 l .. + 3 of chunk c, one product each.  A wavefront takes every fourth group of 4 U rows of the slab, the four
// wavefronts' sums are added in wavefront order through LDS.  16 NT vectors per workgroup (its second index picks them), NC
// chunks of 64 columns: no product is spent on more.  With 32 vectors and 128 columns whatever is given, two rows per
// step and the loads behind branches, a pass was bound by the products and by one load after the other: 700,000 rows
// of 128 columns, bf16 with 1 / 24 vectors 146 / 155 -> 45 / 70 us, fp32 116 / 124 -> 74 / 88; of 64, fp32, 4 vectors 89 -> 38.
template <typename T, int NC, int NT>
__global__ void __launch_bounds__(256, NC * NT * sizeof(T) == 16 ? 3 : 4) attn_score_bwd_multi_param_kernel(ScoreTables q)
{
    constexpr int U = 4, VT = 16 * NT;
    unsigned wg;
    const ScoreTable &tab = score_table_of(q, wg);
    const ScoreMulti &m = tab.m;
    const T *x = static_cast<const T *>(tab.x);
    const int64_t ld_x = tab.ld_x, n = tab.n, slab_rows = tab.slab_rows;
    const int d = tab.d, nb = tab.nb, tile = static_cast<int>(wg / nb), tiles = tab.nvc / VT;
    __shared__ __align__(16) float buf[VT][kMultiCols];
    const int lane = threadIdx.x & 63, l = lane & 15, h = lane >> 4, w = threadIdx.x >> 6;
    const int64_t slab = wg % nb;
    const int64_t i0 = slab * slab_rows, i1 = min(n, i0 + slab_rows);
    // lanes past the vectors and the columns given repeat others; what they sum up is not written out
    const float *ds[NT];
    int col[NC];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int v = min(tile * VT + 16 * t + l, m.NV - 1);
        ds[t] = pick(m.score, v / m.K) + v % m.K;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) col[c] = 64 * c + 4 * l < d ? 64 * c + 4 * l : 0;
    f32x4 acc[NT][NC][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[t][c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t rb = i0 + w * (4 * U); rb < i1; rb += 16 * U) { // uniform per wavefront
        // no load behind a branch, a conversion or a product: all of them are in flight together
        Raw4<T> raw[U][NC];
        float sv[U][NT];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t r = min(rb + 4 * u + h, i1 - 1);
#pragma unroll
            for (int c = 0; c < NC; ++c) raw[u][c].load(x + r * ld_x + col[c]);
#pragma unroll
            for (int t = 0; t < NT; ++t) sv[u][t] = ds[t][r * m.K];
        }
        __builtin_amdgcn_sched_barrier(0); // else each load is moved down to its products
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool past = rb + 4 * u + h >= i1; // a copy of the slab's last row
#pragma unroll
            for (int t = 0; t < NT; ++t) sv[u][t] = past ? 0.f : sv[u][t];
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                float xv[4];
                raw[u][c].get(xv);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xv[j] = past ? 0.f : xv[j];
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t][c][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(sv[u][t], xv[j], acc[t][c][j], 0, 0, 0);
                }
            }
        }
    }
    for (int turn = 0; turn < 4; ++turn) { // wavefront `turn` adds its sums to the buffer, in order
        if (w == turn) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        float4 *b = reinterpret_cast<float4 *>(&buf[16 * t + 4 * h + i][64 * c + 4 * l]);
                        float4 s = make_float4(acc[t][c][0][i], acc[t][c][1][i], acc[t][c][2][i], acc[t][c][3][i]);
                        if (turn > 0) {
                            const float4 o = *b;
                            s.x += o.x; s.y += o.y; s.z += o.z; s.w += o.w;
                        }
                        *b = s;
                    }
        }
        __syncthreads();
    }
    float *o = tab.part + (slab * tiles + tile) * (VT * kMultiCols);
    for (int t = threadIdx.x * 4; t < VT * kMultiCols; t += 1024)
        if (t % kMultiCols < 64 * NC) *reinterpret_cast<float4 *>(o + t) = *reinterpret_cast<const float4 *>(&buf[0][0] + t);
}

// dvec_v[c] = sum over the slabs, in slab order per wavefront and wavefront order through LDS (as attn_slab_sum_kernel)
__global__ void __launch_bounds__(1024) attn_multi_slab_sum_kernel(ScoreTables q)
{
    __shared__ float red[16][64];
    unsigned wg;
    const ScoreTable &tab = score_table_of(q, wg);
    const ScoreMulti &m = tab.m;
    const float *part = tab.part;
    const int64_t n_slabs = tab.n_slabs;
    const int d = tab.d;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t elems = static_cast<int64_t>(tab.nvc) * kMultiCols;
    const int64_t t = static_cast<int64_t>(wg) * 64 + lane;
    if ((t - lane) % kMultiCols >= d) return; // uniform: columns that no slab has written
    float a = 0.f;
    if (t < elems) {
#pragma unroll 8
        for (int64_t s = w; s < n_slabs; s += 16) a += part[s * elems + t];
    }
    red[w][lane] = a;
    __syncthreads();
    const int vi = static_cast<int>(t / kMultiCols), c = static_cast<int>(t % kMultiCols);
    float *out = (t < elems && vi < m.NV) ? pick(m.dvec, vi / m.K) : nullptr;
    if (w == 0 && out && c < d) {
        float r = 0.f;
#pragma unroll
        for (int i = 0; i < 16; ++i) r += red[i][lane];
        out[static_cast<int64_t>(vi % m.K) * d + c] = r;
    }
}

// ---- the source score taken off the input table ------------------------------------------------------
// el[u, k] = <z_u[k, :], a[k, :]> with z_u = W^T h_u equals <h_u, wa[k, :]> with wa[k, j] = sum_f W[j, kF + f] a[k, f]:
// the scores then come from the (narrower, never rounded) input table instead of the stored projection.
// One lane per (k, j), so that the sum over f runs in order; the matrix is small, and what counts is the chain of loads of
// one lane, so sixteen are in flight, on workgroups of one wavefront (128 x 256, 4 heads: 9.5 us one by one, now 3.0, eight
// lanes per element 2.8; 768 x 1,024 34.0, 5.7 and 5.0).
// The relations of a layer share a launch, their workgroups end to end: seven of 64 x 64 in seven launches 33 us, in one 5.
constexpr int kFoldItems = 24;
struct FoldItem {
    const void *W;
    const float *a, *dwa;
    float *wa, *dW, *da;
    int64_t ld_w, ld_dw;
    int d_in, d_out;
    unsigned first, w_blocks; // its first workgroup; backward: workgroups of dW, those of da follow
};
struct FoldItems { // passed by value
    FoldItem it[kFoldItems];
    int n, K;
    float beta;
};
__device__ __forceinline__ const FoldItem &fold_item_of(const FoldItems &q, unsigned &wg)
{
    int c = 0;
    while (c + 1 < q.n && blockIdx.x >= q.it[c + 1].first) ++c; // uniform
    wg = blockIdx.x - q.it[c].first;
    return q.it[c];
}

template <typename T>
__global__ void __launch_bounds__(64) attn_fold_kernel(FoldItems q)
{
    unsigned wg;
    const FoldItem &r = fold_item_of(q, wg);
    const int K = q.K, d_in = r.d_in, F = r.d_out / K;
    const int t = static_cast<int>(wg) * 64 + threadIdx.x;
    if (t >= K * d_in) return;
    const int k = t / d_in, j = t - k * d_in;
    const T *w = static_cast<const T *>(r.W) + static_cast<int64_t>(j) * r.ld_w + k * F;
    const float *a = r.a + k * F;
    float acc = 0.f;
    int f = 0;
    for (; f + 16 <= F; f += 16) {
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) x[i] = ld1(w + f + i);
#pragma unroll
        for (int i = 0; i < 16; ++i) acc = fmaf(x[i], a[f + i], acc);
    }
    for (; f < F; ++f) acc = fmaf(ld1(w + f), a[f], acc);
    r.wa[t] = acc;
}

// Its backward, both halves in one launch (two of 4.9 us before, one of 4.9 now at 128 x 256):
//   dW[j, kF + f] = beta dW[j, kF + f] + dwa[k, j] a[k, f], one thread per element, the first w_blocks workgroups;
//   da[k, f] = sum_j dwa[k, j] W[j, kF + f], one wavefront per (k, f), lanes take j round-robin and are combined by a
//   fixed butterfly, so the order of the sum is fixed.
template <typename T>
__global__ void __launch_bounds__(256) attn_fold_bwd_kernel(FoldItems q)
{
    unsigned wg;
    const FoldItem &r = fold_item_of(q, wg);
    const int K = q.K, d_in = r.d_in, d_out = r.d_out, F = d_out / K;
    const float *dwa = r.dwa;
    const T *W = static_cast<const T *>(r.W);
    if (wg < r.w_blocks) {
        const int t = static_cast<int>(wg) * 256 + threadIdx.x;
        if (t >= d_in * d_out) return;
        const int j = t / d_out, c = t - j * d_out;
        const float v = dwa[(c / F) * d_in + j] * r.a[c];
        float *o = r.dW + static_cast<int64_t>(j) * r.ld_dw + c;
        *o = q.beta != 0.f ? *o + v : v;
        return;
    }
    const int lane = threadIdx.x & 63;
    const int c = static_cast<int>(wg - r.w_blocks) * 4 + (threadIdx.x >> 6);
    if (c >= d_out) return; // uniform per wavefront
    const int k = c / F;
    float acc = 0.f;
    for (int j = lane; j < d_in; j += 64) acc = fmaf(dwa[k * d_in + j], ld1(W + static_cast<int64_t>(j) * r.ld_w + c), acc);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) r.da[c] = acc;
}

heta_status ensure_attn(heta_graph *g, size_t bytes)
{
    bytes = std::max<size_t>(bytes, 256); // never hand out a null workspace (relations without edges)
    if (bytes <= g->attn_bytes) return HETA_OK;
    if (g->d_attn) HETA_HIP(hipFree(g->d_attn)); // waits for earlier users
    g->d_attn = nullptr;
    g->attn_bytes = 0;
    HETA_HIP(hipMalloc(&g->d_attn, bytes));
    g->attn_bytes = bytes;
    return HETA_OK;
}

inline size_t round256(size_t b) { return (b + 255) / 256 * 256; }

heta_status check_attn_args(const char *fn, heta_graph *g, int32_t rel, int32_t d, int32_t heads)
{
    if (!g) return fail(HETA_ERR_INVALID_ARG, "%s: null graph", fn);
    if (rel < 0 || rel >= (int32_t)g->rels.size()) return fail(HETA_ERR_INVALID_ARG, "%s: relation %d out of range", fn, rel);
    if (heads <= 0 || heads > kMaxHeads || d <= 0 || d % heads != 0)
        return fail(HETA_ERR_SHAPE, "%s: need 1 <= heads <= %d dividing d (d=%d heads=%d)", fn, kMaxHeads, d, heads);
    return HETA_OK;
}

// Source side of one relation's backward, checked and with its workspace assigned.
struct SourceSide {
    const Relation *r;
    const void *z;
    heta_dtype z_dt;
    int64_t ld_z;
    const float *el, *nbr_pack, *grad_out;
    int64_t ld_go;
    float *dz;
    int64_t ld_dz;
    float *del;
    float *w_alpha, *corr_s, *R, *hub_scratch; // workspace
    int64_t ld_r;
};

// alpha per CSC slot, its sign bit set where the logit is not positive; one pass over the gathered gradient rows gives both
// dz[u] = sum_e alpha_e g[v_e] and R[u] = sum_e gate_e g[v_e], gate_e = alpha_e LeakyReLU'; del = <z, R> - sum_e gate_e dot[v_e].
heta_status attn_source_side(heta_graph *g, const SourceSide *it, int n, int d, int K, float slope, hipStream_t st)
{
    std::vector<Sweep> sw;
    for (int i = 0; i < n; ++i) {
        SweepParams sp{};
        sp.K = K;
        sp.slope = slope;
        sp.row_a = it[i].el;
        sp.nbr_pack = it[i].nbr_pack;
        sp.alpha = it[i].w_alpha;
        sp.corr = it[i].corr_s;
        sw.push_back({&it[i].r->csc, sp, it[i].hub_scratch, 0});
    }
    heta_status e = launch_sweeps<SWEEP_BWD_CSC>(sw, st, "attn_sweep_bwd_src");
    if (e != HETA_OK) return e;
    // del = <z, R> - corr_s is taken inside the aggregation when the shapes allow it (R is then never written)
    std::vector<SlotAggregation> calls;
    for (int i = 0; i < n; ++i)
        calls.push_back({&it[i].r->csc, it[i].grad_out, it[i].ld_go, it[i].w_alpha, it[i].dz, it[i].ld_dz, it[i].R, it[i].ld_r,
                         {it[i].z, it[i].z_dt, it[i].ld_z, it[i].corr_s, it[i].del}, false});
    e = aggregate_slot_weighted_multi(g, calls, HETA_F32, d, K, HETA_F32, 0.f, true, slope, st);
    for (int i = 0; e == HETA_OK && i < n; ++i) {
        if (calls[i].dot_done) continue;
        DotParams dp{};
        dp.x = it[i].z;
        dp.ld_x = it[i].ld_z;
        dp.y = it[i].R;
        dp.ld_y = it[i].ld_r;
        dp.n = it[i].r->n_src;
        dp.d = d;
        dp.K = K;
        dp.F = d / K;
        dp.per_head = 1;
        dp.scale = 1.f;
        dp.corr = it[i].corr_s;
        dp.out = it[i].del;
        e = launch_rowdot(dp, it[i].z_dt, HETA_F32, st);
    }
    return e;
}

// Relations of one call share their launches while their workspace stays below this: larger ones fill the chip by
// themselves (seven relations of 0.06 - 0.4 M edges, 64 columns and 8 heads together: 0.2 GB; one of 4 M edges and 256
// columns alone: 1.2 GB).
constexpr size_t kAttnGroupBytes = size_t(256) << 20;

// an output of one item of a multi call, as a byte range
struct OutRange {
    uintptr_t lo, hi;
    OutRange(const void *p, int64_t rows, int64_t ld, int d, size_t esz)
        : lo(reinterpret_cast<uintptr_t>(p)), hi(p && rows > 0 ? lo + static_cast<uintptr_t>((rows - 1) * ld + d) * esz : lo) {}
    bool overlaps(const OutRange &o) const { return lo < o.hi && o.lo < hi; }
};

// a table with the vector sets of one call
ScoreTable score_table(const void *x, int64_t ld_x, int64_t n, int32_t d, int32_t n_sets, int32_t heads, const float *const *vecs,
                              const float *const *scores)
{
    ScoreTable t{};
    t.x = x;
    t.ld_x = ld_x;
    t.n = n;
    t.d = d;
    t.m.n_sets = n_sets;
    t.m.K = heads;
    t.m.NV = n_sets * heads;
    for (int j = 0; j < n_sets; ++j) {
        t.m.vec[j] = vecs[j];
        t.m.score[j] = const_cast<float *>(scores[j]);
    }
    return t;
}

// launch(tables, k) for the tables of each kind k < n_kinds, up to kMultiTables at a time
template <typename F> heta_status for_tables_of_a_kind(const std::vector<ScoreTable> &tabs, const std::vector<int> &kind, int n_kinds, F launch)
{
    for (int k = 0; k < n_kinds; ++k) {
        ScoreTables q{};
        for (size_t i = 0; i <= tabs.size(); ++i) {
            if (i < tabs.size() && kind[i] == k) q.t[q.n++] = tabs[i];
            if (q.n == 0 || (q.n < kMultiTables && i < tabs.size())) continue;
            const heta_status e = launch(q, k);
            if (e != HETA_OK) return e;
            q.n = 0;
        }
    }
    return HETA_OK;
}

} // namespace

} // namespace heta

using namespace heta;

extern "C" {

heta_status heta_attn_score(const void *x, heta_dtype dt, int64_t ld_x, int64_t n, int32_t d, const float *vec,
                            int32_t heads, int32_t per_head, float *score, void *hip_stream)
{
    if (!vec || (n > 0 && (!x || !score))) return fail(HETA_ERR_INVALID_ARG, "heta_attn_score: null argument");
    if (!valid_dtype(dt)) return fail(HETA_ERR_INVALID_ARG, "heta_attn_score: bad dtype");
    if (n < 0 || d <= 0 || ld_x < d || heads <= 0 || heads > kMaxHeads || (per_head && d % heads != 0))
        return fail(HETA_ERR_SHAPE, "heta_attn_score: bad shape (n=%lld d=%d ld=%lld heads=%d)", (long long)n, d,
                    (long long)ld_x, heads);
    if (reinterpret_cast<uintptr_t>(x) % dtype_size(dt) || reinterpret_cast<uintptr_t>(vec) % 4 || reinterpret_cast<uintptr_t>(score) % 4)
        return fail(HETA_ERR_INVALID_ARG, "heta_attn_score: pointer not aligned to its element size");
    DotParams p{};
    p.x = x;
    p.ld_x = ld_x;
    p.y = vec;
    p.ld_y = 0;
    p.n = n;
    p.d = d;
    p.K = heads;
    p.F = per_head ? d / heads : d;
    p.per_head = per_head ? 1 : 0;
    p.scale = 1.f;
    p.corr = nullptr;
    p.out = score;
    return launch_rowdot(p, dt, HETA_F32, as_stream(hip_stream));
}

heta_status heta_attn_score_bwd(heta_graph *g, const void *x, heta_dtype dt, int64_t ld_x, int64_t n, int32_t d,
                                const float *vec, int32_t heads, int32_t per_head, const float *dscore, float *dx,
                                int64_t ld_dx, float beta, float *dvec, void *hip_stream)
{
    if (!g || !vec || (n > 0 && (!x || !dscore))) return fail(HETA_ERR_INVALID_ARG, "heta_attn_score_bwd: null argument");
    if (!valid_dtype(dt)) return fail(HETA_ERR_INVALID_ARG, "heta_attn_score_bwd: bad dtype");
    if (n < 0 || d <= 0 || ld_x < d || heads <= 0 || heads > kMaxHeads || (per_head && d % heads != 0) || (dx && ld_dx < d))
        return fail(HETA_ERR_SHAPE, "heta_attn_score_bwd: bad shape (n=%lld d=%d heads=%d)", (long long)n, d, heads);
    if (beta != 0.f && beta != 1.f) return fail(HETA_ERR_SHAPE, "heta_attn_score_bwd: beta must be 0 or 1");
    hipStream_t st = as_stream(hip_stream);
    const int F = per_head ? d / heads : d;
    if (dx && n > 0) {
        ProfScope prof("attn_score_bwd_input_kernel", st, static_cast<double>(n) * (d * (beta != 0.f ? 8.0 : 4.0) + 4.0 * heads), 0);
        const bool vec4 = d % 4 == 0 && F % 4 == 0 && ld_dx % 4 == 0 && aligned16(dx) && aligned16(vec);
        const int64_t blocks = (n * (vec4 ? d / 4 : d) + 255) / 256;
        if (blocks > max_blocks(256)) return fail(HETA_ERR_UNSUPPORTED, "heta_attn_score_bwd: too many elements");
        if (vec4)
            hipLaunchKernelGGL(attn_score_bwd_input_vec_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                               dscore, vec, n, (int)d, (int)heads, F, per_head ? 1 : 0, dx, ld_dx, beta);
        else
            hipLaunchKernelGGL(attn_score_bwd_input_kernel, dim3((unsigned)blocks), dim3(256), 0, st, dscore, vec, n, (int)d,
                               (int)heads, F, per_head ? 1 : 0, dx, ld_dx, beta);
        HETA_LAUNCH_CHECK("attn_score_bwd_input_kernel");
    }
    if (dvec) {
        const int nk = per_head ? 1 : heads;
        const int64_t elems = static_cast<int64_t>(nk) * d;
        const int64_t n_slabs = (n + kSlabRows - 1) / kSlabRows;
        if (n_slabs == 0) {
            HETA_HIP(hipMemsetAsync(dvec, 0, elems * sizeof(float), st));
            return HETA_OK;
        }
        heta_status e = ensure_attn(g, static_cast<size_t>(n_slabs) * elems * sizeof(float));
        if (e != HETA_OK) return e;
        float *part = static_cast<float *>(g->d_attn);
        {
            ProfScope prof("attn_score_bwd_param_kernel", st, static_cast<double>(n) * (d * dtype_size(dt) + 4.0 * heads), 0);
            const dim3 grid((unsigned)n_slabs, (d + 255) / 256);
            const bool vec4 = d % 4 == 0 && F % 4 == 0 && ld_x % 4 == 0 && reinterpret_cast<uintptr_t>(x) % (4 * dtype_size(dt)) == 0;
            if (vec4) {
#define HETA_PARAM_VEC(TT, KH)                                                                                          \
    hipLaunchKernelGGL((attn_score_bwd_param_vec_kernel<TT, KH>), grid, dim3(256), 0, st, static_cast<const TT *>(x), ld_x, \
                       dscore, n, (int)d, (int)heads, F, part)
                if (dt == HETA_F32) {
                    if (per_head) HETA_PARAM_VEC(float, 0);
                    else if (heads <= 4) HETA_PARAM_VEC(float, 4);
                    else HETA_PARAM_VEC(float, 16);
                } else {
                    if (per_head) HETA_PARAM_VEC(bf16_t, 0);
                    else if (heads <= 4) HETA_PARAM_VEC(bf16_t, 4);
                    else HETA_PARAM_VEC(bf16_t, 16);
                }
#undef HETA_PARAM_VEC
            } else if (dt == HETA_F32) {
                hipLaunchKernelGGL((attn_score_bwd_param_kernel<float>), grid, dim3(256), 0, st, static_cast<const float *>(x), ld_x,
                                   dscore, n, (int)d, (int)heads, F, per_head ? 1 : 0, part);
            } else {
                hipLaunchKernelGGL((attn_score_bwd_param_kernel<bf16_t>), grid, dim3(256), 0, st, static_cast<const bf16_t *>(x), ld_x,
                                   dscore, n, (int)d, (int)heads, F, per_head ? 1 : 0, part);
            }
            HETA_LAUNCH_CHECK("attn_score_bwd_param_kernel");
            hipLaunchKernelGGL(attn_slab_sum_kernel, dim3((unsigned)((elems + 63) / 64)), dim3(1024), 0, st, part, n_slabs, elems, dvec);
            HETA_LAUNCH_CHECK("attn_slab_sum_kernel");
        }
    }
    return HETA_OK;
}

// whether the one-pass kernels take this table and these vector sets
static bool multi_ok(const void *x, heta_dtype dt, int64_t ld_x, int32_t d, int32_t n_sets, int32_t heads, const float *const *vecs)
{
    if (d > kMultiCols || d % 4 || n_sets > kMultiSets || n_sets * heads > kMultiVecs) return false;
    if (reinterpret_cast<uintptr_t>(x) % (4 * dtype_size(dt)) || ld_x % 4) return false;
    for (int j = 0; j < n_sets; ++j)
        if (!aligned16(vecs[j])) return false;
    return true;
}

heta_status heta_attn_score_multi(const void *x, heta_dtype dt, int64_t ld_x, int64_t n, int32_t d, int32_t n_sets,
                                  const float *const *vecs, int32_t heads, float *const *scores, void *hip_stream)
{
    const int32_t first[2] = {0, n_sets};
    return heta_attn_score_tables(1, first, &x, dt, &ld_x, &n, &d, vecs, heads, scores, hip_stream);
}

heta_status heta_attn_score_tables(int32_t n, const int32_t *first, const void *const *x, heta_dtype dt, const int64_t *ld_x,
                                   const int64_t *n_rows, const int32_t *d, const float *const *vecs, int32_t heads, float *const *scores,
                                   void *hip_stream)
{
    const char *who = "heta_attn_score_multi";
    if (n < 0 || (n > 0 && (!first || !x || !ld_x || !n_rows || !d))) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n > 0 && first[0] != 0) return fail(HETA_ERR_INVALID_ARG, "%s: first must start at 0", who);
    for (int32_t i = 0; i < n; ++i) {
        const int32_t n_sets = first[i + 1] - first[i];
        if (n_sets < 0 || (n_sets > 0 && (!vecs || !scores))) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (n_sets == 0) continue;
        for (int32_t j = first[i]; j < first[i + 1]; ++j)
            if (!vecs[j] || (n_rows[i] > 0 && !scores[j])) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (n_rows[i] > 0 && !x[i]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (!valid_dtype(dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
        if (n_rows[i] < 0 || d[i] <= 0 || ld_x[i] < d[i] || heads <= 0 || heads > kMaxHeads)
            return fail(HETA_ERR_SHAPE, "%s: bad shape (n=%lld d=%d ld=%lld heads=%d)", who, (long long)n_rows[i], d[i], (long long)ld_x[i], heads);
    }
    hipStream_t st = as_stream(hip_stream);
    try {
        std::vector<ScoreTable> tabs;
        std::vector<int> kind; // of kernel: chunks of 16 columns, tiles of 16 vectors, 16-byte stores
        for (int32_t i = 0; i < n; ++i) {
            const int32_t n_sets = first[i + 1] - first[i];
            if (n_sets == 0) continue;
            if (!multi_ok(x[i], dt, ld_x[i], d[i], n_sets, heads, vecs + first[i])) { // shapes the one-pass kernel does not take: set by set
                for (int32_t j = first[i]; j < first[i + 1]; ++j) {
                    heta_status e = heta_attn_score(x[i], dt, ld_x[i], n_rows[i], d[i], vecs[j], heads, 0, scores[j], hip_stream);
                    if (e != HETA_OK) return e;
                }
                continue;
            }
            if (n_rows[i] == 0) continue;
            ScoreTable t = score_table(x[i], ld_x[i], n_rows[i], d[i], n_sets, heads, vecs + first[i], scores + first[i]);
            bool vec4 = heads % 4 == 0;
            for (int32_t j = first[i]; j < first[i + 1]; ++j) vec4 = vec4 && aligned16(scores[j]);
            const int tiles = (t.m.NV + 15) / 16, groups = (tiles + kScoreTiles - 1) / kScoreTiles;
            t.nvc = (tiles + groups - 1) / groups;
            tabs.push_back(t);
            kind.push_back((d[i] <= 32 ? 0 : d[i] <= 64 ? 2 : 4) + (vec4 ? 1 : 0));
        }
#define HETA_SM(TT, NC, V4) hipLaunchKernelGGL((attn_score_multi_kernel<TT, NC, V4>), dim3(blocks), dim3(256), lds, st, q)
#define HETA_SM_V(TT, NC) do { if (k & 1) HETA_SM(TT, NC, true); else HETA_SM(TT, NC, false); } while (0)
#define HETA_SM_T(TT) do { if (k < 2) HETA_SM_V(TT, 2); else if (k < 4) HETA_SM_V(TT, 4); else HETA_SM_V(TT, 8); } while (0)
        return for_tables_of_a_kind(tabs, kind, 6, [&](ScoreTables &q, int k) {
            // one round of workgroups, as many as are resident (four per CU, three of 128 columns), of the same work each: 64 rows
            // at a time times their tiles of vectors
            int64_t work = 0;
            for (int c = 0; c < q.n; ++c) work += (q.t[c].n + 63) / 64 * ((q.t[c].m.NV + 15) / 16);
            const int64_t slots = k < 4 ? 1024 : 768, each = (work + slots - 1) / slots;
            unsigned blocks = 0, lds = 0;
            double bytes = 0;
            for (int c = 0; c < q.n; ++c) {
                ScoreTable &t = q.t[c];
                const int64_t rounds = (each + t.nvc - 1) / t.nvc; // of 64 rows
                t.nb = static_cast<int>(((t.n + 63) / 64 + rounds - 1) / rounds);
                t.first = blocks;
                blocks += t.nb * (((t.m.NV + 15) / 16 + t.nvc - 1) / t.nvc);
                lds = std::max(lds, static_cast<unsigned>(t.nvc) * ((k < 2 ? 2 : k < 4 ? 4 : 8) * 1024 + 16 * 8));
                bytes += static_cast<double>(t.n) * (t.d * dtype_size(dt) + 4.0 * t.m.NV);
            }
            ProfScope prof("attn_score_multi_kernel", st, bytes, 0);
            if (dt == HETA_F32) HETA_SM_T(float);
            else HETA_SM_T(bf16_t);
            HETA_LAUNCH_CHECK("attn_score_multi_kernel");
            return HETA_OK;
        });
#undef HETA_SM_T
#undef HETA_SM_V
#undef HETA_SM
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "%s: host allocation failed", who);
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "%s: unexpected exception", who);
    }
}

heta_status heta_attn_score_bwd_multi(heta_graph *g, const void *x, heta_dtype dt, int64_t ld_x, int64_t n, int32_t d,
                                      int32_t n_sets, const float *const *vecs, int32_t heads, const float *const *dscores,
                                      float *dx, int64_t ld_dx, float beta, float *const *dvecs, void *hip_stream)
{
    const int32_t first[2] = {0, n_sets};
    return heta_attn_score_bwd_tables(g, 1, first, &x, dt, &ld_x, &n, &d, vecs, heads, dscores, &dx, &ld_dx, &beta, dvecs, hip_stream);
}

heta_status heta_attn_score_bwd_tables(heta_graph *g, int32_t n, const int32_t *first, const void *const *x, heta_dtype dt,
                                       const int64_t *ld_x, const int64_t *n_rows, const int32_t *d, const float *const *vecs, int32_t heads,
                                       const float *const *dscores, float *const *dx, const int64_t *ld_dx, const float *beta,
                                       float *const *dvecs, void *hip_stream)
{
    const char *who = "heta_attn_score_bwd_multi";
    if (!g || n < 0 || (n > 0 && (!first || !x || !ld_x || !n_rows || !d || (dx && (!ld_dx || !beta)))))
        return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n > 0 && first[0] != 0) return fail(HETA_ERR_INVALID_ARG, "%s: first must start at 0", who);
    for (int32_t i = 0; i < n; ++i) {
        const int32_t n_sets = first[i + 1] - first[i];
        if (n_sets < 0 || (n_sets > 0 && (!vecs || !dscores))) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (n_sets == 0) continue;
        for (int32_t j = first[i]; j < first[i + 1]; ++j)
            if (!vecs[j] || (n_rows[i] > 0 && !dscores[j])) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (n_rows[i] > 0 && !x[i]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (!valid_dtype(dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
        if (n_rows[i] < 0 || d[i] <= 0 || ld_x[i] < d[i] || heads <= 0 || heads > kMaxHeads || (dx && dx[i] && ld_dx[i] < d[i]))
            return fail(HETA_ERR_SHAPE, "%s: bad shape (n=%lld d=%d heads=%d)", who, (long long)n_rows[i], d[i], heads);
        if (dx && beta[i] != 0.f && beta[i] != 1.f) return fail(HETA_ERR_SHAPE, "%s: beta must be 0 or 1", who);
    }
    hipStream_t st = as_stream(hip_stream);
    try {
        if (n > 1) { // the tables of one call run concurrently
            std::vector<OutRange> outs;
            for (int32_t i = 0; i < n; ++i) {
                std::vector<OutRange> mine;
                if (first[i + 1] > first[i] && dx && dx[i]) mine.emplace_back(dx[i], n_rows[i], ld_dx[i], d[i], 4);
                for (int32_t j = first[i]; dvecs && j < first[i + 1]; ++j)
                    if (dvecs[j]) mine.emplace_back(dvecs[j], heads, d[i], d[i], 4);
                for (const OutRange &a : mine)
                    for (const OutRange &b : outs)
                        if (a.overlaps(b)) return fail(HETA_ERR_INVALID_ARG, "%s: the outputs of two tables overlap", who);
                outs.insert(outs.end(), mine.begin(), mine.end());
            }
        }
        std::vector<ScoreTable> tabs;
        std::vector<int> vec4_of, kind; // kind of the parameter gradient's kernel: 64-column chunks, tiles of 16 vectors; -1: no dvec asked for
        for (int32_t i = 0; i < n; ++i) {
            const int32_t n_sets = first[i + 1] - first[i];
            if (n_sets == 0) continue;
            float *const dxi = dx ? dx[i] : nullptr;
            const float bi = dx ? beta[i] : 0.f;
            float *const *const dv = dvecs ? dvecs + first[i] : nullptr;
            const bool dx_ok = !dxi || (aligned16(dxi) && ld_dx[i] % 4 == 0);
            if (!multi_ok(x[i], dt, ld_x[i], d[i], n_sets, heads, vecs + first[i]) || !dx_ok) { // set by set, accumulating into dx
                for (int32_t j = 0; j < n_sets; ++j) {
                    heta_status e = heta_attn_score_bwd(g, x[i], dt, ld_x[i], n_rows[i], d[i], vecs[first[i] + j], heads, 0, dscores[first[i] + j],
                                                        dxi, dxi ? ld_dx[i] : 0, j == 0 ? bi : 1.f, dv ? dv[j] : nullptr, hip_stream);
                    if (e != HETA_OK) return e;
                }
                continue;
            }
            ScoreTable t = score_table(x[i], ld_x[i], n_rows[i], d[i], n_sets, heads, vecs + first[i], dscores + first[i]);
            bool vec4 = heads % 4 == 0, any_dvec = false;
            for (int32_t j = 0; j < n_sets; ++j) {
                t.m.dvec[j] = dv ? dv[j] : nullptr;
                any_dvec = any_dvec || t.m.dvec[j];
                vec4 = vec4 && aligned16(dscores[first[i] + j]);
            }
            t.dx = dxi;
            t.ld_dx = dxi ? ld_dx[i] : 0;
            t.beta = bi;
            const int nt = t.m.NV <= 16 ? 1 : 2; // tiles of 16 vectors per workgroup of the parameter gradient
            t.nvc = (t.m.NV + 16 * nt - 1) / (16 * nt) * 16 * nt;
            // slabs of a multiple of 64 rows (16 per wavefront and step), at most 1,024 slabs: enough workgroups for
            // four per CU, and the slab sums (8 or 16 KB each) stay small beside the table
            const int64_t most = dt == HETA_F32 && nt == 2 && t.d > 64 ? 768 : 1024;
            t.slab_rows = std::max<int64_t>(128, (t.n + most * 64 - 1) / (most * 64) * 64);
            t.n_slabs = (t.n + t.slab_rows - 1) / t.slab_rows;
            if (any_dvec && t.slab_rows > 0x7fffffff) return fail(HETA_ERR_UNSUPPORTED, "%s: too many rows", who);
            tabs.push_back(t);
            vec4_of.push_back(!t.dx || t.n == 0 ? -1 : vec4 ? 1 : 0);
            kind.push_back(!any_dvec ? -1 : (nt == 1 ? 0 : 1) + (t.d <= 64 ? 0 : 2));
        }
        heta_status e = for_tables_of_a_kind(tabs, vec4_of, 2, [&](ScoreTables &q, int k) {
            size_t lds = 0; // of the table with the most vectors: at most 62,400 bytes
            unsigned blocks = 0;
            double bytes = 0;
            for (int c = 0; c < q.n; ++c) {
                ScoreTable &t = q.t[c];
                lds = std::max(lds, static_cast<size_t>((t.m.NV + 7) / 8 * 8) * (kMultiCols * sizeof(float) + sizeof(float *)));
                t.nb = static_cast<int>(std::min<int64_t>((t.n + 127) / 128, 768));
                t.first = blocks;
                blocks += t.nb;
                bytes += static_cast<double>(t.n) * (t.d * (t.beta != 0.f ? 8.0 : 4.0) + 4.0 * t.m.NV);
            }
            ProfScope prof("attn_score_bwd_input_kernel", st, bytes, 0);
            if (k) hipLaunchKernelGGL((attn_score_bwd_multi_input_kernel<true>), dim3(blocks), dim3(256), lds, st, q);
            else hipLaunchKernelGGL((attn_score_bwd_multi_input_kernel<false>), dim3(blocks), dim3(256), lds, st, q);
            HETA_LAUNCH_CHECK("attn_score_bwd_multi_input_kernel");
            return HETA_OK;
        });
        if (e != HETA_OK) return e;
        const auto part_bytes = [](const ScoreTable &t) { return static_cast<size_t>(t.n_slabs) * t.nvc * kMultiCols * sizeof(float); };
        for (size_t i0 = 0; i0 < tabs.size();) { // tables whose slab sums fit the workspace together: their launches, then one sum
            std::vector<ScoreTable> some;
            std::vector<int> some_kind;
            size_t total = 0;
            while (i0 < tabs.size() && some.size() < kMultiTables) {
                if (kind[i0] >= 0) {
                    if (!some.empty() && total + part_bytes(tabs[i0]) > kAttnGroupBytes) break;
                    some.push_back(tabs[i0]);
                    some_kind.push_back(kind[i0]);
                    total += part_bytes(tabs[i0]);
                }
                ++i0;
            }
            if (some.empty()) continue;
            e = ensure_attn(g, total);
            if (e != HETA_OK) return e;
            float *part = static_cast<float *>(g->d_attn);
            ScoreTables all{};
            unsigned sum_blocks = 0;
            for (size_t c = 0; c < some.size(); ++c) {
                ScoreTable &t = some[c];
                t.part = part;
                part += part_bytes(t) / sizeof(float);
                t.nb = static_cast<int>(std::max<int64_t>(t.n_slabs, 1));
                all.t[c] = t;
                all.t[c].first = sum_blocks;
                sum_blocks += static_cast<unsigned>((static_cast<int64_t>(t.nvc) * kMultiCols + 63) / 64);
                if (t.n_slabs == 0) some_kind[c] = -1; // no rows: the sum writes zeros
            }
            all.n = static_cast<int>(some.size());
            e = for_tables_of_a_kind(some, some_kind, 4, [&](ScoreTables &q, int k) {
                unsigned blocks = 0;
                double bytes = 0;
                for (int c = 0; c < q.n; ++c) {
                    ScoreTable &t = q.t[c];
                    t.first = blocks;
                    blocks += t.nb * (t.nvc / (k & 1 ? 32 : 16));
                    bytes += static_cast<double>(t.n) * (t.d * dtype_size(dt) + 4.0 * t.m.NV);
                }
                ProfScope prof("attn_score_bwd_param_kernel", st, bytes, 0);
#define HETA_SP(TT, NC, NT) hipLaunchKernelGGL((attn_score_bwd_multi_param_kernel<TT, NC, NT>), dim3(blocks), dim3(256), 0, st, q)
#define HETA_SP_N(TT, NC) do { if (k & 1) HETA_SP(TT, NC, 2); else HETA_SP(TT, NC, 1); } while (0)
#define HETA_SP_T(TT) do { if (k & 2) HETA_SP_N(TT, 2); else HETA_SP_N(TT, 1); } while (0)
                if (dt == HETA_F32) HETA_SP_T(float);
                else HETA_SP_T(bf16_t);
#undef HETA_SP_T
#undef HETA_SP_N
#undef HETA_SP
                HETA_LAUNCH_CHECK("attn_score_bwd_multi_param_kernel");
                return HETA_OK;
            });
            if (e != HETA_OK) return e;
            hipLaunchKernelGGL(attn_multi_slab_sum_kernel, dim3(sum_blocks), dim3(1024), 0, st, all);
            HETA_LAUNCH_CHECK("attn_multi_slab_sum_kernel");
        }
        return HETA_OK;
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "%s: host allocation failed", who);
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "%s: unexpected exception", who);
    }
}

heta_status heta_attn_fold(const void *W, heta_dtype w_dt, int64_t ld_w, int32_t d_in, int32_t d_out, const float *a,
                           int32_t heads, float *wa, void *hip_stream)
{
    return heta_attn_fold_multi(1, &W, w_dt, &ld_w, &d_in, &d_out, &a, heads, &wa, hip_stream);
}

heta_status heta_attn_fold_multi(int32_t n, const void *const *W, heta_dtype w_dt, const int64_t *ld_w, const int32_t *d_in,
                                 const int32_t *d_out, const float *const *a, int32_t heads, float *const *wa, void *hip_stream)
{
    if (n < 0 || (n > 0 && (!W || !ld_w || !d_in || !d_out || !a || !wa))) return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold: null argument");
    for (int32_t i = 0; i < n; ++i) {
        if (!W[i] || !a[i] || !wa[i]) return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold: null argument");
        if (!valid_dtype(w_dt)) return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold: bad dtype");
        if (d_in[i] <= 0 || d_out[i] <= 0 || ld_w[i] < d_out[i] || heads <= 0 || heads > kMaxHeads || d_out[i] % heads != 0 ||
            static_cast<int64_t>(d_in[i]) * d_out[i] > (int64_t(1) << 30))
            return fail(HETA_ERR_SHAPE, "heta_attn_fold: bad shape (d_in=%d d_out=%d ld_w=%lld heads=%d)", d_in[i], d_out[i],
                        (long long)ld_w[i], heads);
        if (reinterpret_cast<uintptr_t>(W[i]) % dtype_size(w_dt) || reinterpret_cast<uintptr_t>(a[i]) % 4 || reinterpret_cast<uintptr_t>(wa[i]) % 4)
            return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold: pointer not aligned to its element size");
    }
    hipStream_t st = as_stream(hip_stream);
    const int64_t most = max_blocks(64);
    for (int32_t i0 = 0; i0 < n;) {
        FoldItems q{};
        q.K = heads;
        int64_t blocks = 0; // of an item at most 2^24 (heads divides d_out, and d_in d_out <= 2^30)
        for (; i0 < n && q.n < kFoldItems; ++i0) {
            const int64_t mine = (static_cast<int64_t>(heads) * d_in[i0] + 63) / 64;
            if (blocks + mine > most) break;
            FoldItem &r = q.it[q.n++];
            r.W = W[i0];
            r.ld_w = ld_w[i0];
            r.d_in = d_in[i0];
            r.d_out = d_out[i0];
            r.a = a[i0];
            r.wa = wa[i0];
            r.first = static_cast<unsigned>(blocks);
            blocks += mine;
        }
        if (w_dt == HETA_F32) hipLaunchKernelGGL(attn_fold_kernel<float>, dim3((unsigned)blocks), dim3(64), 0, st, q);
        else hipLaunchKernelGGL(attn_fold_kernel<bf16_t>, dim3((unsigned)blocks), dim3(64), 0, st, q);
        HETA_LAUNCH_CHECK("attn_fold_kernel");
    }
    return HETA_OK;
}

heta_status heta_attn_fold_bwd(const void *W, heta_dtype w_dt, int64_t ld_w, int32_t d_in, int32_t d_out, const float *a,
                               int32_t heads, const float *dwa, float *dW, int64_t ld_dw, float beta, float *da,
                               void *hip_stream)
{
    return heta_attn_fold_bwd_multi(1, &W, w_dt, &ld_w, &d_in, &d_out, &a, heads, &dwa, &dW, &ld_dw, beta, &da, hip_stream);
}

heta_status heta_attn_fold_bwd_multi(int32_t n, const void *const *W, heta_dtype w_dt, const int64_t *ld_w, const int32_t *d_in,
                                     const int32_t *d_out, const float *const *a, int32_t heads, const float *const *dwa, float *const *dW,
                                     const int64_t *ld_dw, float beta, float *const *da, void *hip_stream)
{
    if (n < 0 || (n > 0 && (!W || !ld_w || !d_in || !d_out || !a || !dwa || (dW && !ld_dw))))
        return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold_bwd: null argument");
    for (int32_t i = 0; i < n; ++i) {
        float *const dWi = dW ? dW[i] : nullptr, *const dai = da ? da[i] : nullptr;
        if (!W[i] || !a[i] || !dwa[i]) return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold_bwd: null argument");
        if (!valid_dtype(w_dt)) return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold_bwd: bad dtype");
        if (d_in[i] <= 0 || d_out[i] <= 0 || ld_w[i] < d_out[i] || heads <= 0 || heads > kMaxHeads || d_out[i] % heads != 0 ||
            (dWi && ld_dw[i] < d_out[i]) || static_cast<int64_t>(d_in[i]) * d_out[i] > (int64_t(1) << 30))
            return fail(HETA_ERR_SHAPE, "heta_attn_fold_bwd: bad shape (d_in=%d d_out=%d heads=%d)", d_in[i], d_out[i], heads);
        if (beta != 0.f && beta != 1.f) return fail(HETA_ERR_SHAPE, "heta_attn_fold_bwd: beta must be 0 or 1");
        if (reinterpret_cast<uintptr_t>(W[i]) % dtype_size(w_dt) || reinterpret_cast<uintptr_t>(a[i]) % 4 ||
            reinterpret_cast<uintptr_t>(dwa[i]) % 4 || reinterpret_cast<uintptr_t>(dWi) % 4 || reinterpret_cast<uintptr_t>(dai) % 4)
            return fail(HETA_ERR_INVALID_ARG, "heta_attn_fold_bwd: pointer not aligned to its element size");
    }
    hipStream_t st = as_stream(hip_stream);
    const int64_t most = max_blocks(256);
    for (int32_t i0 = 0; i0 < n;) {
        FoldItems q{};
        q.K = heads;
        q.beta = beta;
        int64_t blocks = 0; // of an item at most 2^22 + 2^28, fewer than `most` for any matrix that has memory
        for (; i0 < n && q.n < kFoldItems; ++i0) {
            const unsigned w_blocks = dW && dW[i0] ? static_cast<unsigned>((static_cast<int64_t>(d_in[i0]) * d_out[i0] + 255) / 256) : 0;
            const unsigned a_blocks = da && da[i0] ? static_cast<unsigned>((d_out[i0] + 3) / 4) : 0;
            if (q.n > 0 && blocks + w_blocks + a_blocks > most) break;
            if (w_blocks + a_blocks == 0) continue;
            FoldItem &r = q.it[q.n++];
            r.W = W[i0];
            r.ld_w = ld_w[i0];
            r.d_in = d_in[i0];
            r.d_out = d_out[i0];
            r.a = a[i0];
            r.dwa = dwa[i0];
            r.dW = dW ? dW[i0] : nullptr;
            r.ld_dw = dW ? ld_dw[i0] : 0;
            r.da = da ? da[i0] : nullptr;
            r.first = static_cast<unsigned>(blocks);
            r.w_blocks = w_blocks;
            blocks += w_blocks + a_blocks;
        }
        if (q.n == 0) continue;
        if (w_dt == HETA_F32) hipLaunchKernelGGL(attn_fold_bwd_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, q);
        else hipLaunchKernelGGL(attn_fold_bwd_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, st, q);
        HETA_LAUNCH_CHECK("attn_fold_bwd_kernel");
    }
    return HETA_OK;
}

heta_status heta_rel_attn_fwd(heta_graph *g, int32_t rel, const void *z, heta_dtype z_dt, int64_t ld_z, int32_t d,
                              int32_t heads, const float *el, const float *er, float slope, void *out,
                              heta_dtype out_dt, int64_t ld_out, float beta, float *smax, float *sinv, void *out_pos,
                              int64_t ld_pos, void *hip_stream)
{
    return heta_rel_attn_fwd_train(g, rel, z, z_dt, ld_z, d, heads, el, er, slope, out, out_dt, ld_out, beta, smax, sinv, out_pos, ld_pos,
                                   nullptr, hip_stream);
}

heta_status heta_rel_attn_fwd_train(heta_graph *g, int32_t rel, const void *z, heta_dtype z_dt, int64_t ld_z, int32_t d,
                                    int32_t heads, const float *el, const float *er, float slope, void *out,
                                    heta_dtype out_dt, int64_t ld_out, float beta, float *smax, float *sinv, void *out_pos,
                                    int64_t ld_pos, float *apos, void *hip_stream)
{
    const heta_attn_fwd_item it = {rel, z, ld_z, el, er, out, ld_out, smax, sinv, out_pos, ld_pos, apos};
    return heta_rel_attn_fwd_train_multi(g, 1, &it, z_dt, d, heads, slope, out_dt, beta, hip_stream);
}

heta_status heta_rel_attn_fwd_train_multi(heta_graph *g, int32_t n, const heta_attn_fwd_item *items, heta_dtype z_dt, int32_t d, int32_t heads,
                                          float slope, heta_dtype out_dt, float beta, void *hip_stream)
{
    if (n < 0 || (n > 0 && !items)) return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: bad item array");
    heta_status e = HETA_OK;
    for (int32_t i = 0; i < n; ++i) {
        const heta_attn_fwd_item &it = items[i];
        e = check_attn_args("heta_rel_attn_fwd", g, it.rel, d, heads);
        if (e != HETA_OK) return e;
        if (!it.z || !it.el || !it.er || !it.out || ((it.smax == nullptr) != (it.sinv == nullptr)))
            return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: null argument (smax and sinv go together)");
        if ((it.out_pos == nullptr) != (items[0].out_pos == nullptr))
            return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: out_pos goes with every item or with none");
        if (!valid_dtype(z_dt) || !valid_dtype(out_dt)) return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: bad dtype");
        if (it.ld_z < d || it.ld_out < d || (it.out_pos && it.ld_pos < d)) return fail(HETA_ERR_SHAPE, "heta_rel_attn_fwd: need d <= ld");
        if (beta != 0.f && beta != 1.f) return fail(HETA_ERR_SHAPE, "heta_rel_attn_fwd: beta must be 0 or 1");
        if (it.out_pos && beta != 0.f) return fail(HETA_ERR_SHAPE, "heta_rel_attn_fwd: out_pos needs beta = 0");
        if (reinterpret_cast<uintptr_t>(it.z) % dtype_size(z_dt) || reinterpret_cast<uintptr_t>(it.out) % dtype_size(out_dt) ||
            reinterpret_cast<uintptr_t>(it.out_pos) % dtype_size(out_dt))
            return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: pointer not aligned to its element size");
    }
    const size_t osz = dtype_size(out_dt);
    const auto range = [&](int32_t i, bool pos) {
        const heta_attn_fwd_item &it = items[i];
        return OutRange(pos ? it.out_pos : it.out, g->rels[it.rel].n_dst, pos ? it.ld_pos : it.ld_out, d, osz);
    };
    for (int32_t i = 0; i < n; ++i)
        for (int32_t j = 0; j < i; ++j)
            for (int k = 0; k < 4; ++k)
                if (range(i, k & 1).overlaps(range(j, k >> 1)))
                    return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_fwd: the outputs of items %d and %d overlap", j, i);
    hipStream_t st = as_stream(hip_stream);
    const auto need = [&](int32_t i) {
        const Relation &r = g->rels[items[i].rel];
        return std::max<size_t>(256, round256(static_cast<size_t>(r.n_edges) * heads * sizeof(float))) + round256(hub_scratch_bytes(r.csr, heads));
    };
    try {
        for (int32_t i0 = 0; i0 < n;) {
            int32_t i1 = i0;
            size_t bytes = 0;
            while (i1 < n && (i1 == i0 || bytes + need(i1) <= kAttnGroupBytes)) bytes += need(i1++);
            e = ensure_attn(g, bytes);
            if (e != HETA_OK) return e;
            char *base = static_cast<char *>(g->d_attn);
            std::vector<Sweep> sw;
            std::vector<SlotAggregation> calls;
            for (int32_t i = i0; i < i1; ++i) {
                const heta_attn_fwd_item &it = items[i];
                const Relation &r = g->rels[it.rel];
                SweepParams sp{};
                sp.K = heads;
                sp.slope = slope;
                sp.row_a = it.er;
                sp.nbr_a = it.el;
                sp.smax = it.smax;
                sp.sinv = it.sinv;
                sp.alpha = reinterpret_cast<float *>(base);
                sp.sign = it.out_pos != nullptr;
                sp.apos = it.apos;
                float *hub_scratch = reinterpret_cast<float *>(base + need(i) - round256(hub_scratch_bytes(r.csr, heads)));
                sw.push_back({&r.csr, sp, hub_scratch, 0});
                calls.push_back({&r.csr, it.z, it.ld_z, sp.alpha, it.out, it.ld_out, it.out_pos, it.ld_pos, {}, false});
                base += need(i);
            }
            e = launch_sweeps<SWEEP_FWD>(sw, st, "attn_sweep_fwd");
            if (e == HETA_OK) e = aggregate_slot_weighted_multi(g, calls, z_dt, d, heads, out_dt, beta, items[0].out_pos != nullptr, 0.f, st);
            if (e != HETA_OK) return e;
            i0 = i1;
        }
        return HETA_OK;
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_rel_attn_fwd: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_rel_attn_fwd: unexpected exception");
    }
}

heta_status heta_rel_attn_bwd(heta_graph *g, int32_t rel, const void *z, heta_dtype z_dt, int64_t ld_z, int32_t d,
                              int32_t heads, const float *el, const float *er, float slope, const float *smax,
                              const float *sinv, const void *o, const void *o_pos, heta_dtype o_dt, int64_t ld_o,
                              const float *grad_out, int64_t ld_go, float *dz, int64_t ld_dz, float *del, float *der,
                              void *hip_stream)
{
    heta_status e = check_attn_args("heta_rel_attn_bwd", g, rel, d, heads);
    if (e != HETA_OK) return e;
    if (!z || !el || !er || !smax || !sinv || !o || !grad_out || !dz || !del || !der)
        return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_bwd: null argument");
    if (!valid_dtype(z_dt) || !valid_dtype(o_dt)) return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_bwd: bad dtype");
    if (ld_z < d || ld_o < d || ld_go < d || ld_dz < d) return fail(HETA_ERR_SHAPE, "heta_rel_attn_bwd: need d <= ld");
    if (reinterpret_cast<uintptr_t>(z) % dtype_size(z_dt) || reinterpret_cast<uintptr_t>(o) % dtype_size(o_dt) ||
        reinterpret_cast<uintptr_t>(o_pos) % dtype_size(o_dt) || reinterpret_cast<uintptr_t>(grad_out) % 4 ||
        reinterpret_cast<uintptr_t>(dz) % 4)
        return fail(HETA_ERR_INVALID_ARG, "heta_rel_attn_bwd: pointer not aligned to its element size");
    const Relation &r = g->rels[rel];
    hipStream_t st = as_stream(hip_stream);
    const int K = heads;
    // workspace: two per-slot weight arrays, per-row terms, and one [max rows x d] fp32 intermediate
    const size_t w_bytes = std::max<size_t>(256, round256(static_cast<size_t>(r.n_edges) * K * sizeof(float)));
    const size_t dst_bytes = round256(static_cast<size_t>(r.n_dst) * K * sizeof(float));
    const size_t src_bytes = round256(static_cast<size_t>(r.n_src) * K * sizeof(float));
    const int64_t ld_r = (static_cast<int64_t>(d) + 3) / 4 * 4;
    const size_t r_bytes = round256(static_cast<size_t>(o_pos ? r.n_src : std::max(r.n_dst, r.n_src)) * ld_r * sizeof(float));
    const size_t hub_bytes = round256(std::max(hub_scratch_bytes(r.csr, K), hub_scratch_bytes(r.csc, K)));
    const size_t pack_bytes = 4 * dst_bytes;
    e = ensure_attn(g, 2 * w_bytes + 2 * dst_bytes + src_bytes + r_bytes + hub_bytes + pack_bytes);
    if (e != HETA_OK) return e;
    char *base = static_cast<char *>(g->d_attn);
    float *w_alpha = reinterpret_cast<float *>(base);
    float *w_gate = reinterpret_cast<float *>(base + w_bytes);
    float *dot = reinterpret_cast<float *>(base + 2 * w_bytes);
    float *corr_d = reinterpret_cast<float *>(base + 2 * w_bytes + dst_bytes);
    float *corr_s = reinterpret_cast<float *>(base + 2 * w_bytes + 2 * dst_bytes);
    float *R = reinterpret_cast<float *>(base + 2 * w_bytes + 2 * dst_bytes + src_bytes);
    float *hub_scratch = reinterpret_cast<float *>(base + 2 * w_bytes + 2 * dst_bytes + src_bytes + r_bytes);
    float *nbr_pack = reinterpret_cast<float *>(base + 2 * w_bytes + 2 * dst_bytes + src_bytes + r_bytes + hub_bytes);

    // dot[v, k] = <g[v, k, :], o[v, k, :]>
    DotParams dp{};
    dp.x = grad_out;
    dp.ld_x = ld_go;
    dp.y = o;
    dp.ld_y = ld_o;
    dp.n = r.n_dst;
    dp.d = d;
    dp.K = K;
    dp.F = d / K;
    dp.per_head = 1;
    dp.scale = 1.f;
    dp.corr = nullptr;
    dp.out = dot;
    if (o_pos) { // <g, o_pos> in the same pass over g; der = (1 - slope) <g, o_pos> - corr_d is finished after the sweep
        dp.y2 = o_pos;
        dp.scale2 = 1.f - slope;
        dp.out2 = der;
    }
    e = launch_rowdot(dp, HETA_F32, o_dt, st);
    if (e != HETA_OK) return e;
    dp.y2 = nullptr;

    try {
    // Destination side: der = sum_e gate_e <g, z[u_e]> - dot * sum_e gate_e, gate_e = alpha_e * LeakyReLU'.
    SweepParams sp{};
    sp.K = K;
    sp.slope = slope;
    sp.row_a = er;
    sp.nbr_a = el;
    sp.smax = const_cast<float *>(smax);
    sp.sinv = const_cast<float *>(sinv);
    sp.dot = dot;
    sp.corr = corr_d;
    if (o_pos) {
        // gate_e = alpha_e (slope + (1 - slope) [logit_e > 0]), so with o_pos = sum over positive-logit edges of
        // alpha_e z[u_e] (saved by the forward): sum_e gate_e <g, z[u_e]> = slope * dot + (1 - slope) <g, o_pos>,
        // and no feature row is gathered on this side.
        sp.gate = nullptr;
        sp.dot_shift = slope;
        std::vector<Sweep> sw(1, Sweep{&r.csr, sp, hub_scratch, 0});
        e = launch_sweeps<SWEEP_BWD_CSR>(sw, st, "attn_sweep_bwd_dst");
        if (e != HETA_OK) return e;
        const int64_t total = r.n_dst * K;
        if (total > 0) {
            hipLaunchKernelGGL(attn_sub_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, der, corr_d, total);
            HETA_LAUNCH_CHECK("attn_sub_kernel");
        }
    } else {
        // without it: R[v] = sum_e gate_e z[u_e] by one more weighted aggregation over the CSR
        sp.gate = w_gate;
        sp.dot_shift = 0.f;
        std::vector<Sweep> sw(1, Sweep{&r.csr, sp, hub_scratch, 0});
        e = launch_sweeps<SWEEP_BWD_CSR>(sw, st, "attn_sweep_bwd_dst");
        if (e != HETA_OK) return e;
        e = aggregate_slot_weighted(g, r.csr, z, z_dt, ld_z, d, w_gate, K, R, HETA_F32, ld_r, 0.f, st);
        if (e != HETA_OK) return e;
        dp.y = R;
        dp.ld_y = ld_r;
        dp.corr = corr_d;
        dp.out = der;
        e = launch_rowdot(dp, HETA_F32, HETA_F32, st);
        if (e != HETA_OK) return e;
    }

    if (r.n_dst > 0) {
        const int64_t total = r.n_dst * K;
        hipLaunchKernelGGL(attn_pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, er, smax, sinv, dot, total,
                           reinterpret_cast<float4 *>(nbr_pack));
        HETA_LAUNCH_CHECK("attn_pack_kernel");
    }
    const SourceSide side = {&r, z, z_dt, ld_z, el, nbr_pack, grad_out, ld_go, dz, ld_dz, del, w_alpha, corr_s, R, hub_scratch, ld_r};
    return attn_source_side(g, &side, 1, d, K, slope, st);
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_rel_attn_bwd: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_rel_attn_bwd: unexpected exception");
    }
}

heta_status heta_attn_bwd_dst(heta_graph *g, int32_t dst_type, int32_t n_rels, const int32_t *rels, int32_t d, int32_t heads, float slope,
                              heta_act act, const float *h, int64_t ld_h, const float *grad_out, int64_t ld_go, float *grad_in,
                              int64_t ld_gi, const float *const *o, const float *const *o_pos, const int64_t *ld_o,
                              const float *const *er, const float *const *smax, const float *const *sinv, const float *const *apos,
                              float *const *der, float *const *pack, void *hip_stream)
{
    const int32_t first[2] = {0, n_rels};
    return heta_attn_bwd_dst_multi(g, 1, &dst_type, first, rels, d, heads, slope, act, &h, &ld_h, &grad_out, &ld_go, &grad_in, &ld_gi, o, o_pos,
                                   ld_o, er, smax, sinv, apos, der, pack, hip_stream);
}

heta_status heta_attn_bwd_dst_multi(heta_graph *g, int32_t n, const int32_t *dst_type, const int32_t *first, const int32_t *rels, int32_t d,
                                    int32_t heads, float slope, heta_act act, const float *const *h, const int64_t *ld_h,
                                    const float *const *grad_out, const int64_t *ld_go, float *const *grad_in, const int64_t *ld_gi,
                                    const float *const *o, const float *const *o_pos, const int64_t *ld_o, const float *const *er,
                                    const float *const *smax, const float *const *sinv, const float *const *apos, float *const *der,
                                    float *const *pack, void *hip_stream)
{
    const char *who = "heta_attn_bwd_dst";
    if (!g) return fail(HETA_ERR_INVALID_ARG, "%s: null graph", who);
    if (n < 0 || (n > 0 && (!dst_type || !first))) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n > 0 && first[0] != 0) return fail(HETA_ERR_INVALID_ARG, "%s: first must start at 0", who);
    const bool relu = act == HETA_ACT_RELU;
    try {
        std::vector<DstParams> types;
        std::vector<int> kind; // 0: 4-byte loads, 1: row by row, 2: rows held in registers
        std::vector<OutRange> outs;
        std::vector<double> bytes;
        int L = 1, T = 1; // lanes per row, chunks per lane
        for (int32_t i = 0; i < n; ++i) {
            const int32_t n_rels = first[i + 1] - first[i], t = dst_type[i];
            if (t < 0 || t >= (int32_t)g->ntypes.size()) return fail(HETA_ERR_INVALID_ARG, "%s: node type %d out of range", who, t);
            if (n_rels < 1 || n_rels > kDstRels) return fail(HETA_ERR_SHAPE, "%s: need 1 <= n_rels <= %d", who, kDstRels);
            if (act != HETA_ACT_NONE && act != HETA_ACT_RELU) return fail(HETA_ERR_INVALID_ARG, "%s: bad act", who);
            if (!rels || !grad_out || !ld_go || !o || !o_pos || !ld_o || !er || !smax || !sinv || !apos || !der || !pack || !grad_out[i] ||
                (relu && (!h || !grad_in || !ld_h || !ld_gi || !h[i] || !grad_in[i])))
                return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
            if (heads <= 0 || heads > kMaxHeads || d <= 0 || d % heads != 0 || ld_go[i] < d || (relu && (ld_h[i] < d || ld_gi[i] < d)))
                return fail(HETA_ERR_SHAPE, "%s: need 1 <= heads <= %d dividing d and d <= ld", who, kMaxHeads);
            DstParams p{};
            p.g = grad_out[i];
            p.ld_g = ld_go[i];
            uintptr_t all16 = reinterpret_cast<uintptr_t>(p.g), all4 = 0;
            int64_t lds = p.ld_g;
            if (relu) {
                p.h = h[i];
                p.ga = grad_in[i];
                p.ld_h = ld_h[i];
                p.ld_ga = ld_gi[i];
                all16 |= reinterpret_cast<uintptr_t>(p.h) | reinterpret_cast<uintptr_t>(p.ga);
                lds |= p.ld_h | p.ld_ga;
            }
            p.n = g->ntypes[t].num_nodes;
            p.d = d;
            p.K = heads;
            p.F = d / heads;
            p.n_rels = n_rels;
            p.slope = slope;
            for (int j = 0; j < n_rels; ++j) {
                const int q = first[i] + j;
                if (rels[q] < 0 || rels[q] >= (int32_t)g->rels.size() || g->rels[rels[q]].dst_type != t)
                    return fail(HETA_ERR_INVALID_ARG, "%s: relation %d does not lead into type %d", who, rels[q], t);
                if (p.n > 0 && (!o[q] || !o_pos[q] || !er[q] || !smax[q] || !sinv[q] || !apos[q] || !der[q] || !pack[q]))
                    return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
                if (ld_o[q] < d) return fail(HETA_ERR_SHAPE, "%s: need d <= ld", who);
                p.it[j] = DstItem{o[q], o_pos[q], er[q], smax[q], sinv[q], apos[q], der[q], pack[q], ld_o[q]};
                all16 |= reinterpret_cast<uintptr_t>(o[q]) | reinterpret_cast<uintptr_t>(o_pos[q]);
                lds |= ld_o[q];
                all4 |= reinterpret_cast<uintptr_t>(er[q]) | reinterpret_cast<uintptr_t>(smax[q]) | reinterpret_cast<uintptr_t>(sinv[q]) |
                        reinterpret_cast<uintptr_t>(apos[q]) | reinterpret_cast<uintptr_t>(der[q]);
                if (!aligned16(pack[q])) return fail(HETA_ERR_INVALID_ARG, "%s: pack not 16-byte aligned", who);
            }
            if ((all16 | all4) % 4) return fail(HETA_ERR_INVALID_ARG, "%s: pointer not 4-byte aligned", who);
            if (n > 1) { // the types of one call run concurrently
                std::vector<OutRange> mine;
                if (relu) mine.emplace_back(p.ga, p.n, p.ld_ga, d, 4);
                for (int j = 0; j < n_rels; ++j) {
                    mine.emplace_back(p.it[j].der, p.n, heads, heads, 4);
                    mine.emplace_back(p.it[j].pack, p.n, 4 * heads, 4 * heads, 4);
                }
                for (const OutRange &a : mine)
                    for (const OutRange &b : outs)
                        if (a.overlaps(b)) return fail(HETA_ERR_INVALID_ARG, "%s: the outputs of two types overlap", who);
                outs.insert(outs.end(), mine.begin(), mine.end());
            }
            if (p.n == 0) continue;
            const int n_chunks = d / 4, cph = p.F / 4;
            while (L < n_chunks && L < 64) L <<= 1;
            while (L * T < n_chunks) T <<= 1;
            const bool vec = d % 4 == 0 && p.F % 4 == 0 && all16 % 16 == 0 && lds % 4 == 0;
            const bool one_pass = vec && (T == 1 || (T <= 4 && (cph & (cph - 1)) == 0));
            types.push_back(p);
            kind.push_back(one_pass ? 2 : vec ? 1 : 0);
            bytes.push_back(static_cast<double>(p.n) * (4.0 * d * (1 + (relu ? 2 : 0) + 2 * n_rels) + 36.0 * heads * n_rels));
        }
        hipStream_t st = as_stream(hip_stream);
        for (int k = 2; k >= 0; --k) {
            DstTypes m{};
            double group_bytes = 0;
            for (size_t i = 0; i <= types.size(); ++i) {
                const bool mine = i < types.size() && kind[i] == k;
                if (mine) {
                    m.t[m.n++] = types[i];
                    group_bytes += bytes[i];
                }
                if (m.n == 0 || (m.n < kDstTypes && i < types.size())) continue;
                // two rows per lane group once that still leaves eight wavefronts per SIMD, else one; one of four chunks per lane
                int64_t all_rows = 0, blocks = 0;
                for (int c = 0; c < m.n; ++c) all_rows += m.t[c].n;
                const int R = k == 2 && T < 4 && all_rows * L >= int64_t(2) * 64 * 8192 ? 2 : 1;
                const int64_t rows = k == 2 ? static_cast<int64_t>(4) * R * (64 / L) : 4;
                for (int c = 0; c < m.n; ++c) {
                    m.t[c].first = blocks;
                    blocks += (m.t[c].n + rows - 1) / rows;
                }
                ProfScope prof("attn_dst_kernel", st, group_bytes, 0);
                launch_pieces(blocks, 256, [&](unsigned piece, unsigned count) {
                    m.first = piece;
                    if (k == 0) hipLaunchKernelGGL(attn_dst_any_kernel<1>, dim3(count), dim3(256), 0, st, m);
                    else if (k == 1) hipLaunchKernelGGL(attn_dst_any_kernel<4>, dim3(count), dim3(256), 0, st, m);
                    else if (T == 4) hipLaunchKernelGGL((attn_dst_kernel<1, 4>), dim3(count), dim3(256), 0, st, m, L);
                    else if (T == 2 && R == 2) hipLaunchKernelGGL((attn_dst_kernel<2, 2>), dim3(count), dim3(256), 0, st, m, L);
                    else if (T == 2) hipLaunchKernelGGL((attn_dst_kernel<1, 2>), dim3(count), dim3(256), 0, st, m, L);
                    else if (R == 2) hipLaunchKernelGGL((attn_dst_kernel<2, 1>), dim3(count), dim3(256), 0, st, m, L);
                    else hipLaunchKernelGGL((attn_dst_kernel<1, 1>), dim3(count), dim3(256), 0, st, m, L);
                });
                HETA_LAUNCH_CHECK("attn_dst_kernel");
                m.n = 0;
                group_bytes = 0;
            }
        }
        return HETA_OK;
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "%s: host allocation failed", who);
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "%s: unexpected exception", who);
    }
}

heta_status heta_rel_attn_bwd_src(heta_graph *g, int32_t rel, const void *z, heta_dtype z_dt, int64_t ld_z, int32_t d, int32_t heads,
                                  const float *el, float slope, const float *pack, const float *grad_out, int64_t ld_go, float *dz,
                                  int64_t ld_dz, float *del, void *hip_stream)
{
    const heta_attn_src_item it = {rel, z, ld_z, el, pack, grad_out, ld_go, dz, ld_dz, del};
    return heta_rel_attn_bwd_src_multi(g, 1, &it, z_dt, d, heads, slope, hip_stream);
}

heta_status heta_rel_attn_bwd_src_multi(heta_graph *g, int32_t n, const heta_attn_src_item *items, heta_dtype z_dt, int32_t d, int32_t heads,
                                        float slope, void *hip_stream)
{
    const char *fn = "heta_rel_attn_bwd_src";
    if (n < 0 || (n > 0 && !items)) return fail(HETA_ERR_INVALID_ARG, "%s: bad item array", fn);
    heta_status e = HETA_OK;
    for (int32_t i = 0; i < n; ++i) {
        const heta_attn_src_item &it = items[i];
        e = check_attn_args(fn, g, it.rel, d, heads);
        if (e != HETA_OK) return e;
        if (!it.z || !it.el || !it.pack || !it.grad_out || !it.dz || !it.del) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", fn);
        if (!aligned16(it.pack)) return fail(HETA_ERR_INVALID_ARG, "%s: pack not 16-byte aligned", fn);
        if (!valid_dtype(z_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", fn);
        if (it.ld_z < d || it.ld_go < d || it.ld_dz < d) return fail(HETA_ERR_SHAPE, "%s: need d <= ld", fn);
        if (reinterpret_cast<uintptr_t>(it.z) % dtype_size(z_dt) || reinterpret_cast<uintptr_t>(it.grad_out) % 4 ||
            reinterpret_cast<uintptr_t>(it.dz) % 4)
            return fail(HETA_ERR_INVALID_ARG, "%s: pointer not aligned to its element size", fn);
        for (int32_t j = 0; j < i; ++j)
            if (OutRange(it.dz, g->rels[it.rel].n_src, it.ld_dz, d, 4)
                    .overlaps(OutRange(items[j].dz, g->rels[items[j].rel].n_src, items[j].ld_dz, d, 4)))
                return fail(HETA_ERR_INVALID_ARG, "%s: the outputs of items %d and %d overlap", fn, j, i);
    }
    const int64_t ld_r = (static_cast<int64_t>(d) + 3) / 4 * 4;
    struct Bytes {
        size_t w, corr, R, hub;
        size_t all() const { return w + corr + R + hub; }
    };
    const auto need = [&](int32_t i) {
        const Relation &r = g->rels[items[i].rel];
        return Bytes{std::max<size_t>(256, round256(static_cast<size_t>(r.n_edges) * heads * sizeof(float))),
                     round256(static_cast<size_t>(r.n_src) * heads * sizeof(float)), round256(static_cast<size_t>(r.n_src) * ld_r * sizeof(float)),
                     round256(hub_scratch_bytes(r.csc, heads))};
    };
    try {
        for (int32_t i0 = 0; i0 < n;) {
            int32_t i1 = i0;
            size_t bytes = 0;
            while (i1 < n && (i1 == i0 || bytes + need(i1).all() <= kAttnGroupBytes)) bytes += need(i1++).all();
            e = ensure_attn(g, bytes);
            if (e != HETA_OK) return e;
            char *base = static_cast<char *>(g->d_attn);
            std::vector<SourceSide> sides;
            for (int32_t i = i0; i < i1; ++i) {
                const heta_attn_src_item &it = items[i];
                const Bytes b = need(i);
                const auto at = [&](size_t off) { return reinterpret_cast<float *>(base + off); };
                sides.push_back({&g->rels[it.rel], it.z, z_dt, it.ld_z, it.el, it.pack, it.grad_out, it.ld_go, it.dz, it.ld_dz, it.del, at(0),
                                 at(b.w), at(b.w + b.corr), at(b.w + b.corr + b.R), ld_r});
                base += b.all();
            }
            e = attn_source_side(g, sides.data(), static_cast<int>(sides.size()), d, heads, slope, as_stream(hip_stream));
            if (e != HETA_OK) return e;
            i0 = i1;
        }
        return HETA_OK;
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "%s: host allocation failed", fn);
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "%s: unexpected exception", fn);
    }
}

} // extern "C"
