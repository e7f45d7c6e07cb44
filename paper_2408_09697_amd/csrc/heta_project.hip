// Per-relation projection on the matrix cores: Z_r = M_r W_r (forward), dM_r = dZ_r W_r^T and
// dW_r = M_r^T dZ_r (backward) - the per-relation weight matrices of an R-GCN-style AGG_r
// (Section 2.1 of the paper) - and the same three products for all relations into one
// destination type at once, where the forward then is Eq. 1 in one pass:
// H_t = sum_r M_r W_r, a single contraction over the concatenated k ranges of the relations.
// This is the only dense contraction on the path and the only place MFMA is used.
//
// One kernel template computes C[M,N] (+)= A[M,K] . B[K,N] with fp32 accumulation:
//   - a workgroup of 2 x WN wavefronts owns a 128 x (64*WN) tile of C, each wavefront a 64 x 64
//     block held as 2 x 2 MFMA 32x32 accumulators (64 VGPRs per lane); WN = 4 (512 threads,
//     256 output columns) lets a 256-wide projection read its input rows from HBM exactly once;
//   - A and B tiles of 32 k-values are staged through LDS in a k-contiguous layout, rows padded
//     by 16 bytes so that the 128-bit fragment reads of 8 consecutive lanes fall on distinct
//     banks; the global loads of tile i+1 are issued before the MFMAs of tile i and only
//     touched (masked, converted, stored to LDS) after them;
//   - an operand is described by how it lies in memory: "k-contiguous" (element (r,k) at
//     base[r*ld + k], copied with 128-bit loads/stores) or "r-contiguous" (element (r,k) at
//     base[k*ld + r], transposed on the way into LDS);
//   - fp32 operands use v_mfma_f32_32x32x2_f32; as soon as one operand is bf16 both are fed as
//     bf16 to v_mfma_f32_32x32x16_bf16.  The k index a lane supplies only has to agree between
//     the A and B fragments, so each lane reads 16 contiguous bytes and spreads them over
//     consecutive MFMAs;
//   - a launch carries up to 8 "segments": either summed into one output (k-concatenation, the
//     fused forward) or independent products that share an operand (all dM_r or all dW_r of a
//     destination type), scheduled next to each other so the shared operand is fetched from
//     HBM once and served from cache to the others;
//   - the weight gradient contracts over graph rows: the row range is split over workgroups,
//     partial products go to the workspace and are added in split order (no atomics).
#include <algorithm>
#include <new>
#include <vector>

#include "heta_gemm.h"
#include "heta_test_hooks.h"

namespace heta {

template <typename CT, typename SA_T, bool A_RC, typename SB_T, bool B_RC, int WN, bool VEC, int BK, bool B_SPLIT = false>
__global__ void __launch_bounds__(128 * WN) gemm_kernel(GemmParams p)
{
    constexpr int NT = 128 * WN, BN = 64 * WN;
    __shared__ __attribute__((aligned(16))) CT As[LdsTile<CT, A_RC, BM, BK>::elems];
    __shared__ __attribute__((aligned(16))) CT Bs[LdsTile<CT, B_RC, BN, BK>::elems];
    // B_SPLIT: an fp32 B is fed to the bf16 MFMAs as two terms (rounded value + what the rounding left)
    __shared__ __attribute__((aligned(16))) CT Bs_lo[B_SPLIT ? LdsTile<CT, B_RC, BN, BK>::elems : 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave / WN) * 64, wn = (wave % WN) * 64;
    const int half = lane >> 5, l32 = lane & 31;

    // workgroup id -> (XCD, position in that XCD's queue) -> (outer, inner).  Workgroups are dealt
    // round-robin to the 8 XCDs; the tiles that share an operand get consecutive positions of ONE
    // XCD's queue and meet in its L2: for a row-parallel product the column tiles and batch
    // segments of a row block (inner), one row block per outer step; for a split contraction
    // (weight gradient) every tile and segment of one split (they share that split's rows of both
    // operands), one split per outer step.
    const int n_batch = p.batch ? p.n_seg : 1;
    const int64_t inner = p.nt * n_batch * (p.partial ? p.mt : 1);
    const int64_t n_outer = p.partial ? p.n_split : p.mt;
    const int64_t xcd = blockIdx.x % 8, jq = blockIdx.x / 8;
    const int64_t in_idx = jq % inner, outer = (jq / inner) * 8 + xcd;
    if (outer >= n_outer) return;
    const int s0 = p.batch ? static_cast<int>(in_idx % n_batch) : 0;
    const int64_t rest = in_idx / n_batch;
    const int64_t n0 = (rest % p.nt) * BN;
    const int64_t m0 = (p.partial ? rest / p.nt : outer) * BM;
    const int64_t split = p.partial ? outer : 0;
    const GemmSeg &out_seg = p.seg[s0];
    if (m0 >= out_seg.M || n0 >= out_seg.N) return; // uniform per workgroup (smaller segment of a batch)
    const int s_end = p.batch ? s0 + 1 : p.n_seg;
    const int rows_a = static_cast<int>(min(out_seg.M - m0, static_cast<int64_t>(BM)));
    const int rows_b = static_cast<int>(min(out_seg.N - n0, static_cast<int64_t>(BN)));

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    TileLoader<SA_T, CT, A_RC, BM, NT, VEC, BK> la;
    TileLoader<SB_T, CT, B_RC, BN, NT, VEC, BK> lb;

    // The tile sequence runs over the k range of this split in every segment of the block.
    // (ls, lk, lend) describe the tile whose loads are issued next.
    const int64_t kb = split * p.k_per_split;
    int ls = s0 - 1;
    int64_t lk = 0, lend = 0;
    auto next_segment = [&]() -> bool {
        for (++ls; ls < s_end; ++ls) {
            const GemmSeg &g = p.seg[ls];
            lend = min(g.K, kb + p.k_per_split);
            if (kb < lend) {
                lk = kb;
                la.init(static_cast<const SA_T *>(g.A), g.lda, m0, kb, tid);
                lb.init(static_cast<const SB_T *>(g.B), g.ldb, n0, kb, tid);
                return true;
            }
        }
        return false;
    };
    auto issue = [&]() {
        const int k_left = static_cast<int>(min(lend - lk, static_cast<int64_t>(BK)));
        la.load(rows_a, k_left, tid);
        lb.load(rows_b, k_left, tid);
        lk += BK;
    };
    bool have = next_segment();
    if (have) issue();
    while (have) {
        __syncthreads(); // previous tile fully consumed
        la.store(As, tid);
        lb.store(Bs, tid);
        if constexpr (B_SPLIT) lb.store_residual(Bs_lo, tid);
        __syncthreads();
        // start the next tile's loads; they complete behind the MFMAs below
        have = lk < lend || next_segment();
        if (have) issue();
        if constexpr (sizeof(CT) == 4) {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 8) {
                float a[2][4], b[2][4];
#pragma unroll
                for (int i = 0; i < 2; ++i) frag_f32<A_RC, BM, BK>(As, wm + i * 32 + l32, kk, half, a[i]);
#pragma unroll
                for (int j = 0; j < 2; ++j) frag_f32<B_RC, BN, BK>(Bs, wn + j * 32 + l32, kk, half, b[j]);
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][t], b[j][t], acc[i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < BK; kk += 16) {
                union Frag { uint4 u; bf16x8 v; } a[2], b[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) a[i].u = frag_bf16<A_RC, BM, BK>(As, wm + i * 32 + l32, kk, half);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[j].u = frag_bf16<B_RC, BN, BK>(Bs, wn + j * 32 + l32, kk, half);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i].v, b[j].v, acc[i][j], 0, 0, 0);
                if constexpr (B_SPLIT) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) b[j].u = frag_bf16<B_RC, BN, BK>(Bs_lo, wn + j * 32 + l32, kk, half);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i].v, b[j].v, acc[i][j], 0, 0, 0);
                }
            }
        }
    }

    // epilogue: accumulator register v of lane (half, l32) is C[8*(v/4) + 4*half + v%4][l32] of its 32x32 tile
    float *C = out_seg.C + (p.partial ? split * out_seg.M * out_seg.ldc : 0);
    const bool direct = !p.partial;
    const bool plain = !direct || (!p.row_scale && p.beta == 0.f && !p.relu);
    const bool interior = rows_a == BM && rows_b == BN;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int nl = wn + j * 32 + l32;
            float *col = C + (m0 + wm + i * 32 + 4 * half) * out_seg.ldc + n0 + nl;
            if (p.out_bf16) { // bf16 output: same element mapping, 16-bit stores
                if (nl >= rows_b) continue;
                bf16_t *hcol = reinterpret_cast<bf16_t *>(out_seg.C) + (m0 + wm + i * 32 + 4 * half) * out_seg.ldc + n0 + nl;
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (wm + i * 32 + 8 * (v / 4) + 4 * half + (v % 4) < rows_a)
                        hcol[(8 * (v / 4) + (v % 4)) * out_seg.ldc] = to_bf16(acc[i][j][v]);
                continue;
            }
            if (interior && plain) {
#pragma unroll
                for (int v = 0; v < 16; ++v) col[(8 * (v / 4) + (v % 4)) * out_seg.ldc] = acc[i][j][v];
                continue;
            }
            if (nl >= rows_b) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int ml = wm + i * 32 + 8 * (v / 4) + 4 * half + (v % 4);
                if (ml >= rows_a) continue;
                float val = acc[i][j][v];
                float *o = col + (8 * (v / 4) + (v % 4)) * out_seg.ldc;
                if (direct) {
                    if (p.row_scale) val *= p.row_scale[m0 + ml];
                    if (p.beta != 0.f) val += p.beta * *o;
                    if (p.relu) val = fmaxf(val, 0.f);
                }
                *o = val;
            }
        }
}

// out[m, n] = beta * out[m, n] + sum over splits (in split order) of part[s][m][n], for every segment of
// a batched weight gradient in one launch (blockIdx.y = segment)
struct SplitSegs { // passed by value
    const float *part[kMaxLaunchSeg];
    float *out[kMaxLaunchSeg];
    int64_t M[kMaxLaunchSeg], ldo[kMaxLaunchSeg];
    int32_t N[kMaxLaunchSeg], n_split[kMaxLaunchSeg], chains[kMaxLaunchSeg];
    float beta;
    unsigned first; // first workgroup of this launch
};
// NW wavefronts per 64 elements: wavefront w adds the splits w, w + NW, ... (eight loads in flight), the NW sums are
// added in wavefront order through LDS.  16 wavefronts from 128 splits on, else 4 (with one thread per element, a serial
// chain on a few dozen workgroups, 8,192 elements x 688 splits took 17.4 us, now 8); one, four of them in a workgroup,
// below 32 splits of 196,608 elements and more, which are three wavefronts per SIMD by themselves (whole weight
// gradients with four and with one: three of 2,000 rows, 768 x 1,024, bf16 65.7 / 57.5 us; one of 9,000 rows 49.0 / 45.0,
// of 110,000 rows, 789 x 256, 107.8 / 100.4; of 500 rows, 128 x 256, fp32 17.3 / 18.2).  The number follows from each
// gradient's own call, whatever shares the launch: it decides the order of the sum.
static int split_chains(int64_t n_split, int64_t out_elems) { return n_split >= 128 ? 16 : n_split >= 32 || out_elems < 196608 ? 4 : 1; }
// NT threads: NT / (64 NW) times 64 elements.
template <int NW, int NT> __device__ __forceinline__ void splitk_reduce(const SplitSegs &g, float (*red)[64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, w = wave % NW;
    const int seg = blockIdx.y, n_split = g.n_split[seg];
    const int64_t N = g.N[seg], total = g.M[seg] * N;
    const float beta = g.beta;
    const int64_t block = static_cast<int64_t>(g.first) + blockIdx.x;
    const int64_t t = (block * (NT / (64 * NW)) + wave / NW) * 64 + lane;
    const float *part = g.part[seg];
    float a = 0.f;
    if (t < total) {
#pragma unroll 8
        for (int s = w; s < n_split; s += NW) a += part[static_cast<int64_t>(s) * total + t];
    }
    if (NW > 1) {
        red[wave][lane] = a;
        __syncthreads();
    }
    if (w != 0 || t >= total) return;
    if (NW > 1) {
        a = 0.f;
#pragma unroll
        for (int i = 0; i < NW; ++i) a += red[wave + i][lane];
    }
    const int64_t m = t / N, n = t % N;
    float *o = g.out[seg] + m * g.ldo[seg] + n;
    *o = (beta != 0.f) ? beta * *o + a : a;
}
// 1,024 threads where a gradient of the launch has 16 chains, else 256
template <int NT> __global__ void __launch_bounds__(NT) splitk_reduce_kernel(SplitSegs g)
{
    __shared__ float red[NT / 64][64];
    const int chains = g.chains[blockIdx.y]; // uniform
    if (NT == 1024 && chains == 16) splitk_reduce<NT / 64, NT>(g, red);
    else if (chains == 4) splitk_reduce<4, NT>(g, red);
    else splitk_reduce<1, NT>(g, red);
}

// bf16 weight matrices as octets, out[k / 8][n][8 k-values] of B(k, n) = W[k*ldw + n] (TRANS: W[n*ldw + k]), zero beyond K
// and N: the form that the direct-to-LDS pipeline copies 1 KB at a time.  blockIdx.y picks the matrix: the weights of
// every segment of a product in one launch.
struct OctetSegs {
    const bf16_t *W[kMaxLaunchSeg];
    uint4 *out[kMaxLaunchSeg];
    int64_t ldw[kMaxLaunchSeg];
    int K[kMaxLaunchSeg], N[kMaxLaunchSeg], ko[kMaxLaunchSeg], n_pad[kMaxLaunchSeg];
    int vec; // rows of every W 16-byte aligned
};
template <bool TRANS> __global__ void __launch_bounds__(256) pack_octets_kernel(OctetSegs q)
{
    const int s = blockIdx.y;
    const bf16_t *W = q.W[s];
    const int64_t ldw = q.ldw[s];
    const int K = q.K[s], N = q.N[s], ko = q.ko[s], n_pad = q.n_pad[s];
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    // neighbouring threads: neighbouring columns, or (TRANS) neighbouring octets of a column, as W lies in memory
    const int n = static_cast<int>(TRANS ? idx / ko : idx % n_pad), o = static_cast<int>(TRANS ? idx % ko : idx / n_pad);
    if (o >= ko || n >= n_pad) return;
    if (TRANS && q.vec && 8 * o + 8 <= K && n < N) {
        q.out[s][static_cast<int64_t>(o) * n_pad + n] = *reinterpret_cast<const uint4 *>(W + n * ldw + 8 * o);
        return;
    }
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t x[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int k = o * 8 + 2 * j + e;
            x[e] = (k < K && n < N) ? (TRANS ? W[n * ldw + k] : W[k * ldw + n]) : 0;
        }
        w[j] = x[0] | (x[1] << 16);
    }
    q.out[s][static_cast<int64_t>(o) * n_pad + n] = make_uint4(w[0], w[1], w[2], w[3]);
}

// ---- host side -------------------------------------------------------------------------------------

static void gemm_cost(const GemmParams &p, heta_dtype a_dt, heta_dtype b_dt, double *bytes, double *flops);
// test hook: route every projection through the register-staged kernel
static bool g_force_staged = false;

static bool vec_ok(const void *ptr, int64_t ld, heta_dtype dt)
{
    return aligned16(ptr) && (ld * (int64_t)dtype_size(dt)) % 16 == 0;
}

template <typename CT, typename SA_T, bool A_RC, typename SB_T, bool B_RC, int WN, bool VEC>
static heta_status launch_gemm(GemmParams &p, hipStream_t st, int bk)
{
    constexpr int BN = 64 * WN;
    int64_t mt = 0, nt = 0;
    double bytes = 0, flops = 0;
    gemm_cost(p, sizeof(SA_T) == 4 ? HETA_F32 : HETA_BF16, sizeof(SB_T) == 4 ? HETA_F32 : HETA_BF16, &bytes, &flops);
    for (int s = 0; s < p.n_seg; ++s) {
        mt = std::max(mt, (p.seg[s].M + BM - 1) / BM);
        nt = std::max(nt, (p.seg[s].N + BN - 1) / BN);
    }
    p.mt = mt;
    p.nt = nt;
    const int64_t inner = nt * (p.batch ? p.n_seg : 1) * (p.partial ? mt : 1);
    const int64_t n_outer = p.partial ? std::max(1, p.n_split) : mt;
    const int64_t blocks = (n_outer + 7) / 8 * 8 * inner;
    if (blocks <= 0) return HETA_OK;
    if (blocks > max_blocks(128 * WN)) return fail(HETA_ERR_UNSUPPORTED, "projection: matrix too large for one launch");
    ProfScope prof(sizeof(CT) == 4 ? (p.partial ? "gemm_wgrad_f32" : "gemm_f32") : (p.partial ? "gemm_wgrad_bf16" : "gemm_bf16"),
                   st, bytes, flops);
    if constexpr (sizeof(CT) == 2 && A_RC && B_RC && sizeof(SB_T) == 4) {
        if (p.split_b) {
            hipLaunchKernelGGL((gemm_kernel<CT, SA_T, A_RC, SB_T, B_RC, WN, VEC, 64, true>), dim3((unsigned)blocks), dim3(128 * WN), 0, st, p);
            HETA_LAUNCH_CHECK("gemm_kernel");
            return HETA_OK;
        }
    }
    if (sizeof(CT) == 2 && A_RC && B_RC && bk == 64)
        hipLaunchKernelGGL((gemm_kernel<CT, SA_T, A_RC, SB_T, B_RC, WN, VEC, (sizeof(CT) == 2 && A_RC && B_RC) ? 64 : 32>),
                           dim3((unsigned)blocks), dim3(128 * WN), 0, st, p);
    else
        hipLaunchKernelGGL((gemm_kernel<CT, SA_T, A_RC, SB_T, B_RC, WN, VEC, 32>), dim3((unsigned)blocks), dim3(128 * WN), 0, st, p);
    HETA_LAUNCH_CHECK("gemm_kernel");
    return HETA_OK;
}

// work and algorithmic traffic of a launch: every distinct operand once, every output once
// (twice when accumulating)
static void gemm_cost(const GemmParams &p, heta_dtype a_dt, heta_dtype b_dt, double *bytes, double *flops)
{
    *bytes = 0;
    *flops = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        const GemmSeg &g = p.seg[s];
        bool first = p.n_call == 0 && s == 0; // of its call
        float beta = p.beta;
        for (int c = 0; c < p.n_call; ++c)
            if (s >= p.call[c].first) {
                first = s == p.call[c].first;
                beta = p.call[c].beta;
            }
        *flops += 2.0 * g.M * g.N * g.K;
        bool a_seen = false, b_seen = false;
        for (int q = 0; q < s; ++q) {
            a_seen = a_seen || p.seg[q].A == g.A;
            b_seen = b_seen || p.seg[q].B == g.B;
        }
        if (!a_seen) *bytes += static_cast<double>(g.M) * g.K * dtype_size(a_dt);
        if (!b_seen) *bytes += static_cast<double>(g.K) * g.N * dtype_size(b_dt);
        if (p.batch || first) *bytes += static_cast<double>(g.M) * g.N * (p.out_bf16 ? 2.0 : 4.0) * ((beta != 0.f && !p.partial) ? 2.0 : 1.0);
    }
}

// one call by the register-staged kernel
template <bool A_RC, bool B_RC> static heta_status staged_gemm(GemmParams &p, heta_dtype a_dt, heta_dtype b_dt, hipStream_t st, int bk)
{
    int64_t n_max = 0;
    bool vec = true; // 128-bit loads need every operand of the launch to qualify
    for (int s = 0; s < p.n_seg; ++s) {
        vec = vec && vec_ok(p.seg[s].A, p.seg[s].lda, a_dt) && vec_ok(p.seg[s].B, p.seg[s].ldb, b_dt);
        n_max = std::max(n_max, p.seg[s].N);
    }
    const bool wide = n_max > 128;
#define HETA_GEMM(CT, SA, SB)                                                                                   \
    return wide ? (vec ? launch_gemm<CT, SA, A_RC, SB, B_RC, 4, true>(p, st, bk)                                    \
                       : launch_gemm<CT, SA, A_RC, SB, B_RC, 4, false>(p, st, bk))                                  \
                : (vec ? launch_gemm<CT, SA, A_RC, SB, B_RC, 2, true>(p, st, bk)                                    \
                       : launch_gemm<CT, SA, A_RC, SB, B_RC, 2, false>(p, st, bk))
    if (a_dt == HETA_F32 && b_dt == HETA_F32) { HETA_GEMM(float, float, float); }
    if (a_dt == HETA_F32 && b_dt == HETA_BF16) { HETA_GEMM(bf16_t, float, bf16_t); }
    if (a_dt == HETA_BF16 && b_dt == HETA_F32) { HETA_GEMM(bf16_t, bf16_t, float); }
    HETA_GEMM(bf16_t, bf16_t, bf16_t);
#undef HETA_GEMM
}

template <bool A_RC, bool B_RC>
static heta_status dispatch_gemm(GemmParams &p, heta_dtype a_dt, heta_dtype b_dt, hipStream_t st, int bk = 32)
{
    if (!g_force_staged) {
        // the direct-to-LDS pipeline takes every launch whose operands have 16-byte rows
        double bytes, flops;
        gemm_cost(p, a_dt, b_dt, &bytes, &flops);
        const bool f32 = a_dt == HETA_F32 && b_dt == HETA_F32;
        const char *name = f32 ? (p.partial ? "gemm_wgrad_f32" : "gemm_f32") : (p.partial ? "gemm_wgrad_bf16" : "gemm_bf16");
        bool handled = false;
        heta_status e = launch_gemm_direct(p, a_dt, b_dt, A_RC, B_RC, st, name, bytes, flops, &handled);
        if (e != HETA_OK || handled) return e;
    }
    if (p.n_call <= 1) return staged_gemm<A_RC, B_RC>(p, a_dt, b_dt, st, bk);
    for (int c = 0; c < p.n_call; ++c) { // the staged kernel knows nothing of calls: one launch each
        const GemmCall &call = p.call[c];
        GemmParams one = p;
        one.n_call = 0;
        one.n_seg = call.n_seg;
        std::copy(p.seg + call.first, p.seg + call.first + call.n_seg, one.seg);
        one.row_scale = call.row_scale;
        one.beta = call.beta;
        one.relu = call.relu;
        one.n_split = call.n_split;
        one.k_per_split = call.n_split > 1 ? call.k_per_split : int64_t(1) << 40;
        heta_status e = staged_gemm<A_RC, B_RC>(one, a_dt, b_dt, st, bk);
        if (e != HETA_OK) return e;
    }
    return HETA_OK;
}

static bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) != 0; }

// the handle's buffer for rewritten weight matrices holds at least `bytes`
static heta_status ensure_pack(heta_graph *owner, size_t bytes)
{
    if (bytes <= owner->pack_bytes) return HETA_OK;
    if (owner->d_pack) {
        HETA_HIP(hipDeviceSynchronize()); // earlier readers
        scratch_free(owner->d_pack);
    }
    owner->d_pack = nullptr;
    owner->pack_bytes = 0;
    HETA_HIP(scratch_alloc(&owner->d_pack, bytes * 2));
    owner->pack_bytes = bytes * 2;
    return HETA_OK;
}

// fp32 x fp32 products through a graph handle whose B operands are weight matrices (forward, input gradient):
// the weights are rewritten once per launch as the three bf16 terms the product is fed with, into the handle's
// packing buffer, and the k loop splits only A.  Launches the direct pipeline would not take, or would give tiles that
// split both operands, are left as they are.  trans: B(k, n) = W[n*ldb + k].
static heta_status pack_f32_weights(heta_graph *owner, GemmParams &p, int trans, hipStream_t st)
{
    if (!owner || g_force_staged || g_f32_native || p.partial) return HETA_OK;
    p.as_packed = 1;
    if (p.form != kFormPacked) return HETA_OK;
    size_t bytes = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        const GemmSeg &g = p.seg[s];
        if (!aligned16(g.A) || (g.lda * 4) % 16 || !aligned16(g.B) || (g.ldb * 4) % 16) return HETA_OK;
        bytes += split3_weight_bytes(g.K, g.N, trans);
    }
    heta_status e = ensure_pack(owner, bytes);
    if (e != HETA_OK) return e;
    return pack_split3_weights(p, trans, owner->d_pack, st);
}

// bf16 weights through a graph handle: rewritten once per launch as octets into the handle's packing buffer.  A forward
// product's lie with the contraction index outermost and are always rewritten; an input gradient's can be copied into LDS as
// they are, and packing them takes a launch (5 us): from 48 k steps of 64 x 64 x 16 on the product gains more.  In us,
// unpacked and packed (with the packing): 192 tiles of 128 x 128 over 1,024 k-values (48 k steps) 25.0 and 30.4, 544 over 256
// (34 k) 27.9 and 31.9; seven relations of 64 columns summed into 128 columns of 187,000 rows (60 k) 79.8 and 69.3; 20,000 x
// 1,024 x 768 (245 k) 60 and 52, three of 700,000 x 256 x 128 376 and 319.
static heta_status pack_bf16_weights(heta_graph *owner, GemmParams &p, heta_dtype in_dt, int trans, hipStream_t st)
{
    if (!owner || g_force_staged || p.partial) return HETA_OK;
    const auto octets = [](const GemmSeg &g) { return (g.K + 31) / 32 * 4; }; // whole tiles of 32 k-values
    const auto columns = [](const GemmSeg &g) { return (g.N + 63) / 64 * 64; };
    size_t bytes = 0;
    double steps = 0; // of 64 x 64 x 16
    for (int s = 0; s < p.n_seg; ++s) {
        const GemmSeg &g = p.seg[s];
        const int64_t a_row = g.lda * static_cast<int64_t>(dtype_size(in_dt));
        if (!aligned16(g.A) || a_row % 16 || a_row * 256 >= (int64_t(1) << 31)) return HETA_OK; // not for the direct pipeline
        if (g.K >= (int64_t(1) << 30) || g.N >= (int64_t(1) << 30) || octets(g) * columns(g) >= (int64_t(1) << 31)) return HETA_OK;
        bytes += static_cast<size_t>(octets(g) * columns(g)) * 16;
        steps += static_cast<double>((g.M + 63) / 64) * static_cast<double>((g.N + 63) / 64) * static_cast<double>((g.K + 15) / 16);
    }
    if (trans && steps <= 49152) return HETA_OK;
    heta_status e = ensure_pack(owner, bytes);
    if (e != HETA_OK) return e;
    uint4 *dst = static_cast<uint4 *>(owner->d_pack);
    OctetSegs q{};
    q.vec = 1;
    int64_t chunks = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        GemmSeg &g = p.seg[s];
        q.W[s] = static_cast<const bf16_t *>(g.B);
        q.vec = q.vec && vec_ok(g.B, g.ldb, HETA_BF16);
        q.out[s] = dst;
        q.ldw[s] = g.ldb;
        q.K[s] = static_cast<int>(g.K);
        q.N[s] = static_cast<int>(g.N);
        q.ko[s] = static_cast<int>(octets(g));
        q.n_pad[s] = static_cast<int>(columns(g));
        chunks = std::max(chunks, octets(g) * columns(g));
        g.B = g.B3 = dst;
        g.ldb = 8; // (not walked by rows)
        g.n_pad = q.n_pad[s];
        dst += octets(g) * columns(g);
    }
    const dim3 grid((unsigned)((chunks + 255) / 256), p.n_seg);
    if (trans) hipLaunchKernelGGL(pack_octets_kernel<true>, grid, dim3(256), 0, st, q);
    else hipLaunchKernelGGL(pack_octets_kernel<false>, grid, dim3(256), 0, st, q);
    HETA_LAUNCH_CHECK("pack_octets_kernel");
    return HETA_OK;
}

// out = beta*out + row_scale * sum_s in_s . (W_s or W_s^T): the checked arguments as launch parameters (n_seg 0: no rows)
static heta_status project_plan(GemmParams &p, int64_t n_rows, int n_seg, const void *const *ins, heta_dtype in_dt, const int64_t *ld_in,
                                const int32_t *d_in, const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w, int32_t d_out, int32_t transW,
                                const float *row_scale, int relu, void *out, int64_t ld_out, float beta, const char *who, heta_dtype out_dt,
                                void *const *outs, const int64_t *ld_outs)
{
    // outs != nullptr: n_seg independent products, one output each (out / ld_out unused); else one summed output
    if (outs && n_seg >= 1) {
        if (!ld_outs) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        for (int s = 0; s < n_seg && s < kMaxSeg; ++s) {
            if (!outs[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
            if (ld_outs[s] < d_out) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
            if (misaligned(outs[s], dtype_size(valid_dtype(out_dt) ? out_dt : HETA_F32)))
                return fail(HETA_ERR_INVALID_ARG, "%s: out not aligned to its element size", who);
        }
        out = outs[0];
        ld_out = ld_outs[0];
    }
    if (!ins || !Ws || !out || !ld_in || !d_in || !ld_w) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n_seg < 1 || n_seg > kMaxSeg) return fail(HETA_ERR_INVALID_ARG, "%s: between 1 and %d inputs", who, kMaxSeg);
    if (!valid_dtype(in_dt) || !valid_dtype(w_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
    for (int s = 0; s < n_seg; ++s)
        if (!ins[s] || !Ws[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n_rows < 0 || d_out <= 0 || ld_out < d_out) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
    if (!valid_dtype(out_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
    if (misaligned(out, dtype_size(out_dt))) return fail(HETA_ERR_INVALID_ARG, "%s: out not aligned to its element size", who);
    if (out_dt == HETA_BF16 && (beta != 0.f || row_scale || relu))
        return fail(HETA_ERR_UNSUPPORTED, "%s: a bf16 output takes no beta, row_scale or activation", who);
    p = GemmParams{};
    p.out_bf16 = out_dt == HETA_BF16;
    for (int s = 0; s < n_seg; ++s) {
        if (d_in[s] <= 0 || ld_in[s] < d_in[s] || ld_w[s] < (transW ? d_in[s] : d_out))
            return fail(HETA_ERR_SHAPE, "%s: leading dimension smaller than the row width", who);
        if (misaligned(ins[s], dtype_size(in_dt)) || misaligned(Ws[s], dtype_size(w_dt)))
            return fail(HETA_ERR_INVALID_ARG, "%s: pointer not aligned to its element size", who);
        GemmSeg &g = p.seg[s];
        g.A = ins[s];
        g.lda = ld_in[s];
        g.B = Ws[s];
        g.ldb = ld_w[s];
        g.C = static_cast<float *>(outs ? outs[s] : out); // typed by p.out_bf16 in the kernels' epilogue
        g.ldc = outs ? ld_outs[s] : ld_out;
        g.M = n_rows;
        g.N = d_out;
        g.K = d_in[s];
    }
    if (n_rows == 0) return HETA_OK;
    p.n_seg = n_seg;
    p.batch = outs ? 1 : 0;
    p.row_scale = row_scale;
    p.beta = beta;
    p.relu = relu;
    p.k_per_split = int64_t(1) << 40;
    p.n_split = 1;
    p.partial = 0;
    return HETA_OK;
}

// The planned call, or the calls merged into one plan.  pack_bwd: whether transposed bf16 weights may go through the packing
// buffer too.  heta_project_multi only: callers of the single calls may run those on several streams or capture the first
// one, neither of which a shared buffer that grows allows.
static heta_status project_run(GemmParams &p, heta_dtype in_dt, heta_dtype w_dt, int32_t transW, heta_graph *pack_owner, hipStream_t st,
                               bool pack_bwd)
{
    if (p.n_seg == 0) return HETA_OK;
    if (in_dt == HETA_F32 && w_dt == HETA_F32) {
        if (p.form == kFormNone) p.form = f32_product_form(p);
        heta_status pe = pack_f32_weights(pack_owner, p, transW, st);
        if (pe != HETA_OK) return pe;
    }
    if (w_dt == HETA_BF16 && (!transW || pack_bwd)) {
        heta_status pe = pack_bf16_weights(pack_owner, p, in_dt, transW, st);
        if (pe != HETA_OK) return pe;
    }
    // B[k][n] = W[k][n] is n-contiguous (r-contiguous in the loader's terms); W^T is k-contiguous
    if (transW || (w_dt == HETA_BF16 && p.seg[0].B3)) return dispatch_gemm<false, false>(p, in_dt, w_dt, st);
    return dispatch_gemm<false, true>(p, in_dt, w_dt, st);
}

static heta_status project_impl(int64_t n_rows, int n_seg, const void *const *ins, heta_dtype in_dt, const int64_t *ld_in,
                                const int32_t *d_in, const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w,
                                int32_t d_out, int32_t transW, const float *row_scale, int relu, void *out,
                                int64_t ld_out, float beta, hipStream_t st, const char *who, heta_graph *pack_owner = nullptr,
                                heta_dtype out_dt = HETA_F32, void *const *outs = nullptr, const int64_t *ld_outs = nullptr)
{
    GemmParams p;
    heta_status e = project_plan(p, n_rows, n_seg, ins, in_dt, ld_in, d_in, Ws, w_dt, ld_w, d_out, transW, row_scale, relu, out, ld_out, beta, who,
                                 out_dt, outs, ld_outs);
    return e == HETA_OK ? project_run(p, in_dt, w_dt, transW, pack_owner, st, false) : e;
}

// ---- several calls in one launch -------------------------------------------------------------------------------------
// A launch of a few hundred workgroups leaves the chip idle at its end, and one of a few dozen from the start; calls of
// one layer that do not depend on each other (one per node type) run side by side in one launch instead.  Calls of more
// than kMergeTiles tiles of 128 x 128 (three to four rounds of workgroups) have the chip to themselves anyway and keep
// the tiles that suit them; calls whose widest outputs take different tiles do not meet.
constexpr int64_t kMergeTiles = 2048;
static int width_class(const GemmParams &p)
{
    int64_t n = 0;
    for (int s = 0; s < p.n_seg; ++s) n = std::max(n, p.seg[s].N);
    return n <= 64 ? 0 : n <= 128 ? 1 : n <= 256 ? 2 : n <= 320 ? 3 : 4;
}
static bool merges(const GemmParams &p, heta_dtype a_dt, heta_dtype b_dt)
{
    // (the direct pipeline has no kernel for bf16 inputs with fp32 weights)
    if (g_force_staged || (a_dt == HETA_BF16 && b_dt == HETA_F32) || !gemm_direct_takes(p, a_dt, b_dt)) return false;
    int64_t tiles = 0;
    for (int s = 0; s < p.n_seg; ++s) {
        const int64_t t = ((p.seg[s].M + 127) / 128) * ((p.seg[s].N + 127) / 128);
        tiles = p.batch ? tiles + t : std::max(tiles, t);
    }
    return tiles <= kMergeTiles;
}
static bool has_small(const GemmParams &p)
{
    bool any = p.n_call == 0 && p.form == kFormSmall;
    for (int c = 0; c < p.n_call; ++c) any = any || p.call[c].form == kFormSmall;
    return any;
}
// Whether call `q` (both `merges`) joins the calls in `p`.  fp32 products keep the bits that each has by itself: calls of one
// form do; small ones beside moderate ones, whose kernel then adds their terms in their own order (layers of 0.12 M and 0.15 M
// edges 146 and 204 us without, 134 and 189 with); and moderate beside packed forward products, which add theirs in one order
// (input gradients of the two form the negative product for other rows).  Small beside packed ones stay apart: a choice in the
// packed kernel's loop costs it more than their launch (64 columns over 2.1 M edges 493 us, with it 760).
static bool joins(const GemmParams &p, const GemmParams &q, int32_t transW)
{
    const int more = std::max(p.form, q.form);
    const bool small = more != kFormSmall && (has_small(p) || has_small(q));
    if (more == kFormPacked && (small || (transW && p.form != q.form))) return false;
    if (small && product_steps(p) + product_steps(q) > kUnpackedSteps) return false;
    return std::max(1, p.n_call) < kMaxCalls && p.n_seg + q.n_seg <= kMaxLaunchSeg && p.batch == q.batch && p.out_bf16 == q.out_bf16 &&
           width_class(p) == width_class(q);
}
static void join(GemmParams &p, const GemmParams &q, int32_t transW)
{
    const auto call_of = [](const GemmParams &x, int first) { return GemmCall{first, x.n_seg, 0, 0, 0, 1, 0x7fffffff, x.relu, x.beta, x.row_scale, x.form}; };
    if (p.n_call == 0) p.call[p.n_call++] = call_of(p, 0);
    p.call[p.n_call++] = call_of(q, p.n_seg);
    for (int s = 0; s < q.n_seg; ++s) p.seg[p.n_seg++] = q.seg[s];
    p.form = std::max(p.form, q.form);
    if (p.form == kFormModerate && !transW && !has_small(p) && product_steps(p) > kUnpackedSteps) p.form = kFormPacked;
}

// dM_s = gout . W_s^T for every s: products of one depth whose outputs differ in width
static heta_status bwd_plan(GemmParams &p, int64_t n_rows, int n, const void *const *ins, const int64_t *ld_in, int32_t d_out, const void *const *Ws,
                            heta_dtype w_dt, const int64_t *ld_w, const int32_t *d_in, void *const *dM, heta_dtype dm_dt, const int64_t *ld_dm,
                            const char *who)
{
    p = GemmParams{};
    for (int s = 0; s < n; ++s) {
        if (!ins[s] || !Ws[s] || !dM[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (d_in[s] <= 0 || ld_in[s] < d_out || ld_w[s] < d_out || ld_dm[s] < d_in[s]) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
        if (misaligned(ins[s], 4) || misaligned(Ws[s], dtype_size(w_dt)) || misaligned(dM[s], dtype_size(dm_dt)))
            return fail(HETA_ERR_INVALID_ARG, "%s: pointer not aligned to its element size", who);
        GemmSeg &q = p.seg[s];
        q.A = ins[s];
        q.lda = ld_in[s];
        q.B = Ws[s];   // B[k][n] = W[n][k]: W is [d_in, d_out] row-major, k-contiguous
        q.ldb = ld_w[s];
        q.C = static_cast<float *>(dM[s]); // typed by p.out_bf16 in the kernels' epilogue
        q.ldc = ld_dm[s];
        q.M = n_rows;
        q.N = d_in[s];
        q.K = d_out;
    }
    if (n_rows == 0) return HETA_OK;
    p.n_seg = n;
    p.batch = 1;
    p.k_per_split = int64_t(1) << 40;
    p.n_split = 1;
    p.out_bf16 = dm_dt == HETA_BF16;
    return HETA_OK;
}

// A weight gradient dW_s = beta*dW_s + in_s^T . gout_s over n_rows graph rows, all s of one width d_out.
struct Wgrad {
    int64_t n_rows;
    int n_seg;
    const void *const *ins;
    const int64_t *ld_in;
    const int32_t *d_in;
    const float *const *gouts;
    const int64_t *ld_go;
    int32_t d_out;
    float *const *dW;
    const int64_t *ld_dw;
};
// Which kernel and tiles it takes (wgrad_run): calls of one kind can share a launch.
struct WgradKind {
    bool bf16_direct, f32_terms; // neither: the register-staged kernel
    bool tall, wide_direct;
    int BM, BN, width;
    bool operator==(const WgradKind &o) const
    {
        return bf16_direct == o.bf16_direct && f32_terms == o.f32_terms && tall == o.tall && wide_direct == o.wide_direct && BM == o.BM && BN == o.BN &&
               width == o.width;
    }
};

static heta_status wgrad_check(const Wgrad &c, heta_dtype in_dt, const char *who)
{
    if (!c.ins || !c.gouts || !c.dW || !c.ld_in || !c.ld_go || !c.d_in || !c.ld_dw) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (c.n_seg < 1 || c.n_seg > kMaxSeg) return fail(HETA_ERR_INVALID_ARG, "%s: between 1 and %d inputs", who, kMaxSeg);
    for (int s = 0; s < c.n_seg; ++s) {
        if (!c.gouts[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (c.ld_go[s] < c.d_out) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
        if (misaligned(c.gouts[s], 4)) return fail(HETA_ERR_INVALID_ARG, "%s: gout not 4-byte aligned", who);
    }
    if (!valid_dtype(in_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
    if (c.n_rows < 0 || c.d_out <= 0) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
    for (int s = 0; s < c.n_seg; ++s) {
        if (!c.ins[s] || !c.dW[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
        if (c.d_in[s] <= 0 || c.ld_in[s] < c.d_in[s] || c.ld_dw[s] < c.d_out) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
        if (misaligned(c.ins[s], dtype_size(in_dt)) || misaligned(c.dW[s], 4))
            return fail(HETA_ERR_INVALID_ARG, "%s: pointer not aligned to its element size", who);
    }
    return HETA_OK;
}

static WgradKind wgrad_kind(const Wgrad &c, heta_dtype in_dt)
{
    WgradKind k{};
    bool vec = !g_force_staged;
    int d_in_max = 0;
    for (int s = 0; s < c.n_seg; ++s) {
        vec = vec && vec_ok(c.ins[s], c.ld_in[s], in_dt) && vec_ok(c.gouts[s], c.ld_go[s], HETA_F32);
        d_in_max = std::max(d_in_max, c.d_in[s]);
    }
    // bf16 inputs with 16-byte rows take the all-direct kernel: 128 x 128 tiles, three workgroups per CU (wider and
    // taller tiles below)
    k.bf16_direct = in_dt == HETA_BF16 && vec;
    // fp32 inputs on the direct pipeline (six bf16 terms per product): 128 x 128 tiles, three workgroups per CU
    k.f32_terms = in_dt == HETA_F32 && vec && !g_f32_native;
    k.tall = k.bf16_direct && d_in_max > 128;                     // 320 x 128 tiles, one 512-thread workgroup per CU
    k.wide_direct = k.bf16_direct && !k.tall && c.d_out > 128;    // 128 x 256 tiles, two 512-thread workgroups per CU
    const bool tall_wide = k.tall && c.d_out > 128;               // 320 x 256 or 256 x 256 tiles, one workgroup per CU
    k.BN = (c.d_out > 128 && (!k.bf16_direct || k.wide_direct || tall_wide) && !k.f32_terms) ? 256 : 128;
    k.BM = k.tall ? 320 : BM;
    if (tall_wide) { // the tile height the launch will choose (wgrad_tile_rows): the one that pads the input columns less
        int64_t pad320 = 0, pad256 = 0;
        for (int s = 0; s < c.n_seg; ++s) {
            pad320 += (static_cast<int64_t>(c.d_in[s]) + 319) / 320 * 320;
            pad256 += (static_cast<int64_t>(c.d_in[s]) + 255) / 256 * 256;
        }
        if (pad256 < pad320) k.BM = 256;
    }
    k.width = c.d_out <= 64 ? 0 : c.d_out <= 128 ? 1 : 2;
    return k;
}

// Split the graph rows so that a call's workgroups fill the chip exactly once and never spill into a
// second, nearly empty round.  Workgroups are dealt round-robin to the 8 XCDs (32 CUs each) and
// the kernel keeps the `tiles` output tiles of one split on one XCD, so a split costs `tiles`
// workgroup slots of its XCD: 2 resident 512-thread workgroups per CU (3 or 4 of 256 threads).
// Each split keeps at least 4 k-tiles (a few thousand graph rows still spread over the chip: a
// workgroup's k-tiles are latency-bound when few workgroups run).
struct WgradSplit {
    int64_t n, k_tiles_each, k_tile; // splits, k-tiles of each, graph rows per k-tile
};
static WgradSplit wgrad_split(const Wgrad &c, const WgradKind &kind, heta_dtype in_dt)
{
    const int64_t BK = in_dt == HETA_F32 ? 32 : 64, k_tiles = (c.n_rows + BK - 1) / BK, nt = (c.d_out + kind.BN - 1) / kind.BN;
    const int64_t slots_per_xcd =
        32 * (kind.tall ? 1 : kind.wide_direct ? 2 : (kind.bf16_direct || kind.f32_terms) ? 3 : (c.d_out > 128 ? 2 : (in_dt == HETA_F32 ? 3 : 4)));
    int64_t tiles = 0, mt_max = 1;
    for (int s = 0; s < c.n_seg; ++s) {
        const int64_t mt = (static_cast<int64_t>(c.d_in[s]) + kind.BM - 1) / kind.BM;
        tiles += mt * nt;
        mt_max = std::max(mt_max, mt);
    }
    // a split's workgroups are (largest segment's row tiles) x (column tiles) x (segments), all on one XCD
    const int64_t slots_per_split = std::max<int64_t>(tiles, mt_max * nt * c.n_seg);
    const int64_t splits_per_xcd = std::max<int64_t>(1, slots_per_xcd / std::max<int64_t>(1, slots_per_split));
    const int64_t n = std::max<int64_t>(1, std::min<int64_t>((k_tiles + 3) / 4, 8 * splits_per_xcd));
    const int64_t each = std::max<int64_t>(1, (k_tiles + n - 1) / n);
    return WgradSplit{std::max<int64_t>(1, (k_tiles + each - 1) / each), each, BK};
}

// appends the products of a call to a plan
static void wgrad_segs(GemmParams &p, const Wgrad &w)
{
    for (int s = 0; s < w.n_seg; ++s) {
        GemmSeg &q = p.seg[p.n_seg++];
        q.A = w.ins[s];    // A[m = column of `in`][k = graph row] : r-contiguous
        q.lda = w.ld_in[s];
        q.B = w.gouts[s];  // B[k = graph row][n] : r-contiguous
        q.ldb = w.ld_go[s];
        q.M = w.d_in[s];
        q.N = w.d_out;
        q.K = w.n_rows;
        q.ldc = w.d_out;
    }
}

// The listed calls (checked; of one kind if there are several) in one launch, their partial sums in another.  Calls that
// share a launch keep their splits: splits of one length that fill the chip together would be longer, and longer sums are
// further from 64 bits (9.4e-7 -> 1.3e-6, layer of 21 M edges).
static heta_status wgrad_run(heta_graph *g, const Wgrad *calls, int n_calls, heta_dtype in_dt, int gout_two_terms, float beta, hipStream_t st)
{
    const WgradKind kind = wgrad_kind(calls[0], in_dt);
    GemmParams p{};
    int64_t n_split[kMaxCalls], split_max = 1, ws_elems = 0;
    int chains[kMaxCalls];
    for (int c = 0; c < n_calls; ++c) {
        const Wgrad &w = calls[c];
        int64_t elems = 0;
        const int first = p.n_seg;
        wgrad_segs(p, w);
        for (int s = first; s < p.n_seg; ++s) elems += p.seg[s].M * p.seg[s].N;
        const WgradSplit split = wgrad_split(w, kind, in_dt);
        n_split[c] = split.n;
        chains[c] = split_chains(split.n, elems);
        ws_elems += n_split[c] * elems;
        split_max = std::max(split_max, n_split[c]);
        p.k_per_split = split.k_tiles_each * split.k_tile;
        if (n_calls > 1)
            p.call[p.n_call++] = GemmCall{first, w.n_seg, 0, 0, 0, static_cast<int32_t>(n_split[c]),
                                          static_cast<int32_t>(std::min<int64_t>(p.k_per_split, 0x7fffffff)), 0, 0.f, nullptr, kFormNone};
    }
    heta_status e = ensure_workspace(g, static_cast<size_t>(ws_elems) * sizeof(float));
    if (e != HETA_OK) return e;
    SplitSegs sums{};
    int64_t blocks = 0;
    double bytes = 0;
    const int threads = *std::max_element(chains, chains + n_calls) == 16 ? 1024 : 256;
    float *ws = static_cast<float *>(g->d_ws);
    for (int c = 0, at = 0; c < n_calls; ++c)
        for (int s = 0; s < calls[c].n_seg; ++s, ++at) {
            const int64_t total = static_cast<int64_t>(calls[c].d_in[s]) * calls[c].d_out;
            p.seg[at].C = ws;
            ws += n_split[c] * total;
            sums.part[at] = p.seg[at].C;
            sums.out[at] = calls[c].dW[s];
            sums.M[at] = calls[c].d_in[s];
            sums.ldo[at] = calls[c].ld_dw[s];
            sums.N[at] = calls[c].d_out;
            sums.n_split[at] = static_cast<int32_t>(n_split[c]);
            sums.chains[at] = chains[c];
            const int64_t per_block = threads / chains[c];
            blocks = std::max(blocks, (total + per_block - 1) / per_block);
            bytes += (n_split[c] + 1.0) * total * 4.0;
        }
    sums.beta = beta;
    p.batch = 1;
    p.n_split = static_cast<int>(split_max);
    p.partial = 1;
    p.split_b = (gout_two_terms && in_dt == HETA_BF16) ? 1 : 0;
    if ((e = dispatch_gemm<true, true>(p, in_dt, HETA_F32, st, in_dt == HETA_F32 ? 32 : 64)) != HETA_OK) return e;
    ProfScope prof("splitk_reduce_kernel", st, bytes, 0);
    launch_pieces(blocks, threads, [&](unsigned first, unsigned count) {
        sums.first = first;
        const dim3 grid(count, (unsigned)p.n_seg);
        if (threads == 1024) hipLaunchKernelGGL(splitk_reduce_kernel<1024>, grid, dim3(1024), 0, st, sums);
        else hipLaunchKernelGGL(splitk_reduce_kernel<256>, grid, dim3(256), 0, st, sums);
    });
    HETA_LAUNCH_CHECK("splitk_reduce_kernel");
    return HETA_OK;
}

// one call; gouts null: every segment takes gout / ld_go
static heta_status wgrad_impl(heta_graph *g, int64_t n_rows, int n_seg, const void *const *ins, heta_dtype in_dt, const int64_t *ld_in,
                              const int32_t *d_in, const float *gout, int64_t ld_go, int32_t d_out, float *const *dW, const int64_t *ld_dw, float beta,
                              hipStream_t st, const char *who, int gout_two_terms = 0, const float *const *gouts = nullptr,
                              const int64_t *ld_gos = nullptr)
{
    if (!g) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    const float *same[kMaxSeg];
    int64_t ld_same[kMaxSeg];
    if (!gouts) {
        std::fill(same, same + kMaxSeg, gout);
        std::fill(ld_same, ld_same + kMaxSeg, ld_go);
        gouts = same;
        ld_gos = ld_same;
    }
    const Wgrad call{n_rows, n_seg, ins, ld_in, d_in, gouts, ld_gos, d_out, dW, ld_dw};
    heta_status e = wgrad_check(call, in_dt, who);
    return e == HETA_OK ? wgrad_run(g, &call, 1, in_dt, gout_two_terms, beta, st) : e;
}

static heta_status project_multi_impl(heta_graph *g, int32_t n, const int32_t *first, const int64_t *n_rows, int32_t sum, const void *const *ins,
                                      heta_dtype in_dt, const int64_t *ld_in, const int32_t *depth, const void *const *Ws, heta_dtype w_dt,
                                      const int64_t *ld_w, const int32_t *width, int32_t transW, void *const *outs, heta_dtype out_dt,
                                      const int64_t *ld_out, const heta_act *acts, const float *betas, hipStream_t st)
{
    const char *who = "heta_project_multi";
    if (!g || n < 0 || (n > 0 && (!first || !n_rows || !ins || !ld_in || !depth || !Ws || !ld_w || !width || !outs || !ld_out)))
        return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (!valid_dtype(in_dt) || !valid_dtype(w_dt) || !valid_dtype(out_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
    if (n > 0 && first[0] != 0) return fail(HETA_ERR_INVALID_ARG, "%s: first[0] must be 0", who);
    std::vector<GemmParams> plans(n);
    for (int32_t i = 0; i < n; ++i) {
        const int32_t f = first[i], m = first[i + 1] - f;
        if (m < 1 || m > kMaxSeg) return fail(HETA_ERR_INVALID_ARG, "%s: between 1 and %d products per item", who, kMaxSeg);
        if (acts && acts[i] != HETA_ACT_NONE && acts[i] != HETA_ACT_RELU) return fail(HETA_ERR_INVALID_ARG, "%s: bad act", who);
        if (!sum && ((acts && acts[i] != HETA_ACT_NONE) || (betas && betas[i] != 0.f)))
            return fail(HETA_ERR_UNSUPPORTED, "%s: activation and beta belong to sums", who);
        for (int32_t s = f + 1; s < f + m; ++s)
            if (sum ? width[s] != width[f] : depth[s] != depth[f])
                return fail(HETA_ERR_SHAPE, "%s: a sum's products share their width, independent ones their depth", who);
        heta_status e = sum ? project_plan(plans[i], n_rows[i], m, ins + f, in_dt, ld_in + f, depth + f, Ws + f, w_dt, ld_w + f, width[f], transW, nullptr,
                                           acts && acts[i] == HETA_ACT_RELU, outs[i], ld_out[i], betas ? betas[i] : 0.f, who, out_dt, nullptr, nullptr)
                        : HETA_OK;
        if (!sum) { // independent products: one depth, any widths
            if (n_rows[i] < 0 || depth[f] <= 0) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
            GemmParams &p = plans[i];
            p = GemmParams{};
            for (int32_t s = f; s < f + m; ++s) {
                if (!ins[s] || !Ws[s] || !outs[s]) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
                if (width[s] <= 0 || ld_in[s] < depth[s] || ld_w[s] < (transW ? depth[s] : width[s]) || ld_out[s] < width[s])
                    return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
                if (misaligned(ins[s], dtype_size(in_dt)) || misaligned(Ws[s], dtype_size(w_dt)) || misaligned(outs[s], dtype_size(out_dt)))
                    return fail(HETA_ERR_INVALID_ARG, "%s: pointer not aligned to its element size", who);
                p.seg[s - f] = GemmSeg{ins[s], ld_in[s], Ws[s], ld_w[s], static_cast<float *>(outs[s]), ld_out[s], n_rows[i], width[s], depth[s], nullptr, 0, 0};
            }
            if (n_rows[i] > 0) {
                p.n_seg = m;
                p.batch = 1;
                p.k_per_split = int64_t(1) << 40;
                p.n_split = 1;
                p.out_bf16 = out_dt == HETA_BF16;
            }
        }
        if (e != HETA_OK) return e;
    }
    // the items run side by side, and not in the order given
    std::vector<ItemRange> written, read;
    for (int32_t i = 0; i < n; ++i)
        for (int s = 0; s < plans[i].n_seg; ++s) {
            const GemmSeg &a = plans[i].seg[s];
            if (plans[i].batch || s == 0) written.emplace_back(i, RowRange(a.C, a.M, a.ldc, a.N, dtype_size(out_dt)));
            if (n == 1) continue;
            read.emplace_back(i, RowRange(a.A, a.M, a.lda, a.K, dtype_size(in_dt)));
            read.emplace_back(i, RowRange(a.B, transW ? a.N : a.K, a.ldb, transW ? a.K : a.N, dtype_size(w_dt)));
        }
    if (items_collide(written, read)) return fail(HETA_ERR_INVALID_ARG, "%s: an output overlaps another one or what another item reads", who);
    if (in_dt == HETA_F32 && w_dt == HETA_F32)
        for (GemmParams &p : plans) p.form = f32_product_form(p);
    for (int32_t i = 0; i < n; ++i) {
        GemmParams &p = plans[i];
        if (p.n_seg == 0) continue; // no rows, or joined already
        if (merges(p, in_dt, w_dt))
            for (int32_t j = i + 1; j < n; ++j)
                if (plans[j].n_seg > 0 && merges(plans[j], in_dt, w_dt) && joins(p, plans[j], transW)) {
                    join(p, plans[j], transW);
                    plans[j].n_seg = 0;
                }
        heta_status e = project_run(p, in_dt, w_dt, transW, g, st, true);
        if (e != HETA_OK) return e;
    }
    return HETA_OK;
}

constexpr int64_t kMergeKTiles = 32;
static heta_status wgrad_multi_impl(heta_graph *g, int32_t n, const int32_t *first, const int64_t *n_rows, const void *const *ins, heta_dtype in_dt,
                                    const int64_t *ld_in, const int32_t *d_in, const float *const *gouts, const int64_t *ld_go, const int32_t *d_out,
                                    float *const *dW, const int64_t *ld_dw, int32_t gout_two_terms, hipStream_t st)
{
    const char *who = "heta_project_wgrad_multi";
    if (!g || n < 0 || (n > 0 && (!first || !n_rows || !ins || !ld_in || !d_in || !gouts || !ld_go || !d_out || !dW || !ld_dw)))
        return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n > 0 && first[0] != 0) return fail(HETA_ERR_INVALID_ARG, "%s: first[0] must be 0", who);
    std::vector<Wgrad> calls;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t f = first[i];
        calls.push_back(Wgrad{n_rows[i], first[i + 1] - f, ins + f, ld_in + f, d_in + f, gouts + f, ld_go + f, d_out[i], dW + f, ld_dw + f});
        heta_status e = wgrad_check(calls.back(), in_dt, who);
        if (e != HETA_OK) return e;
    }
    std::vector<ItemRange> written, read;
    for (int32_t i = 0; i < n; ++i)
        for (int32_t s = first[i]; s < first[i + 1]; ++s) {
            written.emplace_back(i, RowRange(dW[s], d_in[s], ld_dw[s], d_out[i], 4));
            if (n == 1) continue;
            read.emplace_back(i, RowRange(ins[s], n_rows[i], ld_in[s], d_in[s], dtype_size(in_dt)));
            read.emplace_back(i, RowRange(gouts[s], n_rows[i], ld_go[s], d_out[i], 4));
        }
    if (items_collide(written, read)) return fail(HETA_ERR_INVALID_ARG, "%s: an output overlaps another one or what another item reads", who);
    // Calls of few k-tiles per split share a launch; the others fill the chip for long enough by themselves (kMergeKTiles: five
    // calls of 10^4 to 10^6 rows, 128 x 256, 1.34 ms together and 1.13 one by one; four of 900 to 110,000 rows, 128 x 64, 76 us
    // together and 112).  Calls without rows leave zeros and go alone.
    const auto shares = [&](const Wgrad &c, const WgradKind &kind) {
        if (!(kind.bf16_direct || kind.f32_terms) || c.n_rows == 0) return false;
        const WgradSplit split = wgrad_split(c, kind, in_dt);
        GemmParams p{};
        wgrad_segs(p, c);
        p.n_split = static_cast<int>(split.n);
        p.k_per_split = split.k_tiles_each * split.k_tile;
        return split.k_tiles_each <= kMergeKTiles && gemm_direct_takes(p, in_dt, HETA_F32);
    };
    std::vector<char> done(n, 0);
    for (int32_t i = 0; i < n; ++i) {
        if (done[i]) continue;
        const WgradKind kind = wgrad_kind(calls[i], in_dt);
        Wgrad part[kMaxCalls] = {calls[i]};
        int count = 1, segs = calls[i].n_seg;
        if (shares(calls[i], kind))
            for (int32_t j = i + 1; j < n && count < kMaxCalls; ++j)
                if (!done[j] && segs + calls[j].n_seg <= kMaxLaunchSeg && wgrad_kind(calls[j], in_dt) == kind && shares(calls[j], kind)) {
                    part[count++] = calls[j];
                    segs += calls[j].n_seg;
                    done[j] = 1;
                }
        heta_status e = wgrad_run(g, part, count, in_dt, gout_two_terms, 0.f, st);
        if (e != HETA_OK) return e;
    }
    return HETA_OK;
}

static heta_status check_type(const heta_graph *g, int32_t t, const char *who)
{
    if (!g) return fail(HETA_ERR_INVALID_ARG, "%s: graph is NULL", who);
    if (t < 0 || t >= (int32_t)g->ntypes.size()) return fail(HETA_ERR_INVALID_ARG, "%s: node type %d out of range", who, t);
    return HETA_OK;
}

} // namespace heta

using namespace heta;

extern "C" {

heta_status heta_projection_f32_native(int32_t on)
{
    g_f32_native = on != 0;
    return HETA_OK;
}

heta_status heta_projection_force_staged(int32_t on)
{
    g_force_staged = on != 0;
    return HETA_OK;
}

heta_status heta_project(int64_t n_rows, const void *in, heta_dtype in_dt, int64_t ld_in, int32_t d_in,
                         const void *W, heta_dtype w_dt, int64_t ld_w, int32_t d_out, int32_t transW,
                         const float *row_scale, void *out, heta_dtype out_dt, int64_t ld_out, float beta,
                         void *hip_stream)
{
    return project_impl(n_rows, 1, &in, in_dt, &ld_in, &d_in, &W, w_dt, &ld_w, d_out, transW, row_scale, 0, out, ld_out,
                        beta, as_stream(hip_stream), "heta_project", nullptr, out_dt);
}

heta_status heta_rel_project(heta_graph *g, int32_t rel, const void *in, heta_dtype in_dt,
                             int64_t ld_in, int32_t d_in, const void *W, heta_dtype w_dt, int64_t ld_w,
                             int32_t d_out, int32_t transW, const float *row_scale, void *out,
                             heta_dtype out_dt, int64_t ld_out, float beta, void *hip_stream)
{
    if (!g) return fail(HETA_ERR_INVALID_ARG, "heta_rel_project: graph is NULL");
    if (rel < 0 || rel >= (int32_t)g->rels.size())
        return fail(HETA_ERR_INVALID_ARG, "heta_rel_project: relation %d out of range", rel);
    return project_impl(g->rels[rel].n_dst, 1, &in, in_dt, &ld_in, &d_in, &W, w_dt, &ld_w, d_out, transW, row_scale, 0,
                        out, ld_out, beta, as_stream(hip_stream), "heta_rel_project", g, out_dt);
}

heta_status heta_rel_project_wgrad(heta_graph *g, int32_t rel, const void *in, heta_dtype in_dt,
                                   int64_t ld_in, int32_t d_in, const float *gout, int64_t ld_go,
                                   int32_t d_out, float *dW, int64_t ld_dw, float beta, void *hip_stream)
{
    if (!g) return fail(HETA_ERR_INVALID_ARG, "heta_rel_project_wgrad: null argument");
    if (rel < 0 || rel >= (int32_t)g->rels.size())
        return fail(HETA_ERR_INVALID_ARG, "heta_rel_project_wgrad: relation %d out of range", rel);
    return wgrad_impl(g, g->rels[rel].n_dst, 1, &in, in_dt, &ld_in, &d_in, gout, ld_go, d_out, &dW, &ld_dw, beta,
                      as_stream(hip_stream), "heta_rel_project_wgrad");
}

heta_status heta_project_batch(heta_graph *g, int64_t n_rows, int32_t n, const void *const *ins, heta_dtype in_dt, const int64_t *ld_in,
                               const int32_t *d_in, const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w, int32_t d_out,
                               int32_t transW, void *const *outs, heta_dtype out_dt, const int64_t *ld_out, void *hip_stream)
{
    if (!outs || !ld_out) return fail(HETA_ERR_INVALID_ARG, "heta_project_batch: null argument");
    return project_impl(n_rows, n, ins, in_dt, ld_in, d_in, Ws, w_dt, ld_w, d_out, transW, nullptr, 0, nullptr, 0, 0.f,
                        as_stream(hip_stream), "heta_project_batch", g, out_dt, outs, ld_out);
}

heta_status heta_project_sum(heta_graph *g, int64_t n_rows, int32_t n, const void *const *ins, heta_dtype in_dt, const int64_t *ld_in,
                             const int32_t *d_in, const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w, int32_t d_out,
                             int32_t transW, float *out, int64_t ld_out, float beta, void *hip_stream)
{
    return project_impl(n_rows, n, ins, in_dt, ld_in, d_in, Ws, w_dt, ld_w, d_out, transW, nullptr, 0, out, ld_out, beta,
                        as_stream(hip_stream), "heta_project_sum", g);
}

heta_status heta_project_wgrad_batch(heta_graph *g, int64_t n_rows, int32_t n, const void *const *ins, heta_dtype in_dt,
                                     const int64_t *ld_in, const int32_t *d_in, const float *const *gouts,
                                     const int64_t *ld_go, int32_t d_out, float *const *dW, const int64_t *ld_dw, float beta,
                                     int32_t gout_two_terms, void *hip_stream)
{
    if (!g || !gouts || !ld_go) return fail(HETA_ERR_INVALID_ARG, "heta_project_wgrad_batch: null argument");
    if (n_rows < 0) return fail(HETA_ERR_SHAPE, "heta_project_wgrad_batch: negative row count");
    return wgrad_impl(g, n_rows, n, ins, in_dt, ld_in, d_in, nullptr, 0, d_out, dW, ld_dw, beta, as_stream(hip_stream),
                      "heta_project_wgrad_batch", gout_two_terms, gouts, ld_go);
}

heta_status heta_cross_rel_project(heta_graph *g, int32_t dst_type, int32_t n, const void *const *ins,
                                   heta_dtype in_dt, const int64_t *ld_in, const int32_t *d_in,
                                   const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w, int32_t d_out,
                                   heta_act act, float *out, int64_t ld_out, float beta, void *hip_stream)
{
    heta_status e = check_type(g, dst_type, "heta_cross_rel_project");
    if (e != HETA_OK) return e;
    if (act != HETA_ACT_NONE && act != HETA_ACT_RELU) return fail(HETA_ERR_INVALID_ARG, "heta_cross_rel_project: bad act");
    return project_impl(g->ntypes[dst_type].num_nodes, n, ins, in_dt, ld_in, d_in, Ws, w_dt, ld_w, d_out, 0, nullptr,
                        act == HETA_ACT_RELU, out, ld_out, beta, as_stream(hip_stream), "heta_cross_rel_project", g);
}

heta_status heta_cross_rel_project_bwd(const heta_graph *g, int32_t dst_type, int32_t n, const float *gout,
                                       int64_t ld_go, int32_t d_out, const void *const *Ws, heta_dtype w_dt,
                                       const int64_t *ld_w, const int32_t *d_in, void *const *dM,
                                       heta_dtype dm_dt, const int64_t *ld_dm, void *hip_stream)
{
    const char *who = "heta_cross_rel_project_bwd";
    heta_status e = check_type(g, dst_type, who);
    if (e != HETA_OK) return e;
    if (!gout || !Ws || !ld_w || !d_in || !dM || !ld_dm) return fail(HETA_ERR_INVALID_ARG, "%s: null argument", who);
    if (n < 1 || n > kMaxSeg) return fail(HETA_ERR_INVALID_ARG, "%s: between 1 and %d relations", who, kMaxSeg);
    if (!valid_dtype(w_dt) || !valid_dtype(dm_dt)) return fail(HETA_ERR_INVALID_ARG, "%s: bad dtype", who);
    if (d_out <= 0 || ld_go < d_out) return fail(HETA_ERR_SHAPE, "%s: bad sizes", who);
    if (misaligned(gout, 4)) return fail(HETA_ERR_INVALID_ARG, "%s: gout not 4-byte aligned", who);
    const void *ins[kMaxSeg];
    int64_t ld_in[kMaxSeg];
    GemmParams p;
    std::fill(ins, ins + n, gout);
    std::fill(ld_in, ld_in + n, ld_go);
    if ((e = bwd_plan(p, g->ntypes[dst_type].num_nodes, n, ins, ld_in, d_out, Ws, w_dt, ld_w, d_in, dM, dm_dt, ld_dm, who)) != HETA_OK) return e;
    // the handle's packing buffer is scratch memory, not part of the graph it describes
    return project_run(p, HETA_F32, w_dt, 1, const_cast<heta_graph *>(g), as_stream(hip_stream), false);
}

heta_status heta_cross_rel_project_wgrad(heta_graph *g, int32_t dst_type, int32_t n, const void *const *ins,
                                         heta_dtype in_dt, const int64_t *ld_in, const int32_t *d_in,
                                         const float *gout, int64_t ld_go, int32_t d_out, float *const *dW,
                                         const int64_t *ld_dw, float beta, int32_t gout_two_terms, void *hip_stream)
{
    heta_status e = check_type(g, dst_type, "heta_cross_rel_project_wgrad");
    if (e != HETA_OK) return e;
    return wgrad_impl(g, g->ntypes[dst_type].num_nodes, n, ins, in_dt, ld_in, d_in, gout, ld_go, d_out, dW, ld_dw, beta,
                      as_stream(hip_stream), "heta_cross_rel_project_wgrad", gout_two_terms);
}

// No exception crosses the boundary: host containers may throw std::bad_alloc.
heta_status heta_project_multi(heta_graph *g, int32_t n, const int32_t *first, const int64_t *n_rows, int32_t sum, const void *const *ins, heta_dtype in_dt,
                               const int64_t *ld_in, const int32_t *depth, const void *const *Ws, heta_dtype w_dt, const int64_t *ld_w,
                               const int32_t *width, int32_t transW, void *const *outs, heta_dtype out_dt, const int64_t *ld_out, const heta_act *acts,
                               const float *betas, void *hip_stream)
{
    try {
        return project_multi_impl(g, n, first, n_rows, sum, ins, in_dt, ld_in, depth, Ws, w_dt, ld_w, width, transW, outs, out_dt, ld_out, acts, betas,
                                  as_stream(hip_stream));
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_project_multi: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_project_multi: unexpected exception");
    }
}

heta_status heta_project_wgrad_multi(heta_graph *g, int32_t n, const int32_t *first, const int64_t *n_rows, const void *const *ins, heta_dtype in_dt,
                                     const int64_t *ld_in, const int32_t *d_in, const float *const *gouts, const int64_t *ld_go, const int32_t *d_out,
                                     float *const *dW, const int64_t *ld_dw, int32_t gout_two_terms, void *hip_stream)
{
    try {
        return wgrad_multi_impl(g, n, first, n_rows, ins, in_dt, ld_in, d_in, gouts, ld_go, d_out, dW, ld_dw, gout_two_terms, as_stream(hip_stream));
    } catch (const std::bad_alloc &) {
        return fail(HETA_ERR_OOM, "heta_project_wgrad_multi: host allocation failed");
    } catch (...) {
        return fail(HETA_ERR_DEVICE, "heta_project_wgrad_multi: unexpected exception");
    }
}

} // extern "C"
