// Batch-norm statistics over the active blocks only (Sec. 3.3 of arXiv 1801.02108: the layers of a residual unit
// run in sparse mode, and normalising across the non-sparse elements alone keeps invalid data out of the
// statistics): per channel, the mean and the (biased) variance of x over the pixels of the listed blocks that lie
// inside the image.
//
// Two kernels, no atomics, fixed summation order:
//   bn_partial   one workgroup per (row, slab of 128 bytes of channels per pixel); a row is every rows-th piece of 128
//                pixels.  Eight lanes read one pixel's 128-byte strip; a thread accumulates, in fp32, the sum and the sum
//                of squares of its channels, taken relative to the first active pixel that it holds (which keeps the
//                squares small when the mean is large against the spread; pixels outside the active blocks are never
//                looked at).  The 32 pixel groups' (count, mean, sum of squared deviations) are merged through LDS and
//                go to the workspace.
//   bn_combine   one workgroup per four channels merges the rows' triples with the pairwise update of Chan, Golub and
//                LeVeque (mean += delta * n_b / n; M2 += M2_b + delta^2 * n_a * n_b / n): every thread a strided
//                subset in order, then a fixed tree over the threads.
// Bound by HBM (the active blocks read once) and, at these sizes, by the launches and the round trips of a workgroup.
// bf16, before (a row per block, one workgroup per channel) -> now, partial + combine: 800 x 704 x 64, 880 blocks of 16 x 16
// (28.8 MB): 8.1 + 5.2 -> 8.5 + 4.5 us; 844 x 494 x 64, 3746 blocks of 8 x 8 (30.7 MB): 10.8 + 13.0 -> 9.6 + 4.9 us.
#include "bn_common.h"

namespace sbnet {

// The triples (n[g], mean[g * stride], m2[g * stride]), g < G, as one: the mean relative to the first non-empty one's, then the
// squares about it.  G is small and the loops unrolled: no division but one.
template <int G>
__device__ __forceinline__ void bn_merge_of(const int *n, const float *mean, const float *m2, int stride, int *nt, float *mt, float *m2t) {
    int c[G], total = 0;
    float m[G], s[G], ref = 0.f, a = 0.f, q = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {                                 // (all reads in flight; an empty triple is three zeros)
        c[g] = n[g];
        m[g] = mean[g * stride];
        s[g] = m2[g * stride];
    }
#pragma unroll
    for (int g = G - 1; g >= 0; --g) {
        total += c[g];
        ref = c[g] > 0 ? m[g] : ref;
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float d = m[g] - ref, nd = (float)c[g] * d;
        a += nd;
        q += fmaf(nd, d, s[g]);
    }
    const float md = total > 0 ? a / (float)total : 0.f;
    *nt = total;
    *mt = ref + md;
    *m2t = fmaxf(q - a * md, 0.f);
}

// workspace layout: float part[rows][C][2] (mean, M2), at cnt float cnt[rows]; rows = gridDim.x / slabs <= cap
template <int DT>
__global__ __launch_bounds__(kBnThreads) void bn_partial(const uint4 *__restrict__ x, const int32_t *__restrict__ indices,
                                                         const int32_t *__restrict__ count, float *__restrict__ part,
                                                         float *__restrict__ cnt, int pieces, FastDiv div_pieces, BnParams p) {
    constexpr int EPV = BnElem<DT>::EPV, NCH = 8 * EPV, LD = NCH + 1;
    __shared__ float means[32][LD], squares[32][LD];
    __shared__ int ns[32], nw[4];
    const int pg = threadIdx.x >> 3, k = threadIdx.x & 7;         // pixel group, vector of the slab
    const uint32_t row = fdiv(blockIdx.x, p.div_slabs), rows = fdiv(gridDim.x, p.div_slabs);
    const int slab = (int)(blockIdx.x - row * p.slabs);
    BnWalk it(row, rows, (uint32_t)pieces, div_pieces);
    BnBlock blk = bn_block(indices, it.unit, p.cap);
    const uint32_t nact = (uint32_t)max(min(*count, p.cap), 0);
    if (it.unit >= nact) return;
    float ref[EPV], s1[EPV], s2[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) ref[e] = s1[e] = s2[e] = 0.f;
    int npx = 0;
    while (it.unit < nact) {
        const BnPlace w = bn_place<EPV>(blk, slab, k, p);
        const int q0 = (int)it.piece * kBnPiece + pg;
        it.advance();
        blk = bn_block(indices, it.unit, p.cap);                  // the next item's
        long long at[4];
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {                             // four independent loads in flight
            at[u] = bn_pixel(w, q0 + 32 * u, p);
            if (at[u] >= 0) v[u] = x[at[u]];
        }
        if (npx == 0) {                                           // the thread's first pixel is its reference
            uint4 first = make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int u = 3; u >= 0; --u)
                if (at[u] >= 0) first = v[u];
            BnElem<DT>::unpack(first, ref);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0) {
                ++npx;
                float f[EPV];
                BnElem<DT>::unpack(v[u], f);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float d = f[e] - ref[e];
                    s1[e] += d;
                    s2[e] = fmaf(d, d, s2[e]);
                }
            }
    }
    // the 32 pixel groups by eights, then the four results (in place of their first groups')
    const float share = npx > 0 ? 1.f / (float)npx : 0.f;
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        const float md = s1[e] * share;
        means[pg][k * EPV + e] = ref[e] + md;
        squares[pg][k * EPV + e] = s2[e] - s1[e] * md;
    }
    if (k == 0) ns[pg] = npx;
    __syncthreads();
    const int ch = threadIdx.x % NCH, quarter = threadIdx.x / NCH;
    int n = 0;
    float m = 0.f, m2 = 0.f;
    if (quarter < 4) {
        bn_merge_of<8>(&ns[quarter * 8], &means[quarter * 8][ch], &squares[quarter * 8][ch], LD, &n, &m, &m2);
        means[quarter * 8][ch] = m;
        squares[quarter * 8][ch] = m2;
        if (ch == 0) nw[quarter] = n;
    }
    __syncthreads();
    const int c = slab * p.cs + threadIdx.x;
    if (threadIdx.x >= NCH || c >= p.C) return;
    bn_merge_of<4>(nw, &means[0][ch], &squares[0][ch], 8 * LD, &n, &m, &m2);
    part[((size_t)row * p.C + c) * 2] = m;
    part[((size_t)row * p.C + c) * 2 + 1] = m2;
    if (slab == 0 && threadIdx.x == 0) cnt[row] = (float)n;
}

// merge of two (count, mean, M2) triples; an empty side leaves the other unchanged
__device__ __forceinline__ void bn_merge(float &n, float &m, float &m2, float nb, float mb, float m2b) {
    if (nb <= 0.f) return;
    const float tot = n + nb, delta = mb - m, share = nb / tot;
    m += delta * share;
    m2 += m2b + delta * delta * (n * share);
    n = tot;
}

// Four channels per workgroup: thread (t, channel) merges rows t, t + 256, ... in that order, four in flight, then the 256
// partial triples are merged pairwise in a fixed tree.
__global__ __launch_bounds__(1024) void bn_combine(const float *__restrict__ part, const float *__restrict__ cnt,
                                                   const int32_t *__restrict__ count, int cap, int C, int max_rows, int pieces,
                                                   float *__restrict__ mean, float *__restrict__ var) {
    __shared__ float sn[64], sm[64], sq[64];
    const int ch = threadIdx.x & 3, row = threadIdx.x >> 2, c = blockIdx.x * 4 + ch;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rows = (int)min((long long)min(*count, cap) * pieces, (long long)max_rows);
    float n = 0.f, m = 0.f, m2 = 0.f;
    for (int b0 = row; b0 < rows; b0 += 256 * 4) {
        f32x2_a4 v[4];
        float k[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = min(b0 + 256 * u, rows - 1);
            v[u] = *(const f32x2_a4 *)(part + ((size_t)b * C + min(c, C - 1)) * 2);
            k[u] = cnt[b];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (b0 + 256 * u < rows) bn_merge(n, m, m2, k[u], v[u][0], v[u][1]);
    }
    // a fixed tree: the 16 rows of a wave, then the 16 waves (a wave holds four channels: lane = 4 row + channel)
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int off = 32; off >= 4; off >>= 1) bn_merge(n, m, m2, __shfl_down(n, off), __shfl_down(m, off), __shfl_down(m2, off));
    };
    fold();
    if (lane < 4) { sn[wave * 4 + lane] = n; sm[wave * 4 + lane] = m; sq[wave * 4 + lane] = m2; }
    __syncthreads();
    if (wave > 0) return;
    n = sn[lane]; m = sm[lane]; m2 = sq[lane];
    fold();
    if (lane < 4 && c < C) {
        mean[c] = m;
        var[c] = n > 0.f ? m2 / n : 0.f;
    }
}

}  // namespace sbnet

using namespace sbnet;

extern "C" size_t sbnet_bn_stats_workspace_bytes(int cap, int C) {
    if (cap <= 0 || C <= 0) return 0;
    return ((size_t)cap * C * 2 + (size_t)cap) * sizeof(float);
}

extern "C" sbnet_status sbnet_sparse_bn_stats(const void *x, sbnet_dtype dtype, int N, int H, int W, int C,
                                              const int32_t *indices, const int32_t *count, int cap,
                                              const sbnet_geom *g, float *mean, float *var, void *workspace,
                                              size_t workspace_bytes, void *stream) {
    const char *who = "sbnet_sparse_bn_stats";
    if (!x || !indices || !count || !mean || !var) return fail(SBNET_EINVAL, "%s: null pointer", who);
    BnParams p;
    sbnet_status st = bn_fill_params(who, dtype, N, H, W, C, cap, g, &p);
    if (st != SBNET_OK) return st;
    if ((uintptr_t)x & 15) return fail(SBNET_EINVAL, "%s: x must be 16-byte aligned", who);
    if (cap > 0 && (!workspace || ((uintptr_t)workspace & 3) || workspace_bytes < sbnet_bn_stats_workspace_bytes(cap, C)))
        return fail(SBNET_EINVAL, "%s: workspace missing, misaligned or too small", who);
    hipStream_t s = (hipStream_t)stream;
    float *part = (float *)workspace;
    float *cnt = part ? part + (size_t)cap * C * 2 : nullptr;
    const int rows = bn_rows(cap, p), pieces = bn_pieces(p);
    if (cap > 0) {
        const int grid = rows * p.slabs;
#define SBNET_BN_PARTIAL(DT)                                                                                              \
    hipLaunchKernelGGL(bn_partial<DT>, dim3(grid), dim3(kBnThreads), 0, s, (const uint4 *)x, indices, count, part, cnt, pieces, \
                       make_fastdiv(pieces), p)
        if (dtype == SBNET_F32) SBNET_BN_PARTIAL(SBNET_F32);
        else if (dtype == SBNET_BF16) SBNET_BN_PARTIAL(SBNET_BF16);
        else SBNET_BN_PARTIAL(SBNET_F16);
#undef SBNET_BN_PARTIAL
    }
    hipLaunchKernelGGL(bn_combine, dim3((C + 3) / 4), dim3(1024), 0, s, part, cnt, count, cap, C, rows, pieces, mean, var);
    return launch_status(who);
}
