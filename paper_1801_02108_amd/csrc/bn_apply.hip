// Batch normalisation over the active blocks only (Sec. 3.3 of arXiv 1801.02108: the layers of a residual unit run in
// sparse mode and normalise across the non-sparse elements), forward and backward, on the feature map in place of
// the tile stack: non-overlapping blocks, every active pixel once.
//
//   bn_apply        y = act(gamma (x - mean) / sqrt(var + eps) + beta) on the pixels of the listed blocks that lie
//                   inside the image; every other pixel of y is left as it is.
//   bn_bwd_partial  with z = gamma xhat + beta, g = dy (or dy where z > 0 when the forward call applied a ReLU): per
//                   (row, channel) the sums of g and of g xhat, a row being the pieces that one workgroup walks.
//   bn_bwd_combine  per channel: dbeta = sum g, dgamma = sum g xhat over the rows (every thread a strided subset in
//                   order, then a fixed tree: no atomics, the same bits every run), and the pixel count.
//   bn_bwd_dx       dx = gamma / sqrt(var + eps) * (g - dbeta / n - xhat dgamma / n): the gradient of training-mode
//                   normalisation whose mean and variance are the statistics of these same n pixels.
//
// Work items are (block, piece of 128 pixels, slab of 128 bytes of channels per pixel), with 8 lanes per pixel strip;
// arithmetic in fp32, one rounding to the storage type.  What bounds them is HBM (the active blocks read, and written, once
// per kernel); what kept them from it was the address unit: 32 four-byte coefficient loads per thread and item took as long
// as the pixels.  The coefficients of all channels now pass through LDS, one channel per thread, once per workgroup, and
// partial sums leave a workgroup once (up to 1024 rows of them), not once per block.  bf16, before -> now:
//   800 x 704 x 64, 880 blocks of 16 x 16 (28.8 MB per tensor): apply 19.5 -> 11.9 us (4.8 TB/s), partial 18.4 -> 13.4,
//     combine 4.9 -> 3.9, dx 26.8 -> 18.6 (4.6 TB/s); a large copy runs at 5.1
//   844 x 494 x 64, 3746 blocks of 8 x 8 (30.7 MB): 37.3 -> 12.9, 36.3 -> 13.1, 8.5 -> 3.9, 58.8 -> 18.4 us
#include "bn_common.h"

namespace sbnet {
namespace {

struct BnAffine {
    const float *mean, *var, *gamma, *beta;   // gamma, beta may be null (1, 0)
    float eps;
    int relu;
};

constexpr int kBnCoef = 512;                  // channels whose coefficients one pass through LDS holds

// Per-channel coefficients in LDS, NC arrays of kBnCoef floats.  load() fills channels [c_lo, c_lo + kBnCoef) by all threads of
// the workgroup (barriers around it), get() reads a thread's EPV consecutive channels.
template <int NC>
struct BnCoefs {
    float (*lds)[kBnCoef];
    int c_lo;
    template <typename F>
    __device__ __forceinline__ void load(int first, int C, F f) {
        c_lo = first;
        for (int c = threadIdx.x; c < kBnCoef && first + c < C; c += kBnThreads) {
            float v[NC];
            f(first + c, v);
#pragma unroll
            for (int i = 0; i < NC; ++i) lds[i][c] = v[i];
        }
        __syncthreads();
    }
    template <int EPV>
    __device__ __forceinline__ void get(int i, int c0, float *v) const {
        const int at = min(max(c0 - c_lo, 0), kBnCoef - EPV);     // lanes past the channel count read, and do not use, some value
#pragma unroll
        for (int e = 0; e < EPV; e += 4) {
            const float4 t = *(const float4 *)&lds[i][at + e];
            v[e] = t.x; v[e + 1] = t.y; v[e + 2] = t.z; v[e + 3] = t.w;
        }
    }
};

__device__ __forceinline__ void bn_affine_of(const BnAffine &a, int c, float *v) {
    v[0] = a.mean[c];
    v[1] = 1.0f / sqrtf(a.var[c] + a.eps);
    v[2] = a.gamma ? a.gamma[c] : 1.f;
    v[3] = a.beta ? a.beta[c] : 0.f;
}

// A workgroup walks the items of one group of slabs, whose channels fit the LDS copy; the groups share the grid evenly (a grid
// of bn_grid).  One group after the other in every workgroup left most of them idle where pixels have thousands of
// channels: 32 x 32 x 4096, 10 blocks of 8 x 8: 16.7 us, now 5.3.
__host__ __device__ __forceinline__ int bn_group_slabs(const BnParams &p) { return kBnCoef / p.cs; }
__host__ __device__ __forceinline__ int bn_groups(const BnParams &p) { return (p.slabs + bn_group_slabs(p) - 1) / bn_group_slabs(p); }
struct BnGroup {
    int s0, ns;                               // its slabs
    uint32_t first, step;                     // items of this workgroup
    __device__ __forceinline__ explicit BnGroup(const BnParams &p) {
        const uint32_t groups = (uint32_t)bn_groups(p);
        first = groups == 1 ? blockIdx.x : blockIdx.x / groups;
        step = groups == 1 ? gridDim.x : gridDim.x / groups;
        s0 = (int)(blockIdx.x - first * groups) * bn_group_slabs(p);
        ns = min(bn_group_slabs(p), p.slabs - s0);
    }
};

template <int DT>
__global__ __launch_bounds__(kBnThreads) void bn_apply(const uint4 *x, uint4 *y,                       // y may be x
                                                       const int32_t *__restrict__ indices, const int32_t *__restrict__ count,
                                                       int pieces, FastDiv div_pieces, BnParams p, BnAffine a) {
    constexpr int EPV = BnElem<DT>::EPV;
    __shared__ __align__(16) float cf[4][kBnCoef];
    const int nact = max(min(*count, p.cap), 0);
    const int pg = threadIdx.x >> 3, k = threadIdx.x & 7;
    const BnGroup gr(p);
    const int s0 = gr.s0, ns = gr.ns;
    const uint32_t units = (uint32_t)nact * (uint32_t)ns;     // (block, slab of the group)
    BnWalk it(gr.first, gr.step, (uint32_t)pieces, div_pieces);
    uint32_t b = it.unit / (uint32_t)ns;
    int slab = (int)(it.unit - b * ns);
    BnBlock blk = bn_block(indices, b, p.cap);
    BnCoefs<4> co = {cf, 0};
    co.load(s0 * p.cs, p.C, [&](int c, float *v) { bn_affine_of(a, c, v); });
    while (it.unit < units) {
        const BnPlace w = bn_place<EPV>(blk, s0 + slab, k, p);
        const int q0 = (int)it.piece * kBnPiece + pg;
        it.advance();
        b = ns == 1 ? it.unit : it.unit / (uint32_t)ns;       // the next item's
        slab = (int)(it.unit - b * ns);
        blk = bn_block(indices, b, p.cap);
        long long at[4];
        uint4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            at[u] = bn_pixel(w, q0 + 32 * u, p);
            if (at[u] >= 0) v[u] = x[at[u]];
        }
        float mean[EPV], rstd[EPV], gam[EPV], bet[EPV];
        co.get<EPV>(0, w.c0, mean);
        co.get<EPV>(1, w.c0, rstd);
        co.get<EPV>(2, w.c0, gam);
        co.get<EPV>(3, w.c0, bet);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0) {
                float f[EPV];
                BnElem<DT>::unpack(v[u], f);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float z = fmaf(gam[e], (f[e] - mean[e]) * rstd[e], bet[e]);
                    f[e] = a.relu ? fmaxf(z, 0.f) : z;
                }
                // a vector that straddles the channel count cannot occur: a pixel's channels fill whole vectors
                y[at[u]] = bn_pack<DT>(f);
            }
    }
}

// workspace layout: float part[rows][C][2] (sum g, sum g xhat), at cnt float cnt[rows], ntot; rows = gridDim.x / slabs <= cap
template <int DT>
__global__ __launch_bounds__(kBnThreads) void bn_bwd_partial(const uint4 *__restrict__ x, const uint4 *__restrict__ dy,
                                                             const int32_t *__restrict__ indices,
                                                             const int32_t *__restrict__ count, float *__restrict__ part,
                                                             float *__restrict__ cnt, int pieces, FastDiv div_pieces,
                                                             BnParams p, BnAffine a) {
    constexpr int EPV = BnElem<DT>::EPV, NCH = 8 * EPV;
    __shared__ __align__(16) float cf[4][NCH];
    __shared__ float red[2][32][NCH + 1];
    __shared__ int redn[32];
    const int pg = threadIdx.x >> 3, k = threadIdx.x & 7;
    const uint32_t row = fdiv(blockIdx.x, p.div_slabs), rows = fdiv(gridDim.x, p.div_slabs);
    const int slab = (int)(blockIdx.x - row * p.slabs);
    if (threadIdx.x < NCH && slab * p.cs + (int)threadIdx.x < p.C) {
        float v[4];
        bn_affine_of(a, slab * p.cs + threadIdx.x, v);
#pragma unroll
        for (int i = 0; i < 4; ++i) cf[i][threadIdx.x] = v[i];
    }
    BnWalk it(row, rows, (uint32_t)pieces, div_pieces);
    BnBlock blk = bn_block(indices, it.unit, p.cap);
    const uint32_t nact = (uint32_t)max(min(*count, p.cap), 0);
    if (it.unit >= nact) return;
    __syncthreads();
    float mean[EPV], rstd[EPV], gam[EPV], bet[EPV], s1[EPV], s2[EPV];
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        mean[e] = cf[0][k * EPV + e]; rstd[e] = cf[1][k * EPV + e];
        gam[e] = cf[2][k * EPV + e]; bet[e] = cf[3][k * EPV + e];
        s1[e] = s2[e] = 0.f;
    }
    int npx = 0;
    while (it.unit < nact) {
        const BnPlace w = bn_place<EPV>(blk, slab, k, p);
        const int q0 = (int)it.piece * kBnPiece + pg;
        it.advance();
        blk = bn_block(indices, it.unit, p.cap);                  // the next item's
        long long at[4];
        uint4 vx[4], vg[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            at[u] = bn_pixel(w, q0 + 32 * u, p);
            if (at[u] >= 0) {
                vx[u] = x[at[u]];
                vg[u] = dy[at[u]];
                ++npx;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0) {
                float f[EPV], g[EPV];
                BnElem<DT>::unpack(vx[u], f);
                BnElem<DT>::unpack(vg[u], g);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float xh = (f[e] - mean[e]) * rstd[e];
                    const float ge = (a.relu && !(fmaf(gam[e], xh, bet[e]) > 0.f)) ? 0.f : g[e];
                    s1[e] += ge;
                    s2[e] = fmaf(ge, xh, s2[e]);
                }
            }
    }
    float t1, t2;
    const float n = bn_reduce<EPV>(red, redn, s1, s2, npx, &t1, &t2);
    const int c = slab * p.cs + threadIdx.x;
    if (threadIdx.x < NCH && c < p.C) {
        part[((size_t)row * p.C + c) * 2] = t1;
        part[((size_t)row * p.C + c) * 2 + 1] = t2;
    }
    if (slab == 0 && threadIdx.x == 0) cnt[row] = n;
}

// Four channels per workgroup, 256 threads along the rows of each, four rows in flight per thread.
__global__ __launch_bounds__(1024) void bn_bwd_combine(const float *__restrict__ part, const float *__restrict__ cnt,
                                                       const int32_t *__restrict__ count, int cap, int C, int max_rows, int pieces,
                                                       float *__restrict__ dgamma, float *__restrict__ dbeta,
                                                       float *__restrict__ ntot) {
    __shared__ float s1[64], s2[64], sn[64];
    const int ch = threadIdx.x & 3, row = threadIdx.x >> 2, c = blockIdx.x * 4 + ch;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rows = (int)min((long long)min(*count, cap) * pieces, (long long)max_rows);
    float a = 0.f, q = 0.f, n = 0.f;
    for (int b0 = row; b0 < rows; b0 += 256 * 4) {
        f32x2_a4 v[4];
        float m[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int b = min(b0 + 256 * u, rows - 1);
            v[u] = *(const f32x2_a4 *)(part + ((size_t)b * C + min(c, C - 1)) * 2);
            m[u] = cnt[b];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (b0 + 256 * u < rows) {
                a += v[u][0];
                q += v[u][1];
                n += m[u];
            }
    }
    // a fixed tree: the 16 rows of a wave, then the 16 waves (a wave holds four channels: lane = 4 row + channel)
    auto fold = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int off = 32; off >= 4; off >>= 1) {
            a += __shfl_down(a, off);
            q += __shfl_down(q, off);
            n += __shfl_down(n, off);
        }
    };
    fold();
    if (lane < 4) { s1[wave * 4 + lane] = a; s2[wave * 4 + lane] = q; sn[wave * 4 + lane] = n; }
    __syncthreads();
    if (wave > 0) return;
    a = s1[lane]; q = s2[lane]; n = sn[lane];
    fold();
    if (lane < 4 && c < C) {
        dbeta[c] = a;
        dgamma[c] = q;
        if (c == 0) *ntot = n;
    }
}

template <int DT>
__global__ __launch_bounds__(kBnThreads) void bn_bwd_dx(const uint4 *__restrict__ x, const uint4 *dy,
                                                        uint4 *dx /* may be dy */, const int32_t *__restrict__ indices,
                                                        const int32_t *__restrict__ count, const float *__restrict__ dgamma,
                                                        const float *__restrict__ dbeta, const float *__restrict__ ntot,
                                                        int pieces, FastDiv div_pieces, BnParams p, BnAffine a) {
    constexpr int EPV = BnElem<DT>::EPV;
    __shared__ __align__(16) float cf[6][kBnCoef];
    const int nact = max(min(*count, p.cap), 0);
    const int pg = threadIdx.x >> 3, k = threadIdx.x & 7;
    const float n = *ntot, inv_n = n > 0.f ? 1.0f / n : 0.f;
    const BnGroup gr(p);
    const int s0 = gr.s0, ns = gr.ns;
    const uint32_t units = (uint32_t)nact * (uint32_t)ns;     // (block, slab of the group)
    BnWalk it(gr.first, gr.step, (uint32_t)pieces, div_pieces);
    uint32_t b = it.unit / (uint32_t)ns;
    int slab = (int)(it.unit - b * ns);
    BnBlock blk = bn_block(indices, b, p.cap);
    BnCoefs<6> co = {cf, 0};
    co.load(s0 * p.cs, p.C, [&](int c, float *v) {
        bn_affine_of(a, c, v);
        v[4] = dbeta[c] * inv_n;
        v[5] = dgamma[c] * inv_n;
    });
    while (it.unit < units) {
        const BnPlace w = bn_place<EPV>(blk, s0 + slab, k, p);
        const int q0 = (int)it.piece * kBnPiece + pg;
        it.advance();
        b = ns == 1 ? it.unit : it.unit / (uint32_t)ns;       // the next item's
        slab = (int)(it.unit - b * ns);
        blk = bn_block(indices, b, p.cap);
        long long at[4];
        uint4 vx[4], vg[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            at[u] = bn_pixel(w, q0 + 32 * u, p);
            if (at[u] >= 0) {
                vx[u] = x[at[u]];
                vg[u] = dy[at[u]];
            }
        }
        float mean[EPV], rstd[EPV], gam[EPV], bet[EPV], mg[EPV], mgx[EPV];
        co.get<EPV>(0, w.c0, mean);
        co.get<EPV>(1, w.c0, rstd);
        co.get<EPV>(2, w.c0, gam);
        co.get<EPV>(3, w.c0, bet);
        co.get<EPV>(4, w.c0, mg);
        co.get<EPV>(5, w.c0, mgx);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0) {
                float f[EPV], g[EPV];
                BnElem<DT>::unpack(vx[u], f);
                BnElem<DT>::unpack(vg[u], g);
#pragma unroll
                for (int e = 0; e < EPV; ++e) {
                    const float xh = (f[e] - mean[e]) * rstd[e];
                    const float ge = (a.relu && !(fmaf(gam[e], xh, bet[e]) > 0.f)) ? 0.f : g[e];
                    f[e] = gam[e] * rstd[e] * (ge - mg[e] - xh * mgx[e]);
                }
                dx[at[u]] = bn_pack<DT>(f);
            }
    }
}

// A multiple of the groups, and no more than the device's 256 CUs hold in whole rounds, each workgroup with its coefficients
// loaded once: seven per CU for bn_apply (its registers allow five to nine), twice four for bn_bwd_dx.  With eight, the last
// 256 of bn_apply ran alone at the end: 800 x 704 x 256 in bf16, all blocks of 16 x 16: 2048 workgroups 137 us, 1792 112.
constexpr int kBnApplyGrid = 1792, kBnDxGrid = 2048;
int bn_grid(int cap, const BnParams &p, int pieces, int resident) {
    const int groups = bn_groups(p);
    const long long per = (long long)cap * (p.slabs < bn_group_slabs(p) ? p.slabs : bn_group_slabs(p)) * pieces;
    const long long most = groups < resident ? resident / groups : 1;
    return (int)(per < most ? per : most) * groups;
}

}  // namespace
}  // namespace sbnet

using namespace sbnet;

#define SBNET_BN_DISPATCH(KERNEL, ...)                                                                              \
    do {                                                                                                            \
        if (dtype == SBNET_F32) hipLaunchKernelGGL(KERNEL<SBNET_F32>, dim3(grid), dim3(kBnThreads), 0, s, __VA_ARGS__); \
        else if (dtype == SBNET_BF16) hipLaunchKernelGGL(KERNEL<SBNET_BF16>, dim3(grid), dim3(kBnThreads), 0, s, __VA_ARGS__); \
        else hipLaunchKernelGGL(KERNEL<SBNET_F16>, dim3(grid), dim3(kBnThreads), 0, s, __VA_ARGS__);                  \
    } while (0)

extern "C" sbnet_status sbnet_sparse_bn_apply(const void *x, sbnet_dtype dtype, int N, int H, int W, int C,
                                              const int32_t *indices, const int32_t *count, int cap, const sbnet_geom *g,
                                              const float *mean, const float *var, const float *gamma, const float *beta,
                                              float eps, int relu, void *y, void *stream) {
    const char *who = "sbnet_sparse_bn_apply";
    if (!x || !y || !indices || !count || !mean || !var) return fail(SBNET_EINVAL, "%s: null pointer", who);
    if (!(eps >= 0.f)) return fail(SBNET_EINVAL, "%s: eps must not be negative", who);
    BnParams p;
    sbnet_status st = bn_fill_params(who, dtype, N, H, W, C, cap, g, &p);
    if (st != SBNET_OK) return st;
    if (((uintptr_t)x | (uintptr_t)y) & 15) return fail(SBNET_EINVAL, "%s: x and y must be 16-byte aligned", who);
    if (cap == 0) return SBNET_OK;
    hipStream_t s = (hipStream_t)stream;
    const BnAffine a = {mean, var, gamma, beta, eps, relu ? 1 : 0};
    const int pieces = bn_pieces(p), grid = bn_grid(cap, p, pieces, kBnApplyGrid);
    SBNET_BN_DISPATCH(bn_apply, (const uint4 *)x, (uint4 *)y, indices, count, pieces, make_fastdiv(pieces), p, a);
    return launch_status(who);
}

extern "C" size_t sbnet_bn_backward_workspace_bytes(int cap, int C) {
    if (cap < 0 || C <= 0) return 0;
    return ((size_t)cap * C * 2 + (size_t)cap + 1) * sizeof(float);
}

extern "C" sbnet_status sbnet_sparse_bn_backward(const void *x, const void *dy, sbnet_dtype dtype, int N, int H, int W, int C,
                                                 const int32_t *indices, const int32_t *count, int cap,
                                                 const sbnet_geom *g, const float *mean, const float *var,
                                                 const float *gamma, const float *beta, float eps, int relu, void *dx,
                                                 float *dgamma, float *dbeta, void *workspace, size_t workspace_bytes,
                                                 void *stream) {
    const char *who = "sbnet_sparse_bn_backward";
    if (!x || !dy || !dx || !indices || !count || !mean || !var || !dgamma || !dbeta)
        return fail(SBNET_EINVAL, "%s: null pointer", who);
    if (!(eps >= 0.f)) return fail(SBNET_EINVAL, "%s: eps must not be negative", who);
    BnParams p;
    sbnet_status st = bn_fill_params(who, dtype, N, H, W, C, cap, g, &p);
    if (st != SBNET_OK) return st;
    if (((uintptr_t)x | (uintptr_t)dy | (uintptr_t)dx) & 15)
        return fail(SBNET_EINVAL, "%s: x, dy and dx must be 16-byte aligned", who);
    if (!workspace || ((uintptr_t)workspace & 3) || workspace_bytes < sbnet_bn_backward_workspace_bytes(cap, C))
        return fail(SBNET_EINVAL, "%s: workspace missing, misaligned or too small", who);
    hipStream_t s = (hipStream_t)stream;
    const BnAffine a = {mean, var, gamma, beta, eps, relu ? 1 : 0};
    float *part = (float *)workspace;
    float *cnt = part + (size_t)cap * C * 2;
    float *ntot = cnt + cap;
    const int rows = bn_rows(cap, p), all = bn_pieces(p);
    if (cap > 0) {
        const int grid = rows * p.slabs;
        SBNET_BN_DISPATCH(bn_bwd_partial, (const uint4 *)x, (const uint4 *)dy, indices, count, part, cnt, all, make_fastdiv(all),
                          p, a);
    }
    hipLaunchKernelGGL(bn_bwd_combine, dim3((C + 3) / 4), dim3(1024), 0, s, part, cnt, count, cap, C, rows, all, dgamma, dbeta,
                       ntot);
    if (cap > 0) {
        const int pieces = bn_pieces(p), grid = bn_grid(cap, p, pieces, kBnDxGrid);
        SBNET_BN_DISPATCH(bn_bwd_dx, (const uint4 *)x, (const uint4 *)dy, (uint4 *)dx, indices, count, dgamma, dbeta, ntot, pieces,
                          make_fastdiv(pieces), p, a);
    }
    return launch_status(who);
}
