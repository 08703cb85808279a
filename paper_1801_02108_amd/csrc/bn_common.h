// Shared by the batch-norm kernels over active blocks (bn_stats.hip, bn_apply.hip): the work decomposition
// (an item = a piece of an active block x a slab of 128 bytes of channels per pixel; 8 lanes per pixel strip, 32 pixel groups
// per workgroup) and the element packing of the three storage types.
#pragma once
#include "conv_common.h"

namespace sbnet {

constexpr int kBnThreads = 256;

struct BnParams {
    sbnet_geom g;
    int H, W, C, cap;
    int slabs, cs;               // slabs per pixel, channels per full slab (128 bytes)
    uint32_t pix_vecs;           // 16-byte vectors per pixel
    int hw;                      // pixels per block
    FastDiv div_slabs, div_w;
};

template <int DT> struct BnElem;
template <> struct BnElem<SBNET_F32> {
    static constexpr int EPV = 4;
    static __device__ __forceinline__ void unpack(const uint4 &v, float *f) {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
};
template <> struct BnElem<SBNET_BF16> {
    static constexpr int EPV = 8;
    static __device__ __forceinline__ void unpack(const uint4 &v, float *f) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = bf16_bits_to_float(w[i] & 0xffffu);
            f[2 * i + 1] = bf16_bits_to_float(w[i] >> 16);
        }
    }
};
template <> struct BnElem<SBNET_F16> {
    static constexpr int EPV = 8;
    static __device__ __forceinline__ void unpack(const uint4 &v, float *f) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            union { _Float16 h[2]; uint32_t u; } x;
            x.u = w[i];
            f[2 * i] = (float)x.h[0];
            f[2 * i + 1] = (float)x.h[1];
        }
    }
};

// fp32 -> storage type, round to nearest even
template <int DT>
__device__ __forceinline__ uint4 bn_pack(const float *f) {
    if (DT == SBNET_F32) return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack2<DT>(f[2 * i], f[2 * i + 1]);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

inline sbnet_status bn_fill_params(const char *who, sbnet_dtype dtype, int N, int H, int W, int C, int cap,
                                   const sbnet_geom *g, BnParams *p) {
    if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || cap < 0) return fail(SBNET_EINVAL, "%s: bad sizes", who);
    if (!geom_ok(g)) return fail(SBNET_EINVAL, "%s: bad geometry", who);
    if (!is_float_dtype(dtype)) return fail(SBNET_EUNSUPPORTED, "%s: dtype must be f32, bf16 or f16", who);
    if (g->bstride_h < g->bsize_h || g->bstride_w < g->bsize_w)
        return fail(SBNET_EINVAL, "%s: blocks must not overlap (every pixel counts once)", who);
    const int es = elem_bytes(dtype);
    if ((long long)C * es % 16) return fail(SBNET_EUNSUPPORTED, "%s: a pixel's channels must fill 16-byte vectors", who);
    if ((long long)g->bsize_h * g->bsize_w >= (1LL << 24))
        return fail(SBNET_EUNSUPPORTED, "%s: block too large (pixel counts are kept in fp32)", who);
    p->g = *g;
    p->H = H; p->W = W; p->C = C; p->cap = cap;
    p->cs = 128 / es;
    p->slabs = (C + p->cs - 1) / p->cs;
    p->pix_vecs = (uint32_t)(C * es / 16);
    p->hw = g->bsize_h * g->bsize_w;
    if ((long long)cap * p->slabs >= (1LL << 31)) return fail(SBNET_EUNSUPPORTED, "%s: too many work items", who);
    p->div_slabs = make_fastdiv((uint32_t)p->slabs);
    p->div_w = make_fastdiv((uint32_t)g->bsize_w);
    return SBNET_OK;
}

// ---- work items --------------------------------------------------------------------------------------------------
constexpr int kBnPiece = 128;                 // pixels per item: four per thread
constexpr int kBnSumGroups = 1024;            // workgroups of the kernels that form partial sums, four per CU
typedef float f32x2_a4 __attribute__((ext_vector_type(2), aligned(4)));     // workspaces are 4-byte aligned

inline int bn_pieces(const BnParams &p) { return (p.hw + kBnPiece - 1) / kBnPiece; }
// rows of partial sums: no more than the caller's bound on the blocks, which sizes the workspace
inline int bn_rows(int cap, const BnParams &p) {
    const int rows = p.slabs > 8 ? kBnSumGroups / 8 : kBnSumGroups / p.slabs;
    return cap < rows ? cap : rows;
}

// origin of block b's window and this thread's place in the slab
struct BnPlace {
    int y0, x0, c0;
    bool chan_ok;
    long long base;
};

struct BnBlock {
    int n, by, bx;
};

// Item number `first` + i * `step` of a list of (unit, piece) items, `pieces` of them to a unit, carried along: the number itself
// need not fit 32 bits (a unit's window may lie outside the image for the most part, so the memory does not bound it).
struct BnWalk {
    uint32_t unit, piece, du, dp, pieces;
    __device__ __forceinline__ BnWalk(uint32_t first, uint32_t step, uint32_t pieces_, const FastDiv &div_pieces) : pieces(pieces_) {
        unit = fdiv(first, div_pieces);
        piece = first - unit * pieces;
        du = fdiv(step, div_pieces);
        dp = step - du * pieces;
    }
    __device__ __forceinline__ void advance() {
        unit += du;
        piece += dp;
        if (piece >= pieces) {
            piece -= pieces;
            ++unit;
        }
    }
};
// past the list (the first item of a workgroup, requested beside the count): some block, not used
__device__ __forceinline__ BnBlock bn_block(const int32_t *indices, uint32_t b, int cap) {
    const int32_t *t = indices + 3 * (size_t)min(b, (uint32_t)cap - 1u);
    return {t[0], t[1], t[2]};
}

template <int EPV>
__device__ __forceinline__ BnPlace bn_place(const BnBlock &t, int slab, int k, const BnParams &p) {
    const int n = t.n, by = t.by, bx = t.bx;
    BnPlace w;
    w.y0 = p.g.boffset_h + by * p.g.bstride_h;
    w.x0 = p.g.boffset_w + bx * p.g.bstride_w;
    w.c0 = slab * p.cs + k * EPV;
    w.chan_ok = w.c0 < p.C;
    w.base = (long long)n * p.H * p.W * p.pix_vecs + (long long)(slab * (p.cs / EPV) + k);
    return w;
}

// vector index of pixel q of the block (row-major inside the window), or -1 outside the image / the block
__device__ __forceinline__ long long bn_pixel(const BnPlace &w, int q, const BnParams &p) {
    const int i = (int)fdiv((uint32_t)q, p.div_w), j = q - i * p.g.bsize_w;
    const int yy = w.y0 + i, xx = w.x0 + j;
    if (!w.chan_ok || q >= p.hw || yy < 0 || yy >= p.H || xx < 0 || xx >= p.W) return -1;
    return w.base + ((long long)yy * p.W + xx) * p.pix_vecs;
}


// Sums over the 32 pixel groups of a workgroup: thread c < 8 EPV gets channel c's s1 and s2, every thread the pixel count
// (counted by the lanes that hold a pixel's first vector of the slab).
template <int EPV>
__device__ __forceinline__ float bn_reduce(float (*red)[32][8 * EPV + 1], int *redn, const float *s1, const float *s2, int npx,
                                           float *t1, float *t2) {
    constexpr int NCH = 8 * EPV;
    const int pg = threadIdx.x >> 3, k = threadIdx.x & 7;
#pragma unroll
    for (int e = 0; e < EPV; ++e) {
        red[0][pg][k * EPV + e] = s1[e];
        red[1][pg][k * EPV + e] = s2[e];
    }
    if (k == 0) redn[pg] = npx;
    __syncthreads();
    // in place: thread (quarter, channel) sums eight groups into the first of them, then a thread per channel the four
    const int ch = threadIdx.x % NCH, quarter = threadIdx.x / NCH;
    float a = 0.f, b = 0.f;
    if (quarter < 4) {
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            a += red[0][quarter * 8 + g][ch];
            b += red[1][quarter * 8 + g][ch];
        }
        red[0][quarter * 8][ch] = a;
        red[1][quarter * 8][ch] = b;
    }
    int n = 0;
#pragma unroll
    for (int g = 0; g < 32; ++g) n += redn[g];
    __syncthreads();
    *t1 = (red[0][0][ch] + red[0][8][ch]) + (red[0][16][ch] + red[0][24][ch]);
    *t2 = (red[1][0][ch] + red[1][8][ch]) + (red[1][16][ch] + red[1][24][ch]);
    return (float)n;
}

}  // namespace sbnet
