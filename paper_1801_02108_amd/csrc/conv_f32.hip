// Convolution on tiles (Sec. 3.2 of arXiv 1801.02108) in fp32 arithmetic, unfused and fused with gather and scatter:
// float32 tensors of any channel count, and bf16 / f16 tensors whose channel counts the 16-bit matrix kernels do not
// take (those are widened on their way to LDS).  Implicit GEMM on v_mfma_f32_16x16x4_f32: full fp32 products and sums
// at twice the rate of scalar FMA code (256 against 128 FLOP per clock and CU; packed fp32 instructions are off here).
//
// What bounds it: at the sizes these layers have, one memory round trip after another (count -> block list -> pixels)
// and the matrix work of a wave, not bandwidth.  So an item is small, 64 output pixels x up to 64 output channels (a
// wave: 16 pixels), which gives a layer of 110 active 16 x 16 blocks 440 workgroups, and everything an item
// needs is requested at once: the input rows of its pixels and the weights of the channel chunk, both staged in LDS.
// Where all channels are one chunk and one output group, the weights stay in LDS for the life of the workgroup and
// their request does not wait for the block list.  400 x 704 x 24 -> 24, 110 blocks of 16 x 16: 55 us with one thread
// per output element (conv_direct) -> 10.4 us; 64 x 64 x 16 -> 16, 19 blocks of 8 x 8: 15.1 us -> 5.8 us (kernel
// times of a trace; in-kernel clocks of the latter: 2000 until count and block are known, 3400 until the pixels are requested,
// 1500 until they are in LDS, 2100 of matrix work for 36 steps of 32, 1100 for the results).
//
// Operand order.  A k-step is 8 channels of one tap: lane l holds channels 2 (l/16) and 2 (l/16) + 1 of pixel (input) or
// output channel (weights) l%16, one 8-byte LDS read per operand for two matrix instructions.  LDS pixels are an
// odd multiple of 8 floats apart, so that the 16 pixels of a read start in different banks.
#include "conv_common.h"

namespace sbnet {

namespace {

constexpr int kF32Pix = 64;        // output pixels per item
constexpr int kF32Stage = 8;       // vectors of input, and of weights, in flight per thread while a chunk is staged
constexpr int kF32Lds = 80 * 1024; // two workgroups per CU

// What the kernel needs and no more: arguments that do not fit the scalar registers are kept in vector lanes.
struct F32Params {
    const void *in, *w;
    void *out;
    const float *bias;                    // [Cout] or null
    const int32_t *indices;               // (n, by, bx), or null: work item b is sample b (a tile stack)
    const int32_t *count;
    int cap, relu, add;
    int H, W, Cin, Ho, Wo, Cout;          // of one sample: the map, or one tile of a stack
    int iy_off, iy_str, ix_off, ix_str;   // input window of block (by, bx)
    int oy_off, oy_str, ox_off, ox_str;   // output block
    int kh, kw, sh, sw, oh, ow, tw;
    int mpasses, ngroups, nchunks;
    int C8, cc8, S;                       // groups of 8 input channels: in all, in a chunk; floats between pixels in LDS
    int per_px, d_c, d_px, d_row, d_col;  // staging: vectors per pixel of a chunk; 256 vectors further on = d_px pixels
                                          // (d_row rows and d_col columns) and d_c vectors
    FastDiv div_pn, div_ng, div_ow, div_px, div_tw;
};

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// four stored weights -> fp32
template <int DT> __device__ __forceinline__ float4 widen4(const typename Elem<DT>::T *p) {
    if (DT == SBNET_F32) return *(const float4 *)p;
    const uint2 v = *(const uint2 *)p;
    return make_float4(unpack_lo<DT>(v.x), unpack_hi<DT>(v.x), unpack_lo<DT>(v.y), unpack_hi<DT>(v.y));
}

// NB: blocks of 16 output channels per item; K3: 3 x 3 taps (unrolled); V4: pixels staged four channels at a time
// (float32 with at least four channels; 16-byte loads need 4-byte alignment only), else channel by channel
template <int DT, int NB, bool K3, bool V4>
__global__ __launch_bounds__(256) void conv_f32_kernel(F32Params p) {
    typedef typename Elem<DT>::T T;
    extern __shared__ __align__(16) float lds_f[];
    const T *w = (const T *)p.w;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = lane >> 4, l16 = lane & 15;
    const int M = p.oh * p.ow;
    const int taps = K3 ? 9 : p.kh * p.kw;
    const int kw = K3 ? 3 : p.kw, kh = K3 ? 3 : p.kh;
    float *wl = lds_f;                                  // [NB][cc8][taps][64][2]
    float *xl = lds_f + NB * p.cc8 * taps * 128;        // [rows][tw] pixels of S floats
    constexpr int E = V4 ? 4 : 1;                       // channels per staged input element

    // 16-byte LDS vectors of weights of output group ng, chunk `chunk`: one run per output block, and a single one where
    // the chunk is all channels (runs of existing blocks follow each other in memory and in LDS)
    float4 wv[kF32Stage];
    auto w_request = [&](const T *src, uint32_t L, uint32_t v0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kF32Stage; ++u)
            if (v0 - threadIdx.x + u * 256 < L)         // uniform: a request costs the CU's address unit its time, used or not
                wv[u] = widen4<DT>(src + (size_t)min(v0 + u * 256, L - 1) * 4);
    };
    auto w_store = [&](float *dst, uint32_t L, uint32_t v0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < kF32Stage; ++u)
            if (v0 + u * 256 < L) *(float4 *)(dst + (v0 + u * 256) * 4) = wv[u];
    };
    const int nbt = (p.Cout + 15) >> 4;
    const bool one_chunk = p.nchunks == 1, resident = one_chunk && p.ngroups == 1;
    const uint32_t all = (uint32_t)min(NB, nbt) * p.C8 * taps * 32;
    if (resident) w_request(w, all, threadIdx.x);
    bool fresh = true;
    // Channel by channel, and all channels one chunk: those past Cin are zeroed once and not staged (requesting them took the
    // address unit as long as the others: 800 x 704 x 1 -> 8, all blocks: 50.0 -> 43.7 us)
    if (!V4 && p.per_px < p.cc8 * 8) {
        const int full = (int)fdiv(kF32Pix, p.div_ow), out_rows = min(kF32Pix - full * p.ow ? full + 2 : full, p.oh);      // as on the host
        const int floats = ((out_rows - 1) * p.sh + kh) * p.tw * p.S;
        for (int v = threadIdx.x * 4; v < floats; v += 256 * 4) *(float4 *)(xl + v) = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    // this thread's first staged element, and its step: element index / pixel / row / column carried along instead of divided
    const int px_first = (int)fdiv(threadIdx.x, p.div_px), c_first = (int)threadIdx.x - px_first * p.per_px;
    const int row_first = (int)fdiv(px_first, p.div_tw), col_first = px_first - row_first * p.tw;

    const uint32_t per_tile = (uint32_t)p.mpasses * p.ngroups;
    // the first item's block is requested beside the count, not after it (the grid has no more workgroups than cap has items;
    // past the count the triple is not used)
    int n = 0, by = 0, bx = 0;
    auto locate = [&](uint32_t b) __attribute__((always_inline)) {
        n = (int)b;
        if (p.indices) {
            n = p.indices[3 * b];
            by = p.indices[3 * b + 1];
            bx = p.indices[3 * b + 2];
        }
    };
    locate(fdiv(blockIdx.x, p.div_pn));
    const uint32_t items = (uint32_t)max(min(*p.count, p.cap), 0) * per_tile;
    const uint32_t sample_bytes = (uint32_t)p.H * p.W * p.Cin * (uint32_t)sizeof(T);
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        const uint32_t b = fdiv(item, p.div_pn);
        const uint32_t rest = item - b * per_tile;
        const int pass = (int)fdiv(rest, p.div_ng);
        const int ng = (int)rest - pass * p.ngroups;
        if (item != blockIdx.x) locate(b);
        const int p_lo = pass * kF32Pix, p_hi = min(p_lo + kF32Pix, M);
        const int i_lo = (int)fdiv(p_lo, p.div_ow), i_hi = (int)fdiv(p_hi - 1, p.div_ow);
        const int r_lo = i_lo * p.sh;
        const int npix = ((i_hi - i_lo) * p.sh + kh) * p.tw;
        const int gy0 = p.iy_off + by * p.iy_str + r_lo, gx0 = p.ix_off + bx * p.ix_str;
        const int px = p_lo + wave * 16 + l16;          // this lane's output pixel
        const int pi = (int)fdiv(min(px, M - 1), p.div_ow), pj = min(px, M - 1) - pi * p.ow;
        const int xbase = ((pi * p.sh - r_lo) * p.tw + pj * p.sw) * p.S + 2 * q;
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((const T *)p.in + (size_t)n * p.H * p.W * p.Cin), (short)0, (int)sample_bytes, (int)kBufWord3);

        const float bias = p.bias ? p.bias[min(ng * NB * 16 + lane, p.Cout - 1)] : 0.f;   // lane k: output channel k of the group

        f32x4 acc[NB], acc2[NB];                        // even and odd channel of a pair: two shorter chains
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = acc2[nb] = (f32x4){0.f, 0.f, 0.f, 0.f};

        for (int chunk = 0; chunk < p.nchunks; ++chunk) {
            const int n8 = min(p.cc8, p.C8 - chunk * p.cc8);
            const int nblocks = min(NB, nbt - ng * NB);
            const T *wsrc = w + ((size_t)ng * NB * p.C8 + (size_t)chunk * p.cc8) * taps * 128;
            const uint32_t run = (uint32_t)(one_chunk ? nblocks : 1) * n8 * taps * 32;
            __syncthreads();                            // the previous chunk / item is consumed
            if (fresh && !resident) w_request(wsrc, run, threadIdx.x);
            int pix = px_first, c = c_first, row = row_first, col = col_first;
            bool first = true;
            do {                                        // a batch: kF32Stage elements per thread in flight
                float4 xv[kF32Stage];
                int dst[kF32Stage];                     // LDS position, -1: none
#pragma unroll
                for (int u = 0; u < kF32Stage; ++u) {
                    dst[u] = -1;
                    if (__builtin_amdgcn_readfirstlane(pix) >= npix) continue;      // the wave's elements are all past the end
                    const int ch = chunk * p.cc8 * 8 + c * E;
                    const int gx = gx0 + col;
                    dst[u] = pix < npix ? pix * p.S + c * E : -1;
                    // outside the sample: an offset outside its descriptor, which reads as zeros (of rows far enough below
                    // the product would wrap back into it)
                    const int at = V4 ? min(ch, p.Cin - 4) : ch;
                    uint32_t off = (((uint32_t)(gy0 + row) * p.W + gx) * p.Cin + at) * (uint32_t)sizeof(T);
                    if ((uint32_t)gx >= (uint32_t)p.W || ch >= p.Cin || (uint32_t)(gy0 + row) >= (uint32_t)p.H) off = kOutOfRange;
                    if (V4) {
                        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0);
                        xv[u] = __builtin_bit_cast(float4, t);
                        if (dst[u] >= 0) dst[u] |= (ch - at) & 3;       // the vector's last 1..3 channels do not exist
                    } else if (sizeof(T) == 4) {
                        xv[u].x = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)off, 0, 0));
                    } else {
                        xv[u].x = unpack_lo<DT>(__builtin_amdgcn_raw_buffer_load_b16(rx, (int)off, 0, 0));
                    }
                    c += p.d_c;
                    const bool wrap = c >= p.per_px;
                    if (wrap) c -= p.per_px;
                    pix += p.d_px + (wrap ? 1 : 0);
                    col += p.d_col + (wrap ? 1 : 0);
                    row += p.d_row;
                    if (col >= p.tw) { col -= p.tw; ++row; }
                }
                if (first && fresh) {
                    w_store(wl, run, threadIdx.x);
                    for (uint32_t v0 = threadIdx.x + 256 * kF32Stage; v0 < run; v0 += 256 * kF32Stage) {
                        w_request(wsrc, run, v0);
                        w_store(wl, run, v0);
                    }
                    if (!one_chunk)
                        for (int nb = 1; nb < nblocks; ++nb)
                            for (uint32_t v0 = threadIdx.x; v0 < run; v0 += 256 * kF32Stage) {
                                w_request(wsrc + (size_t)nb * p.C8 * taps * 128, run, v0);
                                w_store(wl + nb * p.cc8 * taps * 128, run, v0);
                            }
                    first = false;
                }
#pragma unroll
                for (int u = 0; u < kF32Stage; ++u)
                    if (dst[u] >= 0) {
                        if (V4) {
                            // a vector that reaches past the pixel's channels was read from its last four
                            float4 t = xv[u];
                            if (dst[u] & 1) t = make_float4(t.y, t.z, t.w, 0.f);
                            if (dst[u] & 2) t = make_float4(t.z, t.w, 0.f, 0.f);
                            *(float4 *)(xl + (dst[u] & ~3)) = t;
                        } else xl[dst[u]] = xv[u].x;
                    }
            } while (pix < npix);
            __syncthreads();
            if (resident) fresh = false;                // the weights stay for the life of the workgroup

            const float *wp = wl + lane * 2;
            for (int g8 = 0; g8 < n8; ++g8) {
                const float *xb = xl + xbase + g8 * 8;
                const float *wb = wp + g8 * taps * 128;
                auto tap_step = [&](int r, int t) __attribute__((always_inline)) {
                    const float2 xv = *(const float2 *)(xb + (r * p.tw + t) * p.S);
                    float2 wv2[NB];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) wv2[nb] = *(const float2 *)(wb + (nb * p.cc8 * taps + r * kw + t) * 128);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc[nb] = mfma_f32(wv2[nb].x, xv.x, acc[nb]);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) acc2[nb] = mfma_f32(wv2[nb].y, xv.y, acc2[nb]);
                };
                if (K3) {
#pragma unroll
                    for (int k = 0; k < 9; ++k) tap_step(k / 3, k % 3);
                } else {
                    for (int r = 0; r < kh; ++r)
                        for (int t = 0; t < kw; ++t) tap_step(r, t);
                }
            }
        }

        // lane: output channels 16 nb + 4 q + 0..3 of its pixel
        float bv[NB][4];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int k = 0; k < 4; ++k) bv[nb][k] = __shfl(bias, nb * 16 + 4 * q + k);
        const int oy = p.oy_off + by * p.oy_str + pi, ox = p.ox_off + bx * p.ox_str + pj;
        if (px < p_hi && oy >= 0 && oy < p.Ho && ox >= 0 && ox < p.Wo) {
            T *dst = (T *)p.out + (((size_t)n * p.Ho + oy) * p.Wo + ox) * p.Cout;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const int o0 = (ng * NB + nb) * 16 + 4 * q;
                float v[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    v[k] = acc[nb][k] + acc2[nb][k] + bv[nb][k];
                    if (p.relu) v[k] = fmaxf(v[k], 0.f);
                }
                if (DT == SBNET_F32 && (p.Cout & 3) == 0) {
                    if (o0 < p.Cout) {
                        float4 r = make_float4(v[0], v[1], v[2], v[3]);
                        if (p.add) {
                            const float4 old = *(const float4 *)(dst + o0);
                            r = make_float4(r.x + old.x, r.y + old.y, r.z + old.z, r.w + old.w);
                        }
                        *(float4 *)(dst + o0) = r;
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (o0 + k < p.Cout) {
                            if (p.add) v[k] += Elem<DT>::load(dst + o0 + k);
                            Elem<DT>::store(dst + o0 + k, v[k]);
                        }
                }
            }
        }
    }
}

template <int DT, bool K3, bool V4>
void launch_nb(const F32Params &p, int nb, int grid, size_t lds, hipStream_t s) {
#define SBNET_F32_LAUNCH(NB)                                                                                         \
    do {                                                                                                             \
        if (lds > 48 * 1024)                                                                                         \
            (void)hipFuncSetAttribute((const void *)conv_f32_kernel<DT, NB, K3, V4>,                                 \
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                         \
        hipLaunchKernelGGL((conv_f32_kernel<DT, NB, K3, V4>), dim3(grid), dim3(256), lds, s, p);                     \
    } while (0)
    if (nb == 1) SBNET_F32_LAUNCH(1);
    else if (nb == 2) SBNET_F32_LAUNCH(2);
    else if (nb == 3) SBNET_F32_LAUNCH(3);
    else SBNET_F32_LAUNCH(4);
#undef SBNET_F32_LAUNCH
}

template <int DT>
void launch_k(const F32Params &p, bool v4, int nb, int grid, size_t lds, hipStream_t s) {
    constexpr bool F = DT == SBNET_F32;
    const bool k3 = p.kh == 3 && p.kw == 3;
    if (F && v4) k3 ? launch_nb<DT, true, F>(p, nb, grid, lds, s) : launch_nb<DT, false, F>(p, nb, grid, lds, s);
    else k3 ? launch_nb<DT, true, false>(p, nb, grid, lds, s) : launch_nb<DT, false, false>(p, nb, grid, lds, s);
}

}  // namespace

// c.oh, c.ow set by the caller.  False: a pass's input rows do not fit LDS even eight channels at a time, or a sample is
// beyond 32-bit offsets.
bool conv_f32_try(sbnet_dtype dt, bool fused, const ConvParams &c, hipStream_t s, sbnet_status *st, const char *who) {
    F32Params p = {};
    p.in = c.in; p.w = c.w; p.out = c.out; p.bias = c.bias;
    p.indices = fused ? c.indices : nullptr;
    p.count = c.count; p.cap = c.cap; p.relu = c.relu; p.add = fused ? c.add : 0;
    p.Cin = c.Cin; p.Cout = c.Cout;
    if (fused) {
        p.H = c.H; p.W = c.W; p.Ho = c.Ho; p.Wo = c.Wo;
        p.iy_off = c.g_in.boffset_h; p.iy_str = c.g_in.bstride_h; p.ix_off = c.g_in.boffset_w; p.ix_str = c.g_in.bstride_w;
        p.oy_off = c.g_out.boffset_h; p.oy_str = c.g_out.bstride_h; p.ox_off = c.g_out.boffset_w; p.ox_str = c.g_out.bstride_w;
    } else {
        p.H = c.th; p.W = c.tw; p.Ho = c.oh; p.Wo = c.ow;
    }
    if ((long long)p.H * p.W * p.Cin * elem_bytes(dt) >= (1LL << 31)) return false;
    p.kh = c.kh; p.kw = c.kw; p.sh = c.sh; p.sw = c.sw; p.oh = c.oh; p.ow = c.ow; p.tw = c.tw;
    const long long M = (long long)p.oh * p.ow;
    const int taps = p.kh * p.kw, nbt = (p.Cout + 15) / 16;
    const bool v4 = dt == SBNET_F32 && p.Cin >= 4;
    p.mpasses = (int)((M + kF32Pix - 1) / kF32Pix);
    // rows of output that 64 consecutive pixels can touch
    long long out_rows = (kF32Pix + p.ow - 1) / p.ow + ((kF32Pix % p.ow) ? 1 : 0);
    if (out_rows > p.oh) out_rows = p.oh;
    const long long rows = (out_rows - 1) * p.sh + p.kh;
    auto stride = [](int c8) { return (c8 & 1) ? c8 * 8 : c8 * 8 + 8; };
    auto lds_for = [&](int c8, int nb) { return (rows * p.tw * stride(c8) + (long long)nb * c8 * taps * 128) * 4; };
    p.C8 = (p.Cin + 7) / 8;
    // Blocks of 16 output channels per item: as many (up to four, none empty) as leave all input channels one chunk, else four
    // or so.  One where the caller's bound on the active blocks leaves the device's 1024 workgroup slots room for an item
    // per channel block: a wave's chain of matrix steps is the time of such a call.  38 -> 40 channels, 121 blocks of
    // 12 x 12: 20.8 us with three blocks in two chunks, 17.7 with one in one.
    int nb = (nbt + (nbt + 3) / 4 - 1) / ((nbt + 3) / 4);
    for (int k = 4; k >= 1; --k)
        if (nbt % k == 0 && lds_for(p.C8, k) <= kF32Lds) { nb = k; break; }
    if ((long long)p.cap * p.mpasses * nbt <= 1024) nb = 1;
    p.ngroups = (nbt + nb - 1) / nb;
    auto lds_of = [&](int c8) { return lds_for(c8, nb); };
    int c8 = p.C8;
    while (c8 > 1 && lds_of(c8) > kF32Lds) --c8;
    p.nchunks = (p.C8 + c8 - 1) / c8;
    p.cc8 = (p.C8 + p.nchunks - 1) / p.nchunks;
    const long long lds = lds_of(p.cc8);
    if (lds > 160 * 1024) return false;
    p.S = stride(p.cc8);
    p.per_px = p.cc8 * 8 / (v4 ? 4 : 1);
    if (!v4 && p.nchunks == 1) p.per_px = p.Cin;
    p.d_px = 256 / p.per_px; p.d_c = 256 % p.per_px;
    p.d_row = p.d_px / p.tw; p.d_col = p.d_px % p.tw;
    p.div_px = make_fastdiv(p.per_px);
    p.div_tw = make_fastdiv(p.tw);
    p.div_ow = make_fastdiv(p.ow);
    p.div_pn = make_fastdiv((uint32_t)p.mpasses * p.ngroups);
    p.div_ng = make_fastdiv(p.ngroups);
    const long long items = (long long)p.cap * p.mpasses * p.ngroups;
    if (items >= (1LL << 31)) return false;
    const int per_cu = (int)(160 * 1024 / lds < 4 ? 160 * 1024 / lds : 4);
    const int grid = (int)(items < 256 * per_cu ? items : 256 * per_cu);
    if (dt == SBNET_F32) launch_k<SBNET_F32>(p, v4, nb, grid, (size_t)lds, s);
    else if (dt == SBNET_BF16) launch_k<SBNET_BF16>(p, v4, nb, grid, (size_t)lds, s);
    else launch_k<SBNET_F16>(p, v4, nb, grid, (size_t)lds, s);
    *st = launch_status(who);
    return true;
}

}  // namespace sbnet
