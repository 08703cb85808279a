// 3x3 tile convolution of stride 1 or 2, bf16 / f16, for layers whose weights stay in LDS: all input channels by a group of 32, 64
// or 96 output channels, at most 160 KB with eight waves' buffers of 2.5 to 12 KB and the bias (Sec. 3.2 and 3.4 of arXiv
// 1801.02108: the regular convolution between gather and scatter; fused with both, and as the data gradient of a tile
// convolution).
//
// conv3.hip stages a chunk of weights with every chunk of pixels and has its workgroup meet at a barrier per chunk.  Here
// the weights are copied to LDS once for the life of the workgroup and every wave works by itself from then on:
//   * Item of a wave = 64 consecutive output pixels of a tile x the group's channels.  The wave stages the input rows of
//     its pixels, 32 channels at a time, in a buffer of its own and waits for nobody: no barrier after the prologue.
//   * Two waves per SIMD: while one waits for its rows or stores results the other has the matrix core, and two waves read
//     LDS twice as fast as one (a wave alone is served a 16-byte read about every 30 clocks, which four fragment reads per
//     four matrix steps just reach).  Three waves per SIMD (168 registers) ran at the same rate.
//   * Rows go from memory to LDS without passing through registers (buffer_load ... lds, 16 bytes a lane).  Lanes out of
//     the descriptor's range write zeros: pixels outside the image and channels past Cin.  The copy's LDS side is linear
//     in the lane, so pixels are 64 bytes apart without padding; bank conflicts are avoided by a key (place_key).
//   * A workgroup serves a contiguous run of items, the runs differ by one item at most: the last round of work is a
//     quarter of a 16x16 block per SIMD instead of a block per CU.
//   * Items of 32 pixels, of all the group's channels or of 32, where that makes fewer or shorter rounds (the count decides
//     on the device).
// Measured, conv3 -> this (400 x 352, bf16, us): 64 -> 64, blocks of 8, 5 % active 6.6 -> 5.5, 20 % 9.3 -> 6.7, all 26.4 -> 16.2;
// blocks of 14 7.7 -> 5.7, 9.3 -> 8.7, 18.2 -> 17.2; 32 -> 32, blocks of 14, all 11.9 -> 8.2 (4.4 TB/s: memory); 48 -> 80, blocks
// of 12, 30 % 16.7 -> 12.2, all 26.9 -> 23.4; 1600 x 1408, half of all blocks, 64 -> 64 blocks of 12 142 -> 113, of 14 112 -> 109.
//   * Stride 2: items of 32 pixels (their rows are twice as many and twice as wide), chunks of 16 channels (so that 64 -> 96 keeps
//     all its weights beside eight buffers), the even columns of a row before its odd ones.  conv3 -> this: 800 x 704 to
//     400 x 352, blocks of 16, 64 -> 96, 5 % active 9.1 -> 7.4, 30 % 18.3 -> 12.5; 32 -> 32, all 17.6 -> 11.7.
// What bounds it at many items (1600 x 1408, half of all blocks of 12, 64 -> 64, counters): matrix cores busy 38 % of the time,
// LDS 45 (11 of them bank conflicts), the address unit (copies of 64-byte pieces, stores) 41, vector
// instructions 42, beside each other; with fewer than two items per wave the latency of an item and the copy of the weights.
// At stride 1 the sum over (chunk of 32 channels, tap, 16 channels) runs in the order of conv3's 32-channel chunks: same bits.  At
// stride 2 it runs over (chunk of 16 channels, tap), conv3's order with 16-channel chunks.
#include "conv_common.h"

#include <type_traits>

namespace sbnet {

constexpr int kLdsW = 160 * 1024;
constexpr int kWavesW = 8;                   // two per SIMD
constexpr int kCopiesW = 12;                 // most 1 KB copies of a chunk's rows: 192 pixels
constexpr int kOstPsW = 80;                  // result transpose: bytes per pixel (32 channels + 16 B pad)

constexpr int kWavePlain = 0, kWaveOwn = 1, kWaveMask = 2;      // ConvForm

struct PlanW {
    FastDiv div_item[3];     // items of a tile: 64 pixels; 32 pixels; 32 pixels by one block of 32 channels
    int copies[2];           // 1 KB copies of a chunk's rows, 64 and 32 pixels
    int nks;                 // 16-channel steps per tap: ceil(Cin / 16)
    int cin16, ks16;         // packed weights: 16-channel steps per tap, per 64-channel group
    int ngroups, per_xcd;    // output-channel groups; workgroups per group and XCD
    FastDiv div_groups, div_wgs;
    uint32_t w_bytes;        // bytes of the packed 32x32x16 operand copy
    uint32_t bias_off, buf_off, buf_bytes;
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) unsigned char lds_byte;      // (a pointer known to be to LDS: a copy's target needs no check)

// The 16-byte piece k of staged pixel q is kept at place k ^ place_key(q) of the pixel's 64 bytes.  Sixteen neighbouring
// pixels take four keys, eight neighbouring ones, read together with the next piece, two that differ in bit 1: either
// way the lanes of a read cover all banks.
// At stride 2 a pixel has two pieces (16 channels a chunk), and the even columns of a row are staged before its odd ones: the
// pixels of a read are neighbours again.
template <int STR>
__device__ __forceinline__ uint32_t place_key(uint32_t px) { return STR == 2 ? (px >> 3) & 1u : ((px >> 1) & 2u) | ((px >> 3) & 1u); }

// The items start + wave, start + wave + 8, ... below end, 32 PBW pixels by CBW blocks of 32 channels each.
// request_weights: copies the group's weights and its bias to LDS.
template <int DT, bool FUSED, bool ADD, int NB, int EPI, int STR, int CBW, int PBW, typename Weights>
__device__ __forceinline__ void wave_items(const ConvParams &p, const PlanW &q, unsigned char *lds, uint32_t start, uint32_t end,
                                           int ng, const Weights &request_weights) {
    constexpr bool OWN = FUSED && EPI != kWavePlain;
    constexpr int SM = PBW == 2 ? 0 : CBW == NB ? 1 : 2;      // which of the plan's item sizes
    constexpr int SPLIT = NB / CBW;                  // items that share their pixels
    constexpr int PP = PBW * 32;
    constexpr int CC = STR == 2 ? 16 : 32, CV = CC / 8;       // channels per chunk; 16-byte pieces of a staged pixel
    constexpr int D = CBW * PBW >= 6 ? 1 : 2;        // steps the fragment reads run ahead of the matrix steps
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 5, m = lane & 31;
    const int M = p.oh * p.ow;
    unsigned char *buf = lds + q.buf_off + wave * q.buf_bytes;
    lds_byte *buf_l = (lds_byte *)lds + (q.buf_off + wave * q.buf_bytes);
    const int nchunks = STR == 2 ? q.nks : (q.nks + 1) >> 1;

    struct Item { uint32_t b; int pass, cb0, n, by, bx; };
    int lane_zero = 0;                               // (a per-lane load of a uniform address: not waited for on the spot)
    asm volatile("" : "+v"(lane_zero));
    auto request = [&](uint32_t it) __attribute__((always_inline)) {
        Item c;
        c.b = fdiv(it, q.div_item[SM]);
        const uint32_t rest = it - c.b * q.div_item[SM].d;
        c.pass = (int)(rest / SPLIT);
        c.cb0 = (int)(rest % SPLIT) * CBW;
        c.n = c.by = c.bx = 0;
        if (FUSED && !OWN) {
            const int32_t *t = p.indices + 3 * (size_t)c.b + lane_zero;
            c.n = t[0];
            c.by = t[1];
            c.bx = t[2];
        }
        return c;
    };
    auto resolve = [&](Item c) __attribute__((always_inline)) {
        if (FUSED && !OWN) {
            c.n = __builtin_amdgcn_readfirstlane(c.n);
            c.by = __builtin_amdgcn_readfirstlane(c.by);
            c.bx = __builtin_amdgcn_readfirstlane(c.bx);
        }
        if (OWN) c.n = (int)c.b;
        return c;
    };

    const int in_w = FUSED ? p.W : p.tw;
    const uint32_t in_bytes = (uint32_t)(FUSED ? p.H : p.th) * in_w * p.Cin * 2u;
    // Copy i moves 16-byte place lane % 4 of staged pixel 16 i + lane / 4 (row by row, tw pixels each): off, relative to the
    // item's first pixel and the chunk's first channel.  Worked out once where registers allow: an item's copies are
    // issued back to back.
    constexpr bool KEEP = STR == 2 || (PBW == 2 && NB < 3);
    struct Place { uint32_t off; int col, ch; };
    auto place_of = [&](int i, int ln) __attribute__((always_inline)) {
        const uint32_t px = (uint32_t)(i * (64 / CV) + ln / CV);
        const uint32_t row = fdiv(px, p.div_tw), slot = px - row * p.tw, even = (uint32_t)(p.tw + 1) >> 1;
        const uint32_t col = STR == 1 ? slot : slot < even ? 2 * slot : 2 * (slot - even) + 1;
        const uint32_t piece = (uint32_t)(ln & (CV - 1)) ^ place_key<STR>(px);
        return Place{((row * in_w + col) * p.Cin + piece * 8) * 2u, (int)col, (int)piece * 8};
    };
    uint32_t gd[KEEP ? kCopiesW : 1];
    constexpr int PK = PBW == 2 ? 0 : 1;             // which of the plan's copy counts
    // rows of channels CC c .. of an item -> the wave's buffer
    auto stage = [&](const Item &c, int chunk) __attribute__((always_inline)) {
        const int r_lo = (int)fdiv((uint32_t)c.pass * PP, p.div_ow);
        const uint16_t *base = (const uint16_t *)p.in;
        int x0 = 0, y0 = r_lo * STR;
        if (FUSED) {
            y0 += p.g_in.boffset_h + c.by * p.g_in.bstride_h;
            x0 = p.g_in.boffset_w + c.bx * p.g_in.bstride_w;
            base += (long long)c.n * p.H * p.W * p.Cin;
        } else {
            base += (long long)c.b * p.th * p.tw * p.Cin;
        }
        // (rows outside the image are outside the descriptor: the offset wraps below zero above it)
        const uint32_t origin = (uint32_t)((y0 * in_w + x0) * p.Cin + chunk * CC) * 2u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, (int)in_bytes, (int)kBufWord3);
        if constexpr (KEEP) {
            if (x0 >= 0 && x0 + p.tw <= in_w && chunk * CC + CC <= p.Cin) {              // no lane to leave out
#pragma unroll
                for (int i = 0; i < kCopiesW; ++i)
                    if (i < q.copies[PK])
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(buf_l + i * 1024), 16, (int)(origin + gd[i]), 0, 0, 0);
                return;
            }
        }
        for (int i = 0; i < q.copies[PK]; ++i) {
            const Place t = place_of(i, lane);
            const bool ok = (uint32_t)(x0 + t.col) < (uint32_t)in_w && chunk * CC + t.ch < p.Cin;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(buf_l + i * 1024), 16, (int)(ok ? origin + t.off : kOutOfRange), 0, 0, 0);
        }
    };

    uint32_t floor16 = p.relu ? 0u : 0x80008000u;
    asm volatile("" : "+s"(floor16));
    int floor_i = p.relu ? 0 : (int)0x80000000;
    asm volatile("" : "+s"(floor_i));

    // the first item's place in the list is on its way while the weights are requested
    uint32_t it = start + wave;
    const Item head = request(min(it, end - 1u));
    request_weights();
    if constexpr (KEEP) {
#pragma unroll
        for (int i = 0; i < kCopiesW; ++i) {
            gd[i] = i < q.copies[PK] ? place_of(i, lane).off : 0u;
            asm volatile("" : "+v"(gd[i]));          // opaque: kept as it is, not regrouped with the origins
        }
    }
    Item cur = resolve(head), nxt = cur;
    bool more = false, fresh = true;                 // fresh: this wave has not been at the barrier
    int chunk = 0;
    f32x16 acc[CBW][PBW];
    uint32_t xlin[PBW], p_lo = 0;
    if (it >= end) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        return;
    }
    for (;;) {                                       // a chunk of an item
        stage(cur, chunk);
        if (chunk == 0) {
            more = it + kWavesW < end;
            nxt = request(more ? it + kWavesW : it);
            // this lane's pixels in the staged rows, pixel block pb of the item
            p_lo = (uint32_t)cur.pass * PP;
            const uint32_t i_lo = fdiv(p_lo, p.div_ow);
#pragma unroll
            for (int pb = 0; pb < PBW; ++pb) {
                const uint32_t px = min(p_lo + (uint32_t)(pb * 32 + m), (uint32_t)M - 1u);
                const uint32_t i = fdiv(px, p.div_ow), j = px - i * p.ow;
                xlin[pb] = (i - i_lo) * STR * p.tw + j;
            }
            if (fresh) {
                __builtin_amdgcn_s_waitcnt(0);
                __syncthreads();                     // weights and bias, from every wave; no barrier after this one
                fresh = false;
            }
            // accumulators start from the bias
#pragma unroll
            for (int cb = 0; cb < CBW; ++cb) {
                const float4 *bl = (const float4 *)(lds + q.bias_off) + ((cur.cb0 + cb) * 32 + g * 16) / 4;
#pragma unroll
                for (int k4 = 0; k4 < 4; ++k4) {
                    const float4 bv = bl[k4];
#pragma unroll
                    for (int pb = 0; pb < PBW; ++pb) {
                        acc[cb][pb][k4 * 4 + 0] = bv.x; acc[cb][pb][k4 * 4 + 1] = bv.y;
                        acc[cb][pb][k4 * 4 + 2] = bv.z; acc[cb][pb][k4 * 4 + 3] = bv.w;
                    }
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the chunk's rows are in LDS
        auto steps = [&](auto kst_tag) __attribute__((always_inline)) {
            constexpr int KST = decltype(kst_tag)::value, NS = 9 * KST;
            const unsigned char *WL = lds + (chunk * (STR == 2 ? 9 : 18) * NB + cur.cb0) * 1024 + lane * 16;
            uint4 xa[D + 1][CBW], xb[D + 1][PBW];
            uint32_t xl[PBW];
#pragma unroll
            for (int pb = 0; pb < PBW; ++pb) {
                xl[pb] = xlin[pb];
                asm volatile("" : "+v"(xl[pb]));     // opaque: otherwise the taps' addresses are hoisted out of the loop and spilled
            }
            auto read = [&](int s) __attribute__((always_inline)) {
                const int slot = s % (D + 1), tap = s / KST, ks = s % KST;
#pragma unroll
                for (int cb = 0; cb < CBW; ++cb) xa[slot][cb] = *(const uint4 *)(WL + (s * NB + cb) * 1024);
#pragma unroll
                for (int pb = 0; pb < PBW; ++pb) {
                    const uint32_t dx = STR == 1 ? tap % 3 : tap % 3 == 1 ? (uint32_t)(p.tw + 1) >> 1 : tap % 3 >> 1;
                    const uint32_t lin = xl[pb] + (uint32_t)((tap / 3) * p.tw) + dx;
                    xb[slot][pb] = *(const uint4 *)(buf + lin * (CC * 2) + (((uint32_t)(ks * 2 + g) ^ place_key<STR>(lin)) * 16));
                }
            };
#pragma unroll
            for (int s = 0; s < D; ++s) read(s);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s + D < NS) read(s + D);
#pragma unroll
                for (int cb = 0; cb < CBW; ++cb)
#pragma unroll
                    for (int pb = 0; pb < PBW; ++pb)
                        acc[cb][pb] = mfma32x32x16<DT>(xa[s % (D + 1)][cb], xb[s % (D + 1)][pb], acc[cb][pb]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (STR == 1 && 2 * chunk + 1 < q.nks) steps(std::integral_constant<int, 2>{});
        else steps(std::integral_constant<int, 1>{});
        if (++chunk < nchunks) {
            __builtin_amdgcn_s_waitcnt(0xC07F);      // lgkmcnt(0): every read of the buffer has been answered
            continue;
        }

        // ---- results: 32 pixels x 32 channels at a time through the wave's buffer, so that a store carries 64-byte runs.
        //      Pixels past the tile's end, columns outside the image and channels past Cout get the out-of-range offset.
        {
            uint16_t *obase = (uint16_t *)p.out;
            uint32_t obytes, origin;
            int ox0 = 0, out_w;
            if (FUSED) {
                const int oy0 = p.g_out.boffset_h + cur.by * p.g_out.bstride_h;
                ox0 = p.g_out.boffset_w + cur.bx * p.g_out.bstride_w;
                out_w = p.Wo;
                obase += (long long)cur.n * p.Ho * p.Wo * p.Cout;
                obytes = (uint32_t)p.Ho * p.Wo * p.Cout * 2u;
                origin = (uint32_t)((oy0 * p.Wo + ox0) * p.Cout) * 2u;
            } else {
                out_w = p.ow;
                obase += (long long)cur.b * M * p.Cout;
                obytes = (uint32_t)M * p.Cout * 2u;
                origin = 0;
            }
            const __amdgpu_buffer_rsrc_t ors = __builtin_amdgcn_make_buffer_rsrc((void *)obase, 0, (int)obytes, (int)kBufWord3);
            auto pixel_offset = [&](uint32_t px, bool &ok) __attribute__((always_inline)) {
                const uint32_t pc = min(px, (uint32_t)M - 1u);
                const uint32_t i = fdiv(pc, p.div_ow), j = pc - i * p.ow;
                ok = px < (uint32_t)M && (!FUSED || (uint32_t)(ox0 + (int)j) < (uint32_t)p.Wo);
                return origin + (uint32_t)((i * out_w + j) * p.Cout) * 2u;
            };
            const int chg = (ng * NB + cur.cb0) * 32;
            uint4 act[EPI == kWaveMask ? PBW : 1][CBW][2];
            if (EPI == kWaveMask) {                  // what the results are masked by, laid out as they are
                const long long at = (const char *)obase - (const char *)p.out;
                const __amdgpu_buffer_rsrc_t mrs = __builtin_amdgcn_make_buffer_rsrc((void *)((const char *)p.indices + at), 0,
                                                                                    (int)obytes, (int)kBufWord3);
#pragma unroll
                for (int pb = 0; pb < PBW; ++pb)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        bool ok;
                        const uint32_t off = pixel_offset(p_lo + (uint32_t)(pb * 32 + j * 16) + (lane >> 2), ok);
#pragma unroll
                        for (int cb = 0; cb < CBW; ++cb) {
                            const int ch = chg + cb * 32 + (lane & 3) * 8;
                            act[EPI == kWaveMask ? pb : 0][cb][j] = buf_load16(mrs, (ok && ch < p.Cout) ? off + (uint32_t)ch * 2u : kOutOfRange);
                        }
                    }
            }
#pragma unroll
            for (int pb = 0; pb < PBW; ++pb) {
                bool ok1 = false;
                const uint32_t off1 = ADD ? pixel_offset(p_lo + (uint32_t)(pb * 32 + m), ok1) : 0u;
                bool ok2[2];
                uint32_t off2[2];
#pragma unroll
                for (int j = 0; j < 2; ++j) off2[j] = pixel_offset(p_lo + (uint32_t)(pb * 32 + j * 16) + (lane >> 2), ok2[j]);
#pragma unroll
                for (int cb = 0; cb < CBW; ++cb) {
                    uint4 old[2];
                    if (ADD) {                       // read in the MFMA layout, so that the sum is formed in fp32 and rounded once
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int ch = chg + cb * 32 + g * 16 + h * 8;
                            old[h] = buf_load16(ors, (ok1 && ch < p.Cout) ? off1 + (uint32_t)ch * 2u : kOutOfRange);
                        }
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        uint32_t w[4];
                        if (ADD) {
                            float v[8];
#pragma unroll
                            for (int k = 0; k < 8; ++k) v[k] = __int_as_float(max(__float_as_int(acc[cb][pb][h * 8 + k]), floor_i));
                            const uint4 o = old[h];
                            v[0] += unpack_lo<DT>(o.x); v[1] += unpack_hi<DT>(o.x);
                            v[2] += unpack_lo<DT>(o.y); v[3] += unpack_hi<DT>(o.y);
                            v[4] += unpack_lo<DT>(o.z); v[5] += unpack_hi<DT>(o.z);
                            v[6] += unpack_lo<DT>(o.w); v[7] += unpack_hi<DT>(o.w);
#pragma unroll
                            for (int k = 0; k < 4; ++k) w[k] = pack2<DT>(v[2 * k], v[2 * k + 1]);
                        } else {
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                w[k] = relu_pair(pack2<DT>(acc[cb][pb][h * 8 + 2 * k], acc[cb][pb][h * 8 + 2 * k + 1]), floor16);
                        }
                        *(uint4 *)(buf + m * kOstPsW + g * 32 + h * 16) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                    __builtin_amdgcn_wave_barrier();     // LDS serves one wave's accesses in order: no wait needed
                    const int ch = chg + cb * 32 + (lane & 3) * 8;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        uint4 v = *(const uint4 *)(buf + (j * 16 + (lane >> 2)) * kOstPsW + (lane & 3) * 16);
                        if (EPI == kWaveMask) {
                            const uint4 a = act[EPI == kWaveMask ? pb : 0][cb][j];
                            v.x &= positive_halves<DT>(a.x); v.y &= positive_halves<DT>(a.y);
                            v.z &= positive_halves<DT>(a.z); v.w &= positive_halves<DT>(a.w);
                        }
                        buf_store16(ors, (ok2[j] && ch < p.Cout) ? off2[j] + (uint32_t)ch * 2u : kOutOfRange, v);
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
        if (!more) return;
        it += kWavesW;
        cur = resolve(nxt);
        chunk = 0;
        __builtin_amdgcn_s_waitcnt(0xC07F);          // the transposes' reads
    }
}

template <int DT, bool FUSED, bool ADD, int NB, int EPI, int STR>
__global__ __launch_bounds__(64 * kWavesW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void conv_wave_kernel(ConvParams p, PlanW q) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups are dealt round-robin to the 8 XCDs: an XCD serves neighbouring runs of items of every group
    const uint32_t local = blockIdx.x >> 3;
    const uint32_t member = fdiv(local, q.div_groups);
    const int ng = (int)(local - member * q.ngroups);
    const uint32_t idx = (blockIdx.x & 7) * q.per_xcd + member, wgs = q.div_wgs.d;

    const uint32_t nact = (uint32_t)max(min(*p.count, p.cap), 0);
    // Rounds of the workgroup's four SIMDs with either item, weighted by the matrix steps of a round and what an item adds
    // to them.  Measured slopes (1600 x 1408, half of the blocks): 32 pixels by 64 channels cost an eighth more per pixel
    // than 64 pixels (four staged rows for two, three fragments per two matrix steps; blocks of 16, 64 -> 64: 97.6 us
    // against 88.9), by 96 channels nothing more (14, 48 -> 96: 124 and 129); 32 pixels by 32 channels three quarters.
    auto rounds = [&](int k) __attribute__((always_inline)) {
        return (fdiv(nact * q.div_item[k].d + wgs - 1, q.div_wgs) + 3) >> 2;
    };
    const uint32_t c64 = STR == 2 ? ~0u : rounds(0) * (16 * NB), c32 = NB > 1 ? rounds(1) * (NB == 2 ? 18u : 24u) : ~0u, c1 = rounds(2) * 14u;
    const int kind = c64 <= c32 && c64 <= c1 ? 0 : c32 <= c1 ? 1 : 2;
    const uint32_t items = nact * q.div_item[kind].d;
    const uint32_t each = fdiv(items, q.div_wgs), extra = items - each * wgs;
    const uint32_t start = idx * each + min(idx, extra), end = start + each + (idx < extra ? 1u : 0u);
    if (start >= end) return;

    const __amdgpu_buffer_rsrc_t wrs = __builtin_amdgcn_make_buffer_rsrc((void *)((const uint4 *)p.w + p.w32_offset), 0,
                                                                        (int)q.w_bytes, (int)kBufWord3);
    // the group's weights: LDS [chunk of 32 channels][tap][16-channel step][block of 32 outputs][lane], packed
    // [group of 64 outputs][tap][step][half][lane]
    auto weights = [&]() __attribute__((always_inline)) {
    const int nblk = 9 * q.nks * NB;
    for (int b = wave; b < nblk; b += kWavesW) {
        const int s = b / NB, cb = b - s * NB;
        const int c = STR == 2 ? s / 9 : s / 18, r = s - c * (STR == 2 ? 9 : 18);
        const bool full = STR == 1 && 2 * c + 1 < q.nks;
        const int tap = full ? r >> 1 : r, ks = full ? r & 1 : 0;
        const uint32_t nbk = (uint32_t)(ng * NB + cb);
        const uint32_t off = (nbk >> 1) * (uint32_t)q.ks16 * 2048u + (uint32_t)(tap * q.cin16 + (STR == 2 ? c : 2 * c + ks)) * 2048u + (nbk & 1u) * 1024u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_void *)((lds_byte *)lds + b * 1024), 16, (int)(off + lane * 16), 0, 0, 0);
    }
    {
        float *bl = (float *)(lds + q.bias_off);
        const int i = threadIdx.x, o = ng * NB * 32 + i;
        if (i < NB * 32) bl[i] = (p.bias && o < p.Cout) ? p.bias[o] : 0.f;
    }
    };
    if constexpr (STR == 1) {
        if (kind == 0) {
            wave_items<DT, FUSED, ADD, NB, EPI, STR, NB, 2>(p, q, lds, start, end, ng, weights);
            return;
        }
    }
    if constexpr (NB > 1) {
        if (kind == 1) {
            wave_items<DT, FUSED, ADD, NB, EPI, STR, NB, 1>(p, q, lds, start, end, ng, weights);
            return;
        }
    }
    wave_items<DT, FUSED, ADD, NB, EPI, STR, 1, 1>(p, q, lds, start, end, ng, weights);
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
template <int DT, bool FUSED, bool ADD, int EPI, int STR>
static void launch_wave_nb(int nb, const ConvParams &p, const PlanW &q, int grid, size_t lds, hipStream_t s) {
#define SBNET_LW(NB)                                                                                                      \
    do {                                                                                                                  \
        auto kern = conv_wave_kernel<DT, FUSED, ADD, NB, EPI, STR>;                                                            \
        (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * kWavesW), lds, s, p, q);                                 \
    } while (0)
    if (nb == 3) SBNET_LW(3);
    else if (nb == 2) SBNET_LW(2);
    else SBNET_LW(1);
#undef SBNET_LW
}
template <int DT>
static void launch_wave(bool fused, ConvForm form, int nb, const ConvParams &p, const PlanW &q, int grid, size_t lds, hipStream_t s) {
    if (form == ConvForm::own) launch_wave_nb<DT, true, false, kWaveOwn, 1>(nb, p, q, grid, lds, s);
    else if (form == ConvForm::mask) launch_wave_nb<DT, true, false, kWaveMask, 1>(nb, p, q, grid, lds, s);
#define SBNET_LWS(STR)                                                                                 \
    do {                                                                                               \
        if (fused && p.add) launch_wave_nb<DT, true, true, kWavePlain, STR>(nb, p, q, grid, lds, s);   \
        else if (fused) launch_wave_nb<DT, true, false, kWavePlain, STR>(nb, p, q, grid, lds, s);      \
        else launch_wave_nb<DT, false, false, kWavePlain, STR>(nb, p, q, grid, lds, s);                \
    } while (0)
    else if (p.sh == 2) SBNET_LWS(2);
    else SBNET_LWS(1);
#undef SBNET_LWS
}

struct LaunchW {
    PlanW q;
    int nb, grid;            // blocks of 32 output channels of a group; workgroups
    size_t lds;
};

// Shape checks and launch shape; false where another kernel takes the call.
static bool conv_wave_plan(sbnet_dtype dt, bool fused, const ConvParams &p, ConvForm form, LaunchW *l) {
    if (dt != SBNET_BF16 && dt != SBNET_F16) return false;
    if (p.kh != 3 || p.kw != 3 || p.sh != p.sw || (p.sh != 1 && p.sh != 2) || p.Cin % 8 != 0 || p.Cout % 8 != 0) return false;
    if (form == ConvForm::inside || (form != ConvForm::plain && (!fused || p.add || p.sh != 1))) return false;
    // byte offsets inside one sample (fused) or one tile are kept in 32 bits and checked by the hardware
    // against a buffer descriptor of that size
    if ((fused ? (long long)p.H * p.W : (long long)p.th * p.tw) * p.Cin >= (1LL << 30)) return false;
    if ((fused ? (long long)p.Ho * p.Wo : (long long)p.oh * p.ow) * p.Cout >= (1LL << 30)) return false;
    const long long M = (long long)p.oh * p.ow;
    const bool strided = p.sh == 2;
    PlanW &q = l->q;
    q = {};
    const int CinP = (p.Cin + 31) / 32 * 32, blocks = (p.Cout + 31) / 32;
    q.nks = (p.Cin + 15) / 16;
    q.cin16 = CinP / 16;
    q.ks16 = 9 * q.cin16;
    const long long wb = (long long)((p.Cout + 63) / 64) * q.ks16 * 2048;
    if (wb >= (1LL << 31)) return false;
    q.w_bytes = (uint32_t)wb;
    long long buf = 0, passes[2];
    for (int v = 0; v < 2; ++v) {
        const int pp = v ? 32 : 64;
        passes[v] = (M + pp - 1) / pp;
        // input rows that pp consecutive output pixels can touch
        long long rows = (pp + p.ow - 1) / p.ow + ((pp % p.ow) ? 1 : 0);
        if (rows > p.oh) rows = p.oh;
        if (strided) {
            if (v == 0) continue;                    // (items of 32 pixels only)
            if (rows > 1 && ((rows - 2) * 2 + 3) * p.tw > kCopiesW * 32) return false;
            long long most = 1;                      // (exactly: where an item begins in a row repeats after at most ow items)
            for (long long k = 0; k < passes[1] && k < p.ow; ++k) {
                const long long last = 32 * k + 31 < M ? 32 * k + 31 : M - 1, r = last / p.ow - 32 * k / p.ow + 1;
                if (r > most) most = r;
            }
            rows = most;
        }
        rows = (rows - 1) * p.sh + 3;
        q.copies[v] = (int)((rows * p.tw * (strided ? 2 : 4) + 63) / 64);
        if (q.copies[v] > kCopiesW) return false;
        if (q.copies[v] * 1024LL > buf) buf = q.copies[v] * 1024LL;
    }
    if (buf < 32 * kOstPsW) buf = (32 * kOstPsW + 15) / 16 * 16;
    // channels per group: the fewest blocks of 32 in all, then the largest group
    int nb = 0;
    for (int t = 3; t >= 1; --t) {
        if ((long long)q.nks * 9 * t * 1024 + kWavesW * buf + t * 128 > kLdsW) continue;
        if (nb == 0 || (blocks + t - 1) / t * t < (blocks + nb - 1) / nb * nb) nb = t;
    }
    if (nb == 0) return false;
    q.ngroups = (blocks + nb - 1) / nb;
    if (q.ngroups > 2) return false;
    // The longest list, in blocks of 256 pixels of its bound, that is served here (`most`).  At stride 2 a line of memory is
    // fetched once for each of its chunks of 16 channels, and long lists, whose maps do not stay in the caches, wait for that:
    // most layers lose from some length on where every block is active and win where few are.  What was measured on either side,
    // us by conv3 and here at 5, 10, 30, 60, 100 % of the bound active unless named, or the change from conv3 to here in % at 10,
    // 40, 70, 100 % (two maps in turn).  The lines of 40, 60 and 180 lie between the numbers of active blocks at which the curves
    // of a list of 550 cross.
    //   layer                                          most  blocks  figures
    //   up to 48 channels (in %):
    //     blocks of up to 64 pixels                      -   8 x 8: -30 to -50 at any length
    //     8 KB a chunk, up to 256 pixels, 12 x 12:
    //       33 to 48 -> 64                             600     600   -16 +3 +5 +10; 2000 -28 +15 +27 +30; 10000 +25 +38 +47 +53
    //       33 to 48 -> 32 or 96                      1000    1000   -22 -6 +2 -6; 2000 -35 +6 +17 +25; 96: -16 -5 -1 -13; -35 +1 +15 +11
    //       up to 32                                  1500    1500   32 -> 64 -38 +1 0 -6; 3000 -10 +4 +19 +12; 32 -> 32 -47 -13 -13 -19; 6000
    //                                                                -11 +6 +12 +15; 24 -> 96 3000 -18 -14 +8 +13
    //     others, groups of 64, 16 x 16               2000    2000   32 -> 64 -32 -8 -8 -3; 3000 -14 -4 +9 +11; 48 -> 64 -28 -16 -6 +1; 3000
    //                                                                -8 -3 0 +8; 10000 -8 +5 +9 +11; 16 -> 128 -15 -3 +4 +3; 4000
    //                                                                -16 +2 +6 +19; 24 x 24, 48 -> 64 -27 -13 -3 +5
    //       10 x 10, which fill their items badly    1000    1000   48 -> 64 +1 +3 -2 -11; 2000 +4 +7 +11 +8
    //     ... of 32                                   6000    6000   16 x 16, 48 -> 32 -26 -6 +1 +6; 10000 -15 -1 +3 +7
    //       10 x 10                                  3000    3000   48 -> 32 -7 -3 0 -1; 4000 -6 +2 +8 +10
    //     ... of 96                                     -    10000   16 x 16, 48 -> 96 -6 -3 -2 -3; 24 x 24 -39 -36 -34 -33
    //     more than 8 KB a chunk, 14 x 14              400     550   32 -> 64 (us) 60 % 12.4 11.4, all 17.0 18.4
    //   from 64 channels (us):
    //   groups of 96: 64 -> 96, 16 x 16                 600    550   10.3 7.8, 13.3 9.9, 20.4 14.8, 27.3 25.9, 39.3 37.9
    //                                                          600   9.5 7.6, 12.9 9.4, 20.0 15.3, 27.1 27.0, 39.5 41.4
    //                                                          800   9.5 7.7, 13.2 10.3, 21.1 18.9, 34.7 33.3, 56.0 55.4
    //                                                          1100  12.9 9.0, 13.7 12.3, 28.3 26.9, 49.3 48.3, 72.9 77.2
    //                                                          2200  13.6 12.2, 21.0 17.1, 50.1 50.0, 86.0 92.4, 133 143
    //   small blocks of more than 64 channels, for
    //   which conv3 has no wide group: 64 -> 128, 8 x 8 600    550   all 53.3 36.7
    //   64 channels, blocks that fill their items:
    //   64 -> 64, 16 x 16                               600    550   5 % 9.1 6.1, 30 % 16.6 10.9, 60 % 21.7 22.4, all 40.1 35.2
    //   two groups of 32: 96 -> 64, 14 x 14              40    550   5 % 14.1 9.5, 15 % 14.3 15.4
    //   blocks that fill their items badly:              60    550   64 -> 128, 10 x 10, 5 % 8.8 8.2, 15 % 10.9 11.4; 14 x 14,
    //                                                                10.4 9.0, 12.6 12.6
    //   others: 64 -> 64, 12 x 12                       180    550   30 % 20.5 12.9, 60 % 22.8 26.4
    // Not taken at any length: more than eight chunks one after the other, where conv3's items of 64 pixels fit the block as well
    // (200 x 176, 192 -> 32, 8 x 8, 5 % 11.4 9.5, 15 % 11.7 12.1, all 11.8 13.0), and 110 KB of weights for a few small blocks (200 x
    // 176, 64 -> 96, 8 x 8, 30 % 7.3 7.5).
    const long long any = 1LL << 40;
    if (strided) {
        const bool bad_fit = M > 64 && passes[1] * 32 * 8 > M * 9;           // an eighth of the items is padding
        long long most = 180;
        if (q.nks <= 3) {
            if (q.copies[1] > 8) most = 400;
            else if (M <= 64) most = any;
            else if (q.copies[1] > 6 && M < 256) most = q.nks < 3 ? 1500 : nb == 2 ? 600 : 1000;
            else most = nb == 3 ? any : (nb == 2 ? 2000 : 6000) / (bad_fit ? 2 : 1);
        } else if (nb == 3 || (M <= 64 && blocks > 2) || (q.nks <= 4 && M >= 256 && M % 32 == 0)) most = 600;
        else if (nb == 1 && q.ngroups == 2) most = 40;
        else if (bad_fit) most = 60;
        if (p.cap * M > most * 256 || (q.nks > 8 && M <= 64)) return false;
        if (nb == 3 && q.nks > 3 && M <= 64 && p.cap * M <= 64 * 256) return false;
    }
    // Two groups of 32, each of which stages the pixels again, while the list is not long: 400 x 352, 128 -> 64, blocks of 16,
    // 5 % active 9.2 us by conv3 and 7.1 here, 30 % 13.8 and 13.2, all 31.3 and 30.1; blocks of 8 47.3 and 30.9; 1600 x 1408,
    // half of all blocks of 16 181 and 207.
    if (!strided && nb == 1 && q.ngroups == 2 && p.cap * M > 640 * 256) return false;
    // Groups of 96 beside conv3's wide items of 256 pixels: blocks of more than 256 pixels are even (24 x 24, 48 -> 80: 20 %
    // active 11.3 us there, 11.8 here, all 28.6 and 28.7), and so are those whose pixels no item size fits better than
    // theirs, with the last round the worse here (14 x 14: 5 % active 8.5 and 6.2, 20 % 11.2 and 10.6, 60 % 18.1 and 18.0, all
    // 754 blocks 23.2 and 25.8): there while the list's bound is two of their rounds.  14 x 14, 5, 30, 60, 100 % active, conv3
    // and here: 48 -> 80, 512 blocks 7.9 6.1, 11.6 10.8, 18.1 14.1, 19.7 20.1, 754 8.4 6.1, 13.2 12.8, 19.2 19.4, 25.4 28.9, 2200 10.1
    // 8.9, 26.1 25.6, 41.8 42.6, 61.6 61.6; 48 -> 96, 512 7.9 5.8, 10.7 9.4, 16.4 12.2, 17.4 16.1, 754 8.0 5.8, 11.2 10.5, 16.9 15.1,
    // 23.3 21.9.
    if (!strided && nb == 3 && (M > 256 || (M > 192 && M < 256 && p.cap > 512))) return false;
    // ... and from 33 channels on 256 pixels, where those items are full: change in % at 10, 40, 70, 100 % active, 16 x 16: 40 -> 80, 800
    // blocks -14 -12 -6 -1, 1100 -16 +1 +21 +9, 2500 -8 +8 +13 +16; 48 -> 80 the same; 48 -> 96, 4000 -16 -3 -1 0, 6000 -21 -1 +11 +13.
    // Up to 32 channels (24 -> 96), for which conv3 has no such groups, -11 to -25 at any length.
    if (!strided && nb == 3 && M > 192 && p.Cin > 32 && p.cap * M > (p.Cout % 96 ? 800 : 4000) * 256) return false;
    // Long lists of blocks whose pixels neither item fits: 64 -> 64 in units of 256 pixels, 15 x 15, 1000 -17 -14 -3 -5, 3000 -22 +5 +4
    // +4; 14 x 14, 4000 -22 -1 0 +3, 6000 -8 +7 +11 +11; 48 -> 64 and 32 -> 64 -15 to +6 up to 10000.
    if (!strided && nb == 2 && q.nks > 3 && M > 192 && M < 256 && p.cap * M > 3000 * 256) return false;
    // Wide rows of one chunk, half of them or more outside the item and the map's lines written in two halves: on tiles, the same units,
    // 35 x 35, 8 -> 64, 1000 -26 -14 -4 -2, 1500 -6 -10 0 +13, 2500 -1 +4 +18 +28; 33 x 33, 16 -> 128, 500 -28 -10 -29 -11, 1000 -3 -12 -1 +13, 1500
    // -29 -3 +18 +23; 28 x 28, 2500 -20 +2 +15 +7.  From 17 channels on -1 to -28 at any length.
    if (!strided && q.nks == 1 && nb == 2 && q.copies[0] > 10 && p.cap * M > 1000 / q.ngroups * 256) return false;
    // Output channels that do not fill their blocks, and little matrix work: the pieces of a line of memory are written apart (by two
    // groups of workgroups, or by two blocks of which the last is 8 or 24 wide).  Change in % at 10, 40, 100 %, same units: 8 -> 120, 12 x 12, 600 -18 -17 -11, 1000 -24 -18 +22,
    // 1500 -21 +6 +45, 2500 -31 +29 +62; 8 -> 104, 16 x 16, 600 -18 -5 -1, 1000 -19 -19 +12, 1500 -20 +1 +22; 24 -> 56, 16 x 16, 2200 -5 0
    // +21, 5000 +7 +17 +22; 24 -> 104, 14 x 14, 1000 -9 +5 +25; 16 -> 112, 14 x 14, 1000 -26 -16 +22, 2500 -20 +22 +47; one group of 96: 16 -> 88,
    // 12 x 12, 1000 -40 -12 -1, 2500 -16 +9 +12.  Wins still: 8 x 8 (24 -> 56, 2500 -8 -20 -25), blocks that are filled (24 -> 64, 16 x 16,
    // 2200 -8 -20 -9; 16 -> 128, 20 x 20, 2500 -28 -19 -23) and from 33 input channels on (48 -> 104, 12 x 12, 2500 -24 -16 -16).
    if (!strided && nb == 2 && q.nks <= 2 && (p.Cout % 16 || (p.Cout % 32 && q.ngroups == 2)) && M > 64 && p.cap * M > 800 * 256) return false;
    if (!strided && nb == 3 && q.nks == 1 && p.Cout % 16 && M > 64 && p.cap * M > 1500 * 256) return false;
    // Long lists of tiles that conv3's items of 384 pixels fit better than six of 64: data gradient of 64 -> 64 on 16 x 16 blocks
    // (18 x 18 results), 880 tiles 28.9 and 28.5 us, 1540 45.8 and 48.4, 2200 62.0 and 65.4.
    if (!strided && nb == 2 && M > 256 && M <= 384 && p.cap * M > 1200 * 256) return false;
    if ((long long)p.cap * passes[1] * nb >= (1LL << 31)) return false;
    q.div_item[0] = make_fastdiv((uint32_t)passes[0]);
    q.div_item[1] = make_fastdiv((uint32_t)passes[1]);
    q.div_item[2] = make_fastdiv((uint32_t)passes[1] * nb);
    q.buf_off = (uint32_t)(q.nks * 9 * nb * 1024);
    q.buf_bytes = (uint32_t)buf;
    q.bias_off = q.buf_off + kWavesW * q.buf_bytes;
    l->lds = q.bias_off + (size_t)nb * 128;
    // Two of the smallest items per workgroup on lists too short to fill the device: eight, one per wave, stood at one CU's address
    // unit together (all active: 100 x 88, 32 -> 32, blocks of 8 5.2 -> 4.0 us, 64 -> 64 6.1 -> 5.5, stride 2 on 200 x 176, 128 -> 32,
    // blocks of 16 12.3 -> 10.2), one is no faster than two.
    long long per_xcd = ((long long)p.cap * passes[1] * nb + 15) / 16;
    if (per_xcd > 32 / q.ngroups) per_xcd = 32 / q.ngroups;
    q.per_xcd = (int)per_xcd;
    q.div_groups = make_fastdiv((uint32_t)q.ngroups);
    q.div_wgs = make_fastdiv((uint32_t)(8 * q.per_xcd));
    l->nb = nb;
    l->grid = 8 * q.per_xcd * q.ngroups;
    return true;
}

bool conv_wave_accepts(sbnet_dtype dt, bool fused, const ConvParams &p) {
    LaunchW l;
    return conv_wave_plan(dt, fused, p, ConvForm::plain, &l);
}

bool conv_wave_try(sbnet_dtype dt, bool fused, const ConvParams &p, hipStream_t s, sbnet_status *st, const char *who, ConvForm form) {
    LaunchW l;
    if (!conv_wave_plan(dt, fused, p, form, &l)) return false;
    if (dt == SBNET_BF16) launch_wave<SBNET_BF16>(fused, form, l.nb, p, l.q, l.grid, l.lds, s);
    else launch_wave<SBNET_F16>(fused, form, l.nb, p, l.q, l.grid, l.lds, s);
    *st = launch_status(who);
    return true;
}

}  // namespace sbnet
