// Weight gradient of the tile convolution (training support for the convolution of Sec. 3.2 of arXiv 1801.02108):
//   dw[r][t][c][o] = sum over tiles b and output pixels (i, j) of x[b][r + sh i][t + sw j][c] * dout[b][i][j][o].
// The contraction runs over pixels, the one index that the channel-last tiles do not keep contiguous, and its result
// is small (kh kw Cin Cout numbers) while its inputs are the whole tile stacks.  So the tiles are split over many
// workgroups, each of which keeps a partial dw in registers for all its tiles and writes it once; a second kernel adds
// the partial results in a fixed order (no atomics: the result does not depend on scheduling).
//
// wgrad_tile (3x3, stride 1, BF16/F16, channel counts multiples of 8) and wgrad_run (1x1, stride 1; the tiles are one run of
// pixels): a workgroup owns 32 x 32 channels by nine taps, or 64 x 64.  Its four matrix waves split the PIXELS of a stage
// among them and add up through LDS at the end, so that a split's partial result costs a quarter of the workgroups it took
// when the waves split the channels: as many workgroups as CUs write 64 partial results of 64 -> 64 weights (9.4 MB) instead of
// up to 256.  Four more waves only move: tiles go from memory to LDS as they lie (buffer_load ... lds, two or three stages ahead,
// never through registers), and the matrix operands, which need eight consecutive pixels of one channel, are read with
// the transposing LDS read (ds_read_b64_tr_b16).  Segments of eight pixels pair up freely, so that rows are padded to 8 pixels
// instead of 16, and pixels beside the tile, rows past its end and channels past the last arrive as zeros by the buffer
// descriptor.  Bound on short lists by start and end (64 -> 64, 440 tiles of 16 x 16, seven stages a workgroup, counters: address unit
// busy 15 % of the time, matrix cores 13 %), on long ones by the wait for a stage: 2900 clocks for one of a 16 x 16 tile (19.1 ns a
// tile), 1300 of them the address unit's (37 copies, 35 clocks each) and 1150 the matrix cores'.
// Both launches, us, before (wgrad_mfma) and after: 3x3, 64 -> 64, tiles of 16 x 16: 165 tiles 22.9 -> 17.5, 440 24.7 -> 20.4; of
// 8 x 8: 440 26.0 -> 16.3; 32 -> 32, 12 x 12, 2200 tiles 50.8 -> 20.5; 96 -> 96, 16 x 16, 440 40.2 -> 33.2.  1x1: 256 -> 64 on 165 tiles of
// 18 x 18 15.0 -> 11.4, on 550 26.3 -> 22.6; 96 -> 24 on 550 23.7 -> 13.0.
//
// wgrad_mfma (long lists, 3x3 and 1x1 with a stride of 2; BF16/F16, channel counts multiples of 8): a workgroup owns 64 input by 64
// output channels, one 32x32 block per wave with one fp32 accumulator per tap (nine, or one).  Tiles pass through LDS a few output
// rows at a time (a "stage"), stored channel-major so that a lane's matrix operand (8 consecutive pixels of one
// channel) is one aligned 16-byte read:
//   * x rows are split by column phase (column % stride), so that the pixels a tap reads for consecutive output
//     pixels are consecutive; a tap's window starts 0 or 1 elements (stride 2) or 0, 1, 2 elements (stride 1) into a
//     16-byte vector and is cut from two neighbouring vectors with one byte-align per word;
//   * the channel planes are an odd number of 16-byte vectors apart and the vector index inside a plane is XOR-ed with
//     channel / 8: the 8-byte transposing writes of a wave (8 channel groups x 8 items of four pixels) and the
//     16-byte operand reads (consecutive channels) both spread over all banks; the spare vector at the end of each
//     plane takes the writes of staging slots that hold nothing, so that the writes need no branch;
//   * columns beyond the output row and rows beyond the tile hold zeros, in both operands, so that a partial row or
//     stage adds nothing.
// Stages alternate between two LDS buffers: the loads of the next stage are issued at the top of a stage, and in its
// second half their data, transposed in registers four pixels at a time, is written to the other buffer between the
// matrix instructions.
//
// wgrad_direct: every other shape and fp32; one thread per weight, plain loops.
#include <hip/hip_runtime.h>

#include "conv_common.h"

namespace sbnet {
namespace {

struct WgradParams {
    const void *x;            // [cap][th][tw][Cin]
    const void *g;            // [cap][oh][ow][Cout]
    float *part;              // [nsplit][taps][CinP][CoutP], split_stride() floats from one split to the next
    const int32_t *count;
    int cap, th, tw, oh, ow, Cin, Cout, kh, kw, sh, sw;
    int nsplit, ncb, nob, CinP, CoutP;
    int split_factor;         // splits used = min(nsplit, n, split_factor * sqrt(n))
    uint32_t x_tile_bytes, g_tile_bytes;
};

template <int KH, int S, int NSEG>
struct WgradShape {
    static constexpr int R = 8 / (S * NSEG);              // output rows per stage
    static constexpr int RX = (R - 1) * S + KH;           // input rows per stage
    // 16-byte vectors per phase row of x: 3x3 keeps one spare for the window of the taps; 1x1 reads 16 NSEG pixels only
    static constexpr int CPV = KH == 1 ? 2 * NSEG : 2 * NSEG + 1;
    static constexpr int XPL = (RX * S * CPV + 7) / 8 * 8;
    static constexpr int CSX = XPL + 1;                   // vectors between channel planes of x (odd)
    static constexpr int GV = 2 * NSEG;                   // vectors per row of dout
    static constexpr int GPL = (R * GV + 7) / 8 * 8;
    static constexpr int CSG = GPL + 1;
    static constexpr int XBYTES = 64 * CSX * 16;
    static constexpr int STAGE = 64 * (CSX + CSG) * 16;
    // staging items: four pixels of one phase row (or of one row of dout) times 8 channels
    static constexpr int QX = KH == 1 ? 4 * NSEG : (16 * NSEG + 2 + 3) / 4;    // items per phase row of x (at most 16 NSEG + KH - 1 pixels)
    static constexpr int QG = 4 * NSEG;                   // items per row of dout
    static constexpr int NIX = (RX * S * QX * 8 + 255) / 256;
    static constexpr int NIG = (R * QG * 8 + 255) / 256;
};

// Floats between the partial results of consecutive splits: the size of one result plus 256 bytes.  All workgroups
// write their results at the same time and at the same offsets inside them; with the bare size (a multiple of 16 KiB
// for 64 x 64 blocks) between them those writes would all fall on a few memory channels.
__host__ __device__ __forceinline__ size_t split_stride(int taps, int CinP, int CoutP) { return (size_t)taps * CinP * CoutP + 64; }

// Splits actually used for n active tiles, of the nsplit the launch provides.  Every split costs a partial result
// (written once, read once by the sum) and every tile of a split costs matrix time, so the best number grows with the
// square root of n: 8 sqrt(n) suits the two costs measured on 64 x 64 channel blocks.  Both kernels call this with
// the same arguments.
__device__ __forceinline__ int splits_used(int n, int nsplit, int factor) {
    int ns = (int)sqrtf((float)(factor * factor) * (float)n);     // factor: 8 for 3x3; a 1x1 partial result is a ninth of that: 16
    if (ns > n) ns = n;
    if (ns > nsplit) ns = nsplit;
    return ns < 1 ? 1 : ns;
}

__device__ __forceinline__ uint4 lds_read16(const char *p) { return *(const uint4 *)p; }

// elements 1..8 of the 16 elements in (v0, v1)
__device__ __forceinline__ uint4 window1(uint4 v0, uint4 v1) {
    return make_uint4(__builtin_amdgcn_alignbyte(v0.y, v0.x, 2), __builtin_amdgcn_alignbyte(v0.z, v0.y, 2),
                      __builtin_amdgcn_alignbyte(v0.w, v0.z, 2), __builtin_amdgcn_alignbyte(v1.x, v0.w, 2));
}
// elements 2..9
__device__ __forceinline__ uint4 window2(uint4 v0, uint4 v1) { return make_uint4(v0.y, v0.z, v0.w, v1.x); }

// two 16-bit halves, one from each word: (lo, lo) or (hi, hi)
__device__ __forceinline__ uint32_t pair_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pair_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

template <int DT, int KH, int S, int NSEG>
__global__ __launch_bounds__(256) void wgrad_mfma(WgradParams p) {
    typedef WgradShape<KH, S, NSEG> Sh;
    constexpr int TAPS = KH * KH;
    constexpr int R = Sh::R, RX = Sh::RX, CPV = Sh::CPV, CSX = Sh::CSX, CSG = Sh::CSG, GV = Sh::GV;
    constexpr int NIX = Sh::NIX, NIG = Sh::NIG, NI = NIX + NIG, QX = Sh::QX, QG = Sh::QG;
    extern __shared__ __align__(16) char lds[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sigma = blockIdx.x % p.nsplit, cbob = blockIdx.x / p.nsplit;
    const int cb = cbob / p.nob, ob = cbob - cb * p.nob;
    int n = *p.count;
    if (n > p.cap) n = p.cap;
    const int ns = splits_used(n, p.nsplit, p.split_factor);
    if (n <= 0 || sigma >= ns) return;                             // the sum reads no partial result of this split
    const int ntiles = (n - sigma + ns - 1) / ns;
    const int H = (p.oh + R - 1) / R;
    const int nstages = ntiles * H;

    // ---- what this thread stages, fixed for the whole kernel: items of four pixels (consecutive in a phase row of x,
    // or in a row of dout) by 8 channels = four 16-byte loads, transposed in registers into 8 writes of four pixels.
    // rel: byte offset of the first pixel inside the stage's first row (kOutOfRange: no item); cnt: pixels that exist.
    uint32_t rel[NI], at[NI], cnt[NI];
    const int cv = tid & 7;                                        // 8-channel group inside the workgroup's 64
#pragma unroll
    for (int u = 0; u < NIX; ++u) {
        const int it = (u * 256 + tid) >> 3;
        const int q = it % QX, rp = it / QX, ph = rp % S, ry = rp / S;
        const int x = 4 * q * S + ph;                              // column of the item's first pixel
        const bool ok = ry < RX && cb * 64 + cv * 8 < p.Cin && x < p.tw;
        rel[u] = ok ? (uint32_t)(((ry * p.tw + x) * p.Cin + cb * 64 + cv * 8) * 2) : kOutOfRange;
        cnt[u] = ok ? (uint32_t)((p.tw - x + S - 1) / S) : 0u;
        const uint32_t v = (uint32_t)((ry * S + ph) * CPV + (q >> 1)) ^ (uint32_t)cv;
        at[u] = (uint32_t)(cv * 8 * CSX * 16) + (ok ? v * 16 + (q & 1) * 8 : (uint32_t)Sh::XPL * 16);
    }
#pragma unroll
    for (int u = 0; u < NIG; ++u) {
        const int it = (u * 256 + tid) >> 3;
        const int q = it % QG, gy = it / QG, x = 4 * q;
        const bool ok = gy < R && ob * 64 + cv * 8 < p.Cout && x < p.ow;
        rel[NIX + u] = ok ? (uint32_t)(((gy * p.ow + x) * p.Cout + ob * 64 + cv * 8) * 2) : kOutOfRange;
        cnt[NIX + u] = ok ? (uint32_t)(p.ow - x) : 0u;
        const uint32_t v = (uint32_t)(gy * GV + (q >> 1)) ^ (uint32_t)cv;
        at[NIX + u] = (uint32_t)(Sh::XBYTES + cv * 8 * CSG * 16) + (ok ? v * 16 + (q & 1) * 8 : (uint32_t)Sh::GPL * 16);
    }
    const uint32_t x_stage_step = (uint32_t)(R * S * p.tw * p.Cin * 2), g_stage_step = (uint32_t)(R * p.ow * p.Cout * 2);
    const uint32_t x_px_step = (uint32_t)(S * p.Cin * 2), g_px_step = (uint32_t)(p.Cout * 2);

    uint4 staged[NI][4];
    auto issue = [&](int b, int h) {
        // one buffer descriptor per tile: offsets stay below the tile size whatever the size of the stack, and an
        // offset beyond the tile (a row past its last one) reads zeros by itself
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((const char *)p.x + (size_t)b * p.x_tile_bytes), 0, (int)p.x_tile_bytes, kBufWord3);
        const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(
            (void *)((const char *)p.g + (size_t)b * p.g_tile_bytes), 0, (int)p.g_tile_bytes, kBufWord3);
#pragma unroll
        for (int u = 0; u < NI; ++u) {
            const bool isx = u < NIX;
            const uint32_t o = (uint32_t)h * (isx ? x_stage_step : g_stage_step) + rel[u];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // pixels beyond the row's end (a slot that holds nothing has cnt = 0): zeros; so are, by the
                // descriptor, pixels beyond the tile (rows past its last one, the rest of a last row it does not fill)
                const uint32_t oj = o + j * (isx ? x_px_step : g_px_step);
                const uint32_t off = (uint32_t)j < cnt[u] ? oj : kOutOfRange;
                staged[u][j] = buf_load16(isx ? xr : gr, off);
            }
        }
    };
    // channel k of item u: its four pixels as one 8-byte write into channel plane k of the item's 8
    auto write_elem = [&](int w, char *base) {
        const int u = w >> 3, k = w & 7;
        uint32_t word[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint4 d = staged[u][j];
            word[j] = (k >> 1) == 0 ? d.x : (k >> 1) == 1 ? d.y : (k >> 1) == 2 ? d.z : d.w;
        }
        uint2 v;
        v.x = (k & 1) ? pair_hi(word[0], word[1]) : pair_lo(word[0], word[1]);
        v.y = (k & 1) ? pair_hi(word[2], word[3]) : pair_lo(word[2], word[3]);
        *(uint2 *)(base + at[u] + k * ((u < NIX ? CSX : CSG) * 16)) = v;
    };

    // ---- matrix operands of this wave ------------------------------------------------------------------------------
    const int cl = (wave >> 1) * 32 + (lane & 31), ol = (wave & 1) * 32 + (lane & 31), m = lane >> 5;
    const uint32_t swa = (uint32_t)(cl >> 3), swb = (uint32_t)(ol >> 3);
    const char *xplane = lds + cl * CSX * 16, *gplane = lds + Sh::XBYTES + ol * CSG * 16;
    f32x16 acc[TAPS];
#pragma unroll
    for (int k = 0; k < TAPS; ++k)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[k][e] = 0.f;

    // one step = 16 output pixels of one row (segment q of row i; q is the outer index so that consecutive steps share
    // input rows): the operand of dout and, per kernel row, the vectors the three taps are cut from.  A step reads
    // only the input rows the step before did not have.
    constexpr int T = R * NSEG, XV = S == 1 ? 2 : 3;
    struct Ops { uint4 b, x[KH][XV]; };
    auto load_row = [&](Ops &o, const char *xb, int i, int q, int r) {
        const uint32_t v = (uint32_t)((i * S + r) * S * CPV + 2 * q + m);          // phase 0 of the row
        o.x[r][0] = lds_read16(xb + (v ^ swa) * 16);
        if (KH == 1) return;                                                       // the one tap is vector 0
        o.x[r][1] = lds_read16(xb + ((v + 1) ^ swa) * 16);
        if (S == 2) o.x[r][XV - 1] = lds_read16(xb + ((v + CPV) ^ swa) * 16);      // phase 1
    };
    auto load_ops = [&](Ops &o, const Ops &prev, int bufno, int t) {
        const char *xb = xplane + bufno * Sh::STAGE, *gb = gplane + bufno * Sh::STAGE;
        const int q = t / R, i = t - q * R;
        o.b = lds_read16(gb + (((uint32_t)(i * GV + 2 * q + m)) ^ swb) * 16);
#pragma unroll
        for (int r = 0; r < KH; ++r) {
            if (i > 0 && r + S < KH) {
#pragma unroll
                for (int k = 0; k < XV; ++k) o.x[r][k] = prev.x[r + S][k];
            } else {
                load_row(o, xb, i, q, r);
            }
        }
    };
    auto mfma1 = [&](const Ops &o, int j) {                       // tap j = 3 r + t of this step
        const int r = j / KH, t = j - KH * r;
        uint4 a;
        if (S == 1) a = t == 0 ? o.x[r][0] : t == 1 ? window1(o.x[r][0], o.x[r][1]) : window2(o.x[r][0], o.x[r][1]);
        else a = t == 0 ? o.x[r][0] : t == 1 ? o.x[r][XV - 1] : window1(o.x[r][0], o.x[r][1]);
        acc[j] = mfma32x32x16<DT>(a, o.b, acc[j]);
    };

    // stages in order: (tile sigma, rows 0..R-1), (tile sigma, rows R..), ..., (tile sigma + ns, rows 0..), ...
    int b = sigma, h = 0, issued = 0;
    auto next_stage = [&]() {                                      // beyond the last stage: the last one again
        if (issued + 1 < nstages) {
            ++issued;
            if (++h == H) { h = 0; b += ns; }
        }
    };

    // ---- zero both buffers once: the padding is never written again ------------------------------------------------
    issue(b, h);
    for (int i = tid; i < 2 * Sh::STAGE / 16; i += 256) ((uint4 *)lds)[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < NI * 8; ++w) write_elem(w, lds);
    __syncthreads();
    for (int st = 0; st < nstages; ++st) {
        // loads of the next stage at the top; matrix work on buffer st % 2, the operands of a step read one step ahead;
        // in the second half of the stage the loaded items go to the other buffer, between the matrix instructions
        next_stage();
        issue(b, h);
        const int cur = st & 1;
        char *other = lds + (cur ^ 1) * Sh::STAGE;
        Ops o0, o1;
        load_ops(o0, o0, cur, 0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            Ops &now = (t & 1) ? o1 : o0, &nxt = (t & 1) ? o0 : o1;
            if (t + 1 < T) load_ops(nxt, now, cur, t + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < TAPS; ++j) {
                mfma1(now, j);
                constexpr int W = NI * 8, SLOTS = T * TAPS, FIRST = SLOTS / 2, LATE = SLOTS - FIRST;
                const int slot = t * TAPS + j - FIRST;
                if (slot >= 0) {
#pragma unroll
                    for (int w = (slot * W + LATE - 1) / LATE; w < ((slot + 1) * W + LATE - 1) / LATE; ++w) write_elem(w, other);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
    }

    // ---- partial result.  A lane holds column (output channel) lane % 32 and rows (input channels)
    // 8 (e / 4) + 4 (lane / 32) + e % 4 of its wave's 32 x 32 block; written like that, every store instruction would
    // carry 4 bytes per lane.  Each block goes through a wave-private LDS tile (the stage buffers are free now: the loop
    // ends with a barrier) and leaves as 16-byte stores along the output channels.
    float *out = p.part + (size_t)sigma * split_stride(TAPS, p.CinP, p.CoutP);
    constexpr int TS = 36;                                         // floats per tile row: 16-byte aligned rows, shifted banks
    float *tiles = (float *)lds + wave * (2 * 32 * TS);
    const int cblk = cb * 64 + (wave >> 1) * 32, oblk = ob * 64 + (wave & 1) * 32;
#pragma unroll
    for (int k = 0; k < TAPS; ++k) {
        float *t = tiles + (k & 1) * (32 * TS);
#pragma unroll
        for (int e = 0; e < 16; ++e) t[(8 * (e >> 2) + 4 * m + (e & 3)) * TS + (lane & 31)] = acc[k][e];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int pass = 0; pass < 4; ++pass) {
            const int row = pass * 8 + (lane >> 3), col = 4 * (lane & 7);
            const float4 v = *(const float4 *)(t + row * TS + col);
            *(float4 *)(out + ((size_t)k * p.CinP + cblk + row) * p.CoutP + oblk + col) = v;
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- 3x3, stride 1: 32 x 32 channels per workgroup
constexpr int kStageT = 48 * 1024;           // LDS bytes of a stage; three of them are also what the four waves' sums take
constexpr int kCopiesT = 12;                 // most 1 KB copies of a stage per moving wave

struct TilePlan {
    int R, tps;              // output rows of a stage; tiles of a stage (1 where a tile takes several stages)
    int slices;              // stages of a tile
    int spr, xp, gp;         // 8-pixel segments per output row; LDS pixels per row of x and of dout
    int x_copies, copies;    // 1 KB copies of a stage: of x, of both
    int steps;               // pairs of segments of a stage
    FastDiv div_xt, div_xp, div_gt, div_gp, div_spr, div_seg, div_slices;     // pixels per tile's rows and per row; segments per row and per tile
};

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) unsigned char lds_byte;
typedef short s16x4 __attribute__((ext_vector_type(4)));

// four pixels of one channel: lane l of a 16-lane group names pixel l / 4 and channels 4 (l % 4) .. + 3 and gets channel l
__device__ __forceinline__ uint2 read_tr(const lds_byte *p) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p));
}
__device__ __forceinline__ void wait_copies(int n) {     // until at most n of this wave's copies are on their way
    switch (n) {
#define SBNET_WAIT(N) case N: __builtin_amdgcn_s_waitcnt(0x0F70 | N); break
        SBNET_WAIT(1); SBNET_WAIT(2); SBNET_WAIT(3); SBNET_WAIT(4); SBNET_WAIT(5); SBNET_WAIT(6);
        SBNET_WAIT(7); SBNET_WAIT(8); SBNET_WAIT(9); SBNET_WAIT(10); SBNET_WAIT(11); SBNET_WAIT(12);
#undef SBNET_WAIT
        default: __builtin_amdgcn_s_waitcnt(0x0F70);
    }
}

template <int DT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void wgrad_tile(WgradParams p, TilePlan q) {
    extern __shared__ __align__(16) char lds[];
    lds_byte *const ldsb = (lds_byte *)lds;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sigma = blockIdx.x % p.nsplit, cbob = blockIdx.x / p.nsplit;
    const int cb = cbob / p.nob, ob = cbob - cb * p.nob;
    int n = *p.count;
    if (n > p.cap) n = p.cap;
    const int ns = splits_used(n, p.nsplit, p.split_factor);
    if (n <= 0 || sigma >= ns) return;
    // stages sigma, sigma + ns, ... of all: stage u is slice u % slices of tile u / slices, or tiles u tps .. + tps - 1
    const int total = q.tps > 1 ? (n + q.tps - 1) / q.tps : n * q.slices;
    const int nst = sigma < total ? (total - sigma + ns - 1) / ns : 0;

    if (wave >= 4) {
        // ---- moving: copy j of a stage is 16 pixels of 32 channels, 64 bytes each, linear in LDS; wave w moves copies w, w + 4, ...
        const int first = wave - 4;
        uint32_t rel[kCopiesT];                      // byte offset in the stage's first tile at its first row
#pragma unroll
        for (int i = 0; i < kCopiesT; ++i) {
            const int j = first + 4 * i;
            const bool isx = j < q.x_copies;
            const uint32_t px = (uint32_t)((isx ? j : j - q.x_copies) * 16 + (lane >> 2));
            const int ch = (isx ? cb : ob) * 32 + (lane & 3) * 8;
            const FastDiv dt = isx ? q.div_xt : q.div_gt, dp = isx ? q.div_xp : q.div_gp;
            const uint32_t t = fdiv(px, dt), in = px - t * dt.d, row = fdiv(in, dp), col = in - row * dp.d;
            const uint32_t w = isx ? p.tw : p.ow, h = isx ? p.th : p.oh, C = isx ? p.Cin : p.Cout;
            // (rows below a tile that is cut in slices are outside its descriptor)
            const bool ok = (int)t < q.tps && col < w && row < h && ch < (int)C;
            rel[i] = ok ? t * (isx ? p.x_tile_bytes : p.g_tile_bytes) + ((row * w + col) * C + ch) * 2u : kOutOfRange;
        }
        const int mine = (q.copies - first + 3) / 4;
        auto move = [&](int k) __attribute__((always_inline)) {         // the workgroup's stage k
            const uint32_t u = (uint32_t)(sigma + k * ns);
            const uint32_t b = q.tps > 1 ? u * q.tps : fdiv(u, q.div_slices);
            const uint32_t h = q.tps > 1 ? 0u : u - b * q.slices;
            const uint32_t tiles = q.tps > 1 ? min((uint32_t)n - b, (uint32_t)q.tps) : 1u;
            const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
                (void *)((const char *)p.x + (size_t)b * p.x_tile_bytes), 0, (int)(tiles * p.x_tile_bytes), kBufWord3);
            const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(
                (void *)((const char *)p.g + (size_t)b * p.g_tile_bytes), 0, (int)(tiles * p.g_tile_bytes), kBufWord3);
            const uint32_t xs = h * (uint32_t)(q.R * p.tw * p.Cin * 2), gs = h * (uint32_t)(q.R * p.ow * p.Cout * 2);
            lds_byte *to = ldsb + (k % 3) * kStageT;
#pragma unroll
            for (int i = 0; i < kCopiesT; ++i) {
                const int j = first + 4 * i;
                if (j < q.x_copies)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(to + j * 1024), 16, (int)(rel[i] + xs), 0, 0, 0);
                else if (j < q.copies)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(gr, (lds_void *)(to + j * 1024), 16, (int)(rel[i] + gs), 0, 0, 0);
            }
        };
        if (nst > 0) move(0);
        if (nst > 1) move(1);
        wait_copies(nst > 1 ? mine : 0);
        __builtin_amdgcn_s_barrier();
        for (int k = 0; k < nst; ++k) {
            if (k + 2 < nst) move(k + 2);
            __builtin_amdgcn_sched_barrier(0);
            wait_copies(k + 2 < nst ? mine : 0);     // stage k + 1 has landed
            __builtin_amdgcn_s_barrier();
        }
        __syncthreads();                             // (the sums below)
    } else {
        f32x16 acc[9];
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[k][e] = 0.f;
        // ---- matrix steps: step s takes segments 2 s (lanes 0..31) and 2 s + 1 of the stage, wave w steps w, w + 4, ...
        const uint32_t lane_at = (uint32_t)(((lane & 15) >> 2) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
        struct Ops { uint2 g[2], x[3][3]; };
        auto load = [&](Ops &o, const lds_byte *st, int s) __attribute__((always_inline)) {
            const uint32_t seg = (uint32_t)(2 * s + (lane >> 5));
            const uint32_t t = fdiv(seg, q.div_seg), in = seg - t * q.div_seg.d, row = fdiv(in, q.div_spr), c = in - row * q.div_spr.d;
            const lds_byte *gp = st + q.x_copies * 1024 + (t * q.div_gt.d + row * q.gp + c * 8) * 64 + lane_at;
            const lds_byte *xp = st + (t * q.div_xt.d + row * q.xp + c * 8) * 64 + lane_at;
#pragma unroll
            for (int k = 0; k < 2; ++k) o.g[k] = read_tr(gp + k * 256);
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int k = 0; k < 3; ++k) o.x[r][k] = read_tr(xp + r * q.xp * 64 + k * 256);
        };
        auto step = [&](const Ops &o) __attribute__((always_inline)) {
            const uint4 b = make_uint4(o.g[0].x, o.g[0].y, o.g[1].x, o.g[1].y);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                const uint4 v0 = make_uint4(o.x[r][0].x, o.x[r][0].y, o.x[r][1].x, o.x[r][1].y);
                const uint4 v1 = make_uint4(o.x[r][2].x, o.x[r][2].y, 0u, 0u);
                acc[3 * r] = mfma32x32x16<DT>(v0, b, acc[3 * r]);
                acc[3 * r + 2] = mfma32x32x16<DT>(window2(v0, v1), b, acc[3 * r + 2]);
                acc[3 * r + 1] = mfma32x32x16<DT>(window1(v0, v1), b, acc[3 * r + 1]);
            }
        };
        __syncthreads();                             // stage 0
        for (int k = 0; k < nst; ++k) {
            const lds_byte *st = ldsb + (k % 3) * kStageT;
            Ops o0, o1;
            if (wave < q.steps) load(o0, st, wave);
            for (int s = wave; s < q.steps; s += 8) {
                if (s + 4 < q.steps) load(o1, st, s + 4);
                __builtin_amdgcn_sched_barrier(0);
                step(o0);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 4 < q.steps) {
                    if (s + 8 < q.steps) load(o0, st, s + 8);
                    __builtin_amdgcn_sched_barrier(0);
                    step(o1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __syncthreads();
        }
        // ---- the four waves' sums (each over its own pixels) through LDS, [wave][tap][input channel][output channel]
        float *mine = (float *)lds + wave * (9 * 1024);
#pragma unroll
        for (int k = 0; k < 9; ++k)
#pragma unroll
            for (int e = 0; e < 16; ++e) mine[k * 1024 + (8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 32 + (lane & 31)] = acc[k][e];
        __syncthreads();
    }
    // added in the order of the waves and written as the split's partial result
    float *out = p.part + (size_t)sigma * split_stride(9, p.CinP, p.CoutP);
    for (int i = threadIdx.x; i < 9 * 256; i += 512) {
        const float4 *a = (const float4 *)lds + i;
        const float4 v0 = a[0], v1 = a[9 * 256], v2 = a[2 * 9 * 256], v3 = a[3 * 9 * 256];
        const float4 v = make_float4(((v0.x + v1.x) + v2.x) + v3.x, ((v0.y + v1.y) + v2.y) + v3.y, ((v0.z + v1.z) + v2.z) + v3.z,
                                     ((v0.w + v1.w) + v2.w) + v3.w);
        const int tap = i >> 8, row = (i >> 3) & 31, col = (i & 7) * 4;
        *(float4 *)(out + ((size_t)tap * p.CinP + cb * 32 + row) * p.CoutP + ob * 32 + col) = v;
    }
}

// ---- 1x1, stride 1: 64 x 64 channels per workgroup; the tiles are one run of pixels, whatever their shape
constexpr int kRunPx = 128;                  // pixels of a stage: 16 KB of x and 16 KB of dout
constexpr int kRunStage = 2 * kRunPx * 128;
constexpr int kRunDepth = 4;                 // LDS buffers

template <int DT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void wgrad_run(WgradParams p) {
    extern __shared__ __align__(16) char lds[];
    lds_byte *const ldsb = (lds_byte *)lds;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sigma = blockIdx.x % p.nsplit, cbob = blockIdx.x / p.nsplit;
    const int cb = cbob / p.nob, ob = cbob - cb * p.nob;
    int n = *p.count;
    if (n > p.cap) n = p.cap;
    const int ns = splits_used(n, p.nsplit, p.split_factor);
    if (n <= 0 || sigma >= ns) return;
    const long long px = (long long)n * p.th * p.tw;
    const int total = (int)((px + kRunPx - 1) / kRunPx);
    const int nst = sigma < total ? (total - sigma + ns - 1) / ns : 0;          // stages sigma, sigma + ns, ...

    if (wave >= 4) {
        // ---- moving: a copy is 8 pixels of 64 channels, 128 bytes each; piece k of pixel q lies at place k ^ 4 (q / 2 % 2), which
        //      spreads the four pixels of a transposing read over all banks.  Wave w moves every fourth copy.
        constexpr int N = kRunPx / 8 / 4;            // copies of either operand per wave and stage
        const int q = (wave - 4) * 8 + (lane >> 3);
        const int ch = ((lane & 7) ^ (((q >> 1) & 1) << 2)) * 8;
        const uint32_t xrel = cb * 64 + ch < p.Cin ? (uint32_t)(q * p.Cin + cb * 64 + ch) * 2u : kOutOfRange;
        const uint32_t grel = ob * 64 + ch < p.Cout ? (uint32_t)(q * p.Cout + ob * 64 + ch) * 2u : kOutOfRange;
        auto move = [&](int k) __attribute__((always_inline)) {
            const long long at = (long long)(sigma + (long long)k * ns) * kRunPx;
            const uint32_t here = (uint32_t)min((long long)kRunPx, px - at);     // pixels beyond the run are outside the descriptors
            const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
                (void *)((const char *)p.x + at * p.Cin * 2), 0, (int)(here * p.Cin * 2u), kBufWord3);
            const __amdgpu_buffer_rsrc_t gr = __builtin_amdgcn_make_buffer_rsrc(
                (void *)((const char *)p.g + at * p.Cout * 2), 0, (int)(here * p.Cout * 2u), kBufWord3);
            lds_byte *to = ldsb + (k % kRunDepth) * kRunStage + (wave - 4) * 1024;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_void *)(to + i * 4096), 16, (int)(xrel + (uint32_t)i * 64u * p.Cin), 0, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(gr, (lds_void *)(to + kRunPx * 128 + i * 4096), 16,
                                                         (int)(grel + (uint32_t)i * 64u * p.Cout), 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // (stages past the last one are not requested: then everything is waited for)
        auto wait = [&](int k) __attribute__((always_inline)) {                  // until stage k has landed, k + 1 and k + 2 behind it
            if (k + 2 < nst) __builtin_amdgcn_s_waitcnt(0x0F70 | ((4 * N) & 15) | (((4 * N) >> 4) << 14));
            else if (k + 1 < nst) __builtin_amdgcn_s_waitcnt(0x0F70 | ((2 * N) & 15) | (((2 * N) >> 4) << 14));
            else __builtin_amdgcn_s_waitcnt(0x0F70);
        };
        for (int k = 0; k < 3 && k < nst; ++k) move(k);
        wait(0);
        __builtin_amdgcn_s_barrier();
        for (int k = 0; k < nst; ++k) {
            if (k + 3 < nst) move(k + 3);
            wait(k + 1);
            __builtin_amdgcn_s_barrier();
        }
        __syncthreads();                             // (the sums below)
    } else {
        f32x16 acc[2][2];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
        const int l16 = lane & 15;
        uint32_t at[2];                              // this lane's part of a read of channels 32 h .. + 31
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int piece = (h * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ ((l16 >> 3) << 2);
            at[h] = (uint32_t)(((lane >> 5) * 8 + (l16 >> 2)) * 128 + piece * 16 + (lane & 1) * 8);
        }
        __syncthreads();                             // stage 0
        for (int k = 0; k < nst; ++k) {
            const lds_byte *st = ldsb + (k % kRunDepth) * kRunStage + wave * 2 * 2048;
#pragma unroll
            for (int s = 0; s < 2; ++s) {            // 16 pixels each
                uint4 x[2], g[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const lds_byte *a = st + s * 2048 + at[h], *b = a + kRunPx * 128;
                    const uint2 a0 = read_tr(a), a1 = read_tr(a + 512), b0 = read_tr(b), b1 = read_tr(b + 512);
                    x[h] = make_uint4(a0.x, a0.y, a1.x, a1.y);
                    g[h] = make_uint4(b0.x, b0.y, b1.x, b1.y);
                }
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) acc[a][b] = mfma32x32x16<DT>(x[a], g[b], acc[a][b]);
            }
            __syncthreads();
        }
        // ---- the four waves' sums (each over its own pixels) through LDS, [wave][input channel][output channel]
        float *mine = (float *)lds + wave * 4096;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    mine[(a * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 64 + b * 32 + (lane & 31)] = acc[a][b][e];
        __syncthreads();
    }
    float *out = p.part + (size_t)sigma * split_stride(1, p.CinP, p.CoutP);
    for (int i = threadIdx.x; i < 1024; i += 512) {
        const float4 *a = (const float4 *)lds + i;
        const float4 v0 = a[0], v1 = a[1024], v2 = a[2048], v3 = a[3072];
        const float4 v = make_float4(((v0.x + v1.x) + v2.x) + v3.x, ((v0.y + v1.y) + v2.y) + v3.y, ((v0.z + v1.z) + v2.z) + v3.z,
                                     ((v0.w + v1.w) + v2.w) + v3.w);
        *(float4 *)(out + (size_t)(cb * 64 + (i >> 4)) * p.CoutP + ob * 64 + (i & 15) * 4) = v;
    }
}

template <int DT>
__device__ __forceinline__ float load_elem(const void *p, size_t i) {
    if (DT == SBNET_F32) return ((const float *)p)[i];
    const uint32_t bits = ((const uint16_t *)p)[i];
    return DT == SBNET_BF16 ? bf16_bits_to_float(bits) : unpack_lo<SBNET_F16>(bits);
}

// one thread per weight (tap, c, o); blockIdx.y is the split
template <int DT>
__global__ __launch_bounds__(256) void wgrad_direct(WgradParams p) {
    const int total = p.kh * p.kw * p.Cin * p.Cout;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= total) return;
    int n = *p.count;
    if (n > p.cap) n = p.cap;
    const int sigma = blockIdx.y, ns = splits_used(n, p.nsplit, p.split_factor);
    if (n <= 0 || sigma >= ns) return;
    const int o = e % p.Cout, c = (e / p.Cout) % p.Cin, tap = e / (p.Cout * p.Cin);
    const int r = tap / p.kw, t = tap - r * p.kw;
    float acc = 0.f;
    for (int b = sigma; b < n; b += ns) {
        for (int i = 0; i < p.oh; ++i) {
            const size_t xrow = ((size_t)b * p.th + r + (size_t)p.sh * i) * p.tw + t;
            const size_t grow = ((size_t)b * p.oh + i) * p.ow;
            for (int j = 0; j < p.ow; ++j)
                acc = fmaf(load_elem<DT>(p.x, (xrow + (size_t)p.sw * j) * p.Cin + c), load_elem<DT>(p.g, (grow + j) * p.Cout + o), acc);
        }
    }
    p.part[(size_t)sigma * split_stride(p.kh * p.kw, p.CinP, p.CoutP) + e] = acc;
}

// dw[tap][c][o] = partial results of the splits that had a tile, added in a fixed order: the NW waves of a workgroup
// each add every NW-th split in ascending order (many independent loads in flight, where one chain of dependent
// loads would be bound by latency), then the NW sums are added in ascending order of the wave.  NW = 16 where the
// weights fill at most 256 workgroups (1x1 kernels: the launch is short and the splits are many), else 4.
template <int NW>
__global__ __launch_bounds__(64 * NW) void wgrad_sum(const float *__restrict__ part, const int32_t *__restrict__ count, int cap,
                                                  int nsplit, int split_factor, int taps, int Cin, int Cout, int CinP,
                                                  int CoutP, float *__restrict__ dw) {
    __shared__ float slice[NW][64];
    const int total = taps * Cin * Cout;
    const int lane = threadIdx.x & 63, k = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;
    int n = *count;
    if (n > cap) n = cap;
    n = n > 0 ? splits_used(n, nsplit, split_factor) : 0;
    float acc = 0.f;
    if (e < total) {
        const int o = e % Cout, c = (e / Cout) % Cin, tap = e / (Cout * Cin);
        const size_t at = ((size_t)tap * CinP + c) * CoutP + o, step = split_stride(taps, CinP, CoutP);
        // batches of 8 loads in flight (splits beyond the last read as the first one and count as zero)
        for (int s = k; s < n; s += 8 * NW) {
            float a[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int sj = s + NW * j;
                const float v = part[at + (size_t)(sj < n ? sj : 0) * step];
                a[j] = sj < n ? v : 0.f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) acc += a[j];
        }
    }
    slice[k][lane] = acc;
    __syncthreads();
    if (k == 0 && e < total) {
        float t = slice[0][lane];
#pragma unroll
        for (int i = 1; i < NW; ++i) t += slice[i][lane];
        dw[e] = t;
    }
}

struct WgradPlan {
    bool mfma;
    int kh, s, nseg, nsplit, ncb, nob, CinP, CoutP;
    bool flat;               // 1x1 at stride 1: the tile as one run of pixels
    bool run;                // ... by wgrad_run
    bool tile;               // wgrad_tile, with t
    TilePlan t;
    size_t part_bytes;
};

// 3x3 stride 1: false where a stage does not hold a row of outputs
bool plan_tile(int th, int tw, int oh, int ow, TilePlan *t) {
    const int spr = (ow + 7) / 8, gp = 8 * spr, xp = gp + 2;
    auto x_bytes = [&](long long rows, int tps) { return (tps * (rows + 2) * xp * 64 + 1023) / 1024 * 1024; };
    auto g_bytes = [&](long long rows, int tps) { return (tps * rows * gp * 64 + 1023) / 1024 * 1024; };
    auto fits = [&](long long rows, int tps) {
        // (a fragment's last read goes up to 128 bytes beyond the rows of x, into those of dout)
        return x_bytes(rows, tps) + g_bytes(rows, tps) <= kStageT && (x_bytes(rows, tps) + g_bytes(rows, tps)) / 1024 <= 4 * kCopiesT;
    };
    int R = spr % 2 ? (oh + 1) / 2 * 2 : oh;               // an even number of segments
    t->tps = 1;
    if (fits(R, 1)) {
        while (t->tps < 4 && fits(R, t->tps + 1)) ++t->tps;
    } else {
        const int unit = spr % 2 ? 2 : 1;
        R = R / unit * unit;
        while (R > 0 && !fits(R, 1)) R -= unit;
        if (R <= 0) return false;
        const int slices = (oh + R - 1) / R;               // slices of about the same height
        R = ((oh + slices - 1) / slices + unit - 1) / unit * unit;
    }
    t->R = R;
    t->slices = (oh + R - 1) / R;
    t->spr = spr;
    t->xp = xp;
    t->gp = gp;
    t->x_copies = (int)(x_bytes(R, t->tps) / 1024);
    t->copies = t->x_copies + (int)(g_bytes(R, t->tps) / 1024);
    t->steps = t->tps * R * spr / 2;
    t->div_xt = make_fastdiv((uint32_t)((R + 2) * xp));
    t->div_xp = make_fastdiv((uint32_t)xp);
    t->div_gt = make_fastdiv((uint32_t)(R * gp));
    t->div_gp = make_fastdiv((uint32_t)gp);
    t->div_spr = make_fastdiv((uint32_t)spr);
    t->div_seg = make_fastdiv((uint32_t)(R * spr));
    t->div_slices = make_fastdiv((uint32_t)t->slices);
    return true;
}

bool plan_wgrad(sbnet_dtype dt, int cap, int th, int tw, int Cin, int kh, int kw, int sh, int sw, int Cout, WgradPlan *q) {
    const int oh = (th - kh) / sh + 1, ow = (tw - kw) / sw + 1;
    const int taps = kh * kw;
    q->flat = kh == 1 && kw == 1 && sh == 1 && sw == 1;
    q->mfma = (dt == SBNET_BF16 || dt == SBNET_F16) && (kh == 3 || kh == 1) && kw == kh && sh == sw && (sh == 1 || sh == 2) && Cin % 8 == 0 &&
              Cout % 8 == 0 && (q->flat || (ow <= 32 && tw <= 32 * sw + 2)) &&
              (long long)th * tw * Cin * 2 < (1LL << 30) && (long long)oh * ow * Cout * 2 < (1LL << 30);
    q->kh = kh;
    q->tile = (dt == SBNET_BF16 || dt == SBNET_F16) && kh == 3 && kw == 3 && sh == 1 && sw == 1 && Cin % 8 == 0 && Cout % 8 == 0 &&
              4LL * th * tw * Cin * 2 < (1LL << 30) && 4LL * oh * ow * Cout * 2 < (1LL << 30) &&
              plan_tile(th, tw, oh, ow, &q->t);
    if (q->tile && q->mfma) {
        // Long lists of tiles that 64 x 64 blocks and 16-pixel rows fit: wgrad_mfma, which stages a pixel once for twice the
        // channels (64 -> 64, tiles of 16 x 16: 14.1 ns a tile against 19.1), though it starts and ends slower (its partial
        // results are two to four times as many bytes): us by it and by wgrad_tile, 440 tiles 24.7 and 20.4, 2200 49.6 and
        // 54.1; 128 -> 128, 165 tiles 27.5 and 25.6, 440 42.6 and 46.1; 256 -> 256, 60 tiles 37.7 and 37.7, 440 125 and 155.  The
        // line lies at 1000 tiles of 256 pixels by the number of 64 x 64 blocks.  Where more than a fifth of its work is
        // padding wgrad_tile wins on lists up to four times as long (224 -> 224, 16 x 16, 110 tiles 47.6 and 48.8, at 44 of them
        // 34.4 and 31.5; 440 130 and 143, 62.4 and 67.1; 2200 570 and 625), and where nearly a quarter is at any length (2200 tiles:
        // 96 -> 96 147 and 116, 32 -> 32 46.7 and 24.0, 64 -> 64 of 8 x 8 35.2 and 22.7, of 24 x 24 142 and 135; 512 -> 512, 12 x 12,
        // 2126 and 2112).
        const long long p64 = (long long)((Cin + 63) / 64) * ((Cout + 63) / 64), p32 = (long long)((Cin + 31) / 32) * ((Cout + 31) / 32);
        const long long px16 = ow <= 16 ? (oh + 7LL) / 8 * 8 * 16 : (oh + 3LL) / 4 * 4 * 32, px8 = (long long)q->t.slices * q->t.R * q->t.gp;
        const long long work8 = p32 * px8 * 100, work16 = p64 * 4 * px16, most = work8 >= work16 * 80 ? 1000 : 4000;
        if (work8 >= work16 * 76 && (long long)cap * oh * ow * p64 > most * 256) q->tile = false;
    }
    const long long p64 = (long long)((Cin + 63) / 64) * ((Cout + 63) / 64), px = (long long)th * tw;
    // 1x1: past these lengths, in tiles of 256 pixels, several channel blocks read their operands from memory again, and wgrad_mfma
    // with its two workgroups per CU waits less.  us by it and by wgrad_run, 16 x 16, 40 % of the bound active and all: 64 -> 96, 3500
    // tiles 26.7 23.8, 60.3 60.2, 5000 38.0 35.6, 80.7 88.0, 8800 59.2 62.3, 135 170; 256 -> 256, 2200 80.1 78.2, 189 181, 3500 118 120,
    // 281 292, 8800 293 286, 698 766; 160 -> 160, 1760 50.6 33.3, 105 113, 3500 83.5 92.8, 191 221; 512 -> 512, 300 42.4 34.7, 99 100,
    // 700 90.8 92.6, 212 230, 2200 265 296, 638 816; 384 -> 384, 700 73.7 58.5, 186 189, 1200 130 122, 310 366.  At a tenth active wgrad_run
    // is 5 to 30 % the faster everywhere.  One channel block (64 -> 64 47.9 45.0, 106 99 at 8800) and tiles that leave a tenth of
    // wgrad_mfma's stages of 128 pixels empty (18 x 18, 128 -> 128, 5500 84.4 69.1, 190 174): wgrad_run at any length.
    const long long most1 = p64 > 16 ? 700 : p64 > 4 ? 3000 : 4000;
    q->run = q->flat && !(p64 >= 2 && px * 10 >= (px + 127) / 128 * 128 * 9 && (long long)cap * px > most1 * 256);
    if (q->tile) {
        q->s = q->nseg = 1;
        q->ncb = (Cin + 31) / 32;
        q->nob = (Cout + 31) / 32;
        q->CinP = q->ncb * 32;
        q->CoutP = q->nob * 32;
        q->nsplit = 256 / (q->ncb * q->nob);               // one workgroup per CU
        if (q->nsplit > 8) q->nsplit = q->nsplit / 8 * 8;  // splits of one channel block share an XCD's L2 with the others
        if (q->nsplit < 1) q->nsplit = 1;
    } else if (q->mfma) {
        q->s = sh;
        q->nseg = q->flat || (ow <= 16 && tw <= 16 * sw + 2) ? 1 : 2;
        q->ncb = (Cin + 63) / 64;
        q->nob = (Cout + 63) / 64;
        q->CinP = q->ncb * 64;
        q->CoutP = q->nob * 64;
        // one workgroup per CU for 3x3 (its two stages take 100 KB of LDS) and wgrad_run (its four 128 KB); two for 1x1
        // otherwise (70 KB), whose stages hold little matrix work and wait on memory: the second workgroup's loads fill that wait
        int ns = (kh == 1 && !q->run ? 512 : 256) / (q->ncb * q->nob);
        ns = ns / 8 * 8;                                   // splits of one channel block share an XCD's L2 with the others
        if (ns < 8) ns = 8;
        q->nsplit = ns;
    } else {
        q->s = q->nseg = 0;
        q->ncb = q->nob = 1;
        q->CinP = Cin;
        q->CoutP = Cout;
        const long long e = (long long)taps * Cin * Cout;
        if (e >= (1LL << 31)) return false;
        long long ns = (256LL * 1024 + e - 1) / e;
        if (ns > 1024) ns = 1024;
        q->nsplit = (int)ns;
    }
    if (q->nsplit > cap) q->nsplit = cap < 1 ? 1 : cap;
    q->part_bytes = (size_t)q->nsplit * split_stride(taps, q->CinP, q->CoutP) * sizeof(float);
    return true;
}

template <int DT, int KH, int S, int NSEG>
void launch_mfma(const WgradParams &p, hipStream_t s) {
    constexpr int bytes = 2 * WgradShape<KH, S, NSEG>::STAGE;
    static_assert(bytes <= 160 * 1024, "two stages must fit in LDS");
    (void)hipFuncSetAttribute((const void *)wgrad_mfma<DT, KH, S, NSEG>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    hipLaunchKernelGGL((wgrad_mfma<DT, KH, S, NSEG>), dim3(p.nsplit * p.ncb * p.nob), dim3(256), bytes, s, p);
}

template <int DT>
void launch_mfma_dt(const WgradPlan &q, const WgradParams &p, hipStream_t s) {
    if (q.run) {
        constexpr int bytes = kRunDepth * kRunStage;
        static_assert(bytes >= 4 * 4096 * 4 && bytes <= 160 * 1024, "the stages; the four waves' sums");
        (void)hipFuncSetAttribute((const void *)wgrad_run<DT>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        hipLaunchKernelGGL(wgrad_run<DT>, dim3(p.nsplit * p.ncb * p.nob), dim3(512), bytes, s, p);
        return;
    }
    if (q.tile) {
        constexpr int bytes = 3 * kStageT;
        static_assert(bytes >= 4 * 9 * 1024 * 4 && bytes <= 160 * 1024, "three stages; the four waves' sums");
        (void)hipFuncSetAttribute((const void *)wgrad_tile<DT>, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        hipLaunchKernelGGL(wgrad_tile<DT>, dim3(p.nsplit * p.ncb * p.nob), dim3(512), bytes, s, p, q.t);
        return;
    }
    if (q.kh == 3) {
        if (q.s == 1 && q.nseg == 1) launch_mfma<DT, 3, 1, 1>(p, s);
        else if (q.s == 1) launch_mfma<DT, 3, 1, 2>(p, s);
        else if (q.nseg == 1) launch_mfma<DT, 3, 2, 1>(p, s);
        else launch_mfma<DT, 3, 2, 2>(p, s);
    } else if (q.flat) {
        launch_mfma<DT, 1, 1, 1>(p, s);
    } else if (q.nseg == 1) {
        launch_mfma<DT, 1, 2, 1>(p, s);
    } else {
        launch_mfma<DT, 1, 2, 2>(p, s);
    }
}

}  // namespace

extern "C" size_t sbnet_conv_backward_weights_workspace_bytes(sbnet_dtype dtype, int cap, int th, int tw, int Cin, int kh,
                                                              int kw, int sh, int sw, int Cout) {
    if (!is_float_dtype(dtype) || cap < 0 || th < kh || tw < kw || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || Cin <= 0 ||
        Cout <= 0)
        return 0;
    WgradPlan q;
    if (!plan_wgrad(dtype, cap, th, tw, Cin, kh, kw, sh, sw, Cout, &q)) return 0;
    return (q.part_bytes + 255) / 256 * 256;
}

extern "C" sbnet_status sbnet_conv_on_tiles_backward_weights(const void *tiles_in, const void *dout_tiles, sbnet_dtype dtype,
                                                             const int32_t *count, int cap, int th, int tw, int Cin, int kh,
                                                             int kw, int sh, int sw, int Cout, float *dw, void *workspace,
                                                             size_t workspace_bytes, void *stream) {
    const char *who = "sbnet_conv_on_tiles_backward_weights";
    if (!tiles_in || !dout_tiles || !count || !dw || !workspace) return fail(SBNET_EINVAL, "%s: null pointer", who);
    if (!is_float_dtype(dtype)) return fail(SBNET_EUNSUPPORTED, "%s: dtype must be f32, bf16 or f16", who);
    if (cap < 0 || Cin <= 0 || Cout <= 0 || kh <= 0 || kw <= 0 || sh <= 0 || sw <= 0 || th < kh || tw < kw)
        return fail(SBNET_EINVAL, "%s: bad sizes", who);
    if (((uintptr_t)tiles_in | (uintptr_t)dout_tiles | (uintptr_t)workspace) & 15)
        return fail(SBNET_EINVAL, "%s: pointers must be 16-byte aligned", who);
    WgradPlan q;
    if (!plan_wgrad(dtype, cap, th, tw, Cin, kh, kw, sh, sw, Cout, &q)) return fail(SBNET_EUNSUPPORTED, "%s: too many weights", who);
    if (workspace_bytes < q.part_bytes) return fail(SBNET_EINVAL, "%s: workspace too small", who);
    hipStream_t s = (hipStream_t)stream;
    const int taps = kh * kw, total = taps * Cin * Cout;
    WgradParams p = {};
    p.x = tiles_in; p.g = dout_tiles; p.part = (float *)workspace; p.count = count;
    p.cap = cap; p.th = th; p.tw = tw; p.oh = (th - kh) / sh + 1; p.ow = (tw - kw) / sw + 1;
    p.Cin = Cin; p.Cout = Cout; p.kh = kh; p.kw = kw; p.sh = sh; p.sw = sw;
    p.nsplit = q.nsplit; p.ncb = q.ncb; p.nob = q.nob; p.CinP = q.CinP; p.CoutP = q.CoutP;
    const sbnet_tuning tune = tuning();
    p.split_factor = taps == 1 ? tune.wgrad_split_factor_1x1 : tune.wgrad_split_factor_3x3;
    p.x_tile_bytes = (uint32_t)((size_t)th * tw * Cin * 2);
    p.g_tile_bytes = (uint32_t)((size_t)p.oh * p.ow * Cout * 2);
    if (q.mfma && q.flat && !q.run) {
        // 1x1 at stride 1 pairs pixel with pixel, whatever the tile's shape: wgrad_mfma sees rows of 16 pixels
        // (the tile sizes in bytes stay the true ones, so the pixels past the end of the last row read as zeros)
        p.th = p.oh = (th * tw + 15) / 16;
        p.tw = p.ow = 16;
    }
    if (cap > 0) {
        if (q.mfma || q.tile) {
            if (dtype == SBNET_BF16) launch_mfma_dt<SBNET_BF16>(q, p, s);
            else launch_mfma_dt<SBNET_F16>(q, p, s);
        } else {
            dim3 grid((unsigned)((total + 255) / 256), (unsigned)q.nsplit);
            if (dtype == SBNET_F32) hipLaunchKernelGGL(wgrad_direct<SBNET_F32>, grid, dim3(256), 0, s, p);
            else if (dtype == SBNET_BF16) hipLaunchKernelGGL(wgrad_direct<SBNET_BF16>, grid, dim3(256), 0, s, p);
            else hipLaunchKernelGGL(wgrad_direct<SBNET_F16>, grid, dim3(256), 0, s, p);
        }
        sbnet_status st = launch_status(who);
        if (st != SBNET_OK) return st;
    }
    const unsigned sum_grid = (unsigned)((total + 63) / 64);
    if (sum_grid <= 256)
        hipLaunchKernelGGL(wgrad_sum<16>, dim3(sum_grid), dim3(1024), 0, s, (const float *)workspace, count, cap, q.nsplit, p.split_factor,
                           taps, Cin, Cout, q.CinP, q.CoutP, dw);
    else
        hipLaunchKernelGGL(wgrad_sum<4>, dim3(sum_grid), dim3(256), 0, s, (const float *)workspace, count, cap, q.nsplit, p.split_factor,
                           taps, Cin, Cout, q.CinP, q.CoutP, dw);
    return launch_status(who);
}

}  // namespace sbnet
