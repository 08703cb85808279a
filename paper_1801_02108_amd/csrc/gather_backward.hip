// Gradient of the overlapping gather (end of Sec. 3.3 of arXiv 1801.02108, "End-to-end training of SBNet"): the
// gradient of a gather is a scatter-add of the tile gradients, and because neighbouring tiles share their halo, a
// pixel on a tile edge receives contributions from up to four tiles.  (The gradient of the scatter is the plain
// gather and needs no kernel of its own.)
//
// The paper adds with atomics.  Here the sum is pulled instead of pushed: a small map from block coordinates to
// the block's position in the index list is built first, then every pixel's contributions are added in ascending
// (by, bx) order, in fp32, onto dx, rounding once.  No atomics, results do not depend on scheduling, every dx vector
// is read and written once, whole vectors.  Two kernels do that:
//   gb_tiles       tiles that reach over at most one following block per axis (any 3x3, blocks of at least half the
//                  kernel otherwise): work items are pieces of active tiles; a pixel that several tiles cover belongs
//                  to the first of them.
//   gb_cells       tiles that reach further, and dense lists of small cells: work items are cells of the block grid
//                  (bstride_h x bstride_w pixels), each looking up the at most (R+1)^2 tiles that can cover it,
//                  R = ceil((bsize - bstride) / bstride).
// gb_either holds both and lets the device-side count pick; gb_near and gb_far go by cells only.
#include "tile_add.h"

namespace sbnet {

constexpr int kGbThreads = 256;
constexpr int kGbMaxR = 3;       // tiles may reach over at most three following cells per axis

struct GbParams {
    sbnet_geom g;
    int N, H, W, cap;
    int cells_h, cells_w;        // cells that a tile can touch: bcount + R
    int R_h, R_w;
    uint32_t pix_vecs;           // vectors per pixel
    uint32_t cell_vecs;          // vectors per cell: bstride_h * bstride_w * pix_vecs
    uint32_t row_vecs;           // vectors per cell row: bstride_w * pix_vecs
    uint32_t tile_row_vecs;      // vectors per tile row: bsize_w * pix_vecs
    uint32_t tile_vecs;
    FastDiv div_cells, div_cw, div_row, div_pv;
};

__global__ void gb_map_clear(int32_t *map, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) map[i] = -1;
}

__global__ void gb_map_fill(int32_t *map, const int32_t *__restrict__ indices, const int32_t *__restrict__ count,
                            int cap, int N, int bh, int bw) {
    const int nact = min(*count, cap);
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < nact; b += gridDim.x * blockDim.x) {
        const int n = indices[3 * b], by = indices[3 * b + 1], bx = indices[3 * b + 2];
        if (n >= 0 && n < N && by >= 0 && by < bh && bx >= 0 && bx < bw) map[(n * bh + by) * bw + bx] = b;
    }
}

// both steps in one workgroup (one launch less) when the map and the list are small enough for it
__global__ __launch_bounds__(1024) void gb_map_build(int32_t *map, int nmap, const int32_t *__restrict__ indices,
                                                     const int32_t *__restrict__ count, int cap, int N, int bh, int bw) {
    for (int i = threadIdx.x; i < nmap; i += blockDim.x) map[i] = -1;
    __syncthreads();
    const int nact = min(*count, cap);
    for (int b = threadIdx.x; b < nact; b += blockDim.x) {
        const int n = indices[3 * b], by = indices[3 * b + 1], bx = indices[3 * b + 2];
        if (n >= 0 && n < N && by >= 0 && by < bh && bx >= 0 && bx < bw) map[(n * bh + by) * bw + bx] = b;
    }
}

// fp32 sum of storage words, element-wise
template <int DT> struct Acc;
template <> struct Acc<SBNET_F32> {
    static constexpr int N = 1;
    static __device__ __forceinline__ void add(float *a, uint32_t w) { a[0] += __uint_as_float(w); }
    static __device__ __forceinline__ uint32_t pack(const float *a) { return __float_as_uint(a[0]); }
};
template <> struct Acc<SBNET_BF16> {
    static constexpr int N = 2;
    static __device__ __forceinline__ void add(float *a, uint32_t w) {
        a[0] += bf16_bits_to_float(w & 0xffffu);
        a[1] += bf16_bits_to_float(w >> 16);
    }
    static __device__ __forceinline__ uint32_t pack(const float *a) {
        return float_to_bf16_bits(a[0]) | (float_to_bf16_bits(a[1]) << 16);
    }
};
template <> struct Acc<SBNET_F16> {
    static constexpr int N = 2;
    static __device__ __forceinline__ float h2f(uint32_t b) {
        union { _Float16 h; uint16_t u; } x;
        x.u = (uint16_t)b;
        return (float)x.h;
    }
    static __device__ __forceinline__ uint32_t f2h(float f) {
        union { _Float16 h; uint16_t u; } x;
        x.h = (_Float16)f;
        return x.u;
    }
    static __device__ __forceinline__ void add(float *a, uint32_t w) {
        a[0] += h2f(w & 0xffffu);
        a[1] += h2f(w >> 16);
    }
    static __device__ __forceinline__ uint32_t pack(const float *a) { return f2h(a[0]) | (f2h(a[1]) << 16); }
};

// V: uint4 / uint2 / uint32_t (whole 32-bit words of the storage type)
template <typename V> struct Words;
template <> struct Words<uint4> { static constexpr int N = 4; };
template <> struct Words<uint2> { static constexpr int N = 2; };
template <> struct Words<uint32_t> { static constexpr int N = 1; };
__device__ __forceinline__ uint32_t word_of(const uint4 &v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
__device__ __forceinline__ uint32_t word_of(const uint2 &v, int i) { return i == 0 ? v.x : v.y; }
__device__ __forceinline__ uint32_t word_of(const uint32_t &v, int) { return v; }
__device__ __forceinline__ void make_vec(uint4 &v, const uint32_t *w) { v = make_uint4(w[0], w[1], w[2], w[3]); }
__device__ __forceinline__ void make_vec(uint2 &v, const uint32_t *w) { v = make_uint2(w[0], w[1]); }
__device__ __forceinline__ void make_vec(uint32_t &v, const uint32_t *w) { v = w[0]; }

// U vectors per thread are processed together, all of
// their loads (tile gradients and dx) issued before the first is used: a thread's memory round trips overlap
// instead of adding up (more than two at a time was measured slower: fewer workgroups fit a CU).
// RM: largest reach in cells.
template <typename V, int DT, int RM, int U>
__device__ __forceinline__ void gb_cells(V *__restrict__ dx, const V *__restrict__ dtiles, const int32_t *__restrict__ map,
                                         const GbParams &p) {
    constexpr int NW = Words<V>::N, NA = Acc<DT>::N;
    constexpr int NT = (RM + 1) * (RM + 1);
    const uint32_t ncells = (uint32_t)p.N * p.cells_h * p.cells_w;
    for (uint32_t cell = blockIdx.x; cell < ncells; cell += gridDim.x) {
        const uint32_t n = fdiv(cell, p.div_cells);
        const uint32_t rest = cell - n * (uint32_t)(p.cells_h * p.cells_w);
        const int cy = (int)fdiv(rest, p.div_cw), cx = (int)rest - cy * p.cells_w;
        // tiles that can cover this cell: blocks (cy - R_h .. cy, cx - R_w .. cx), ascending; the lookups are
        // issued together (indices clamped into the map, results masked)
        int tb[NT];
        int nt = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int dy = RM - t / (RM + 1), dxc = RM - t % (RM + 1);
            const int by = cy - dy, bx = cx - dxc;
            const bool ok = dy <= p.R_h && dxc <= p.R_w && by >= 0 && by < p.g.bcount_h && bx >= 0 && bx < p.g.bcount_w;
            const int e = map[((int)n * p.g.bcount_h + min(max(by, 0), p.g.bcount_h - 1)) * p.g.bcount_w +
                              min(max(bx, 0), p.g.bcount_w - 1)];
            tb[t] = ok ? e : -1;
            nt += tb[t] >= 0;
        }
        if (nt == 0) continue;                                   // workgroup-uniform
        const int py0 = p.g.boffset_h + cy * p.g.bstride_h, px0 = p.g.boffset_w + cx * p.g.bstride_w;
        for (uint32_t v0 = threadIdx.x; v0 < p.cell_vecs; v0 += kGbThreads * U) {
            V tv[U][NT], old[U];
            bool use[U][NT], any[U];
            size_t o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t v = v0 + u * kGbThreads;
                const uint32_t r = fdiv(v, p.div_row), rem = v - r * p.row_vecs;
                const uint32_t c = fdiv(rem, p.div_pv), k = rem - c * p.pix_vecs;
                const int yy = py0 + (int)r, xx = px0 + (int)c;
                const bool live = v < p.cell_vecs && yy >= 0 && yy < p.H && xx >= 0 && xx < p.W;
                any[u] = false;
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    const int dy = RM - t / (RM + 1), dxc = RM - t % (RM + 1);
                    // position inside that tile: its origin lies dy (dxc) cells up (left)
                    const int i = (int)r + dy * p.g.bstride_h, j = (int)c + dxc * p.g.bstride_w;
                    use[u][t] = live && tb[t] >= 0 && i < p.g.bsize_h && j < p.g.bsize_w;
                    if (use[u][t])
                        tv[u][t] = dtiles[(size_t)tb[t] * p.tile_vecs + (uint32_t)i * p.tile_row_vecs + (uint32_t)j * p.pix_vecs + k];
                    any[u] |= use[u][t];
                }
                o[u] = (((size_t)n * p.H + yy) * p.W + xx) * p.pix_vecs + k;
                if (any[u]) old[u] = dx[o[u]];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!any[u]) continue;
                float acc[NW * NA];
#pragma unroll
                for (int i = 0; i < NW * NA; ++i) acc[i] = 0.f;
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (use[u][t]) {
#pragma unroll
                        for (int w = 0; w < NW; ++w) Acc<DT>::add(acc + w * NA, word_of(tv[u][t], w));
                    }
                uint32_t out[NW];
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    Acc<DT>::add(acc + w * NA, word_of(old[u], w));
                    out[w] = Acc<DT>::pack(acc + w * NA);
                }
                V res;
                make_vec(res, out);
                dx[o[u]] = res;
            }
        }
    }
}

// Piece `seg` of active tile b.  Every pixel of the tile looks which neighbouring tiles cover it too (at most one
// vertically, one horizontally and their diagonal); the first existing one in (by, bx) order owns the pixel and adds all
// of them, so what an owner adds after its own value comes in ascending order by itself.
// Bound by HBM (tile gradients read once, dx read and written once).  A cell per workgroup, as in gb_cells, left most
// workgroups without work and the others with a chain of up to sixteen memory round trips.
template <typename V, int DT, int U>
__device__ __forceinline__ void gb_tiles(V *__restrict__ dx, const V *__restrict__ dtiles,
                                         const int32_t *__restrict__ map, const int32_t *__restrict__ indices, uint32_t nact,
                                         int segs, uint32_t piece, const FastDiv &div_segs, const FastDiv &div_tr, const GbParams &p) {
    constexpr int NW = Words<V>::N, NA = Acc<DT>::N;
    // the first item's block is requested beside the count (past the count, and the list, it is not used)
    uint32_t b = min(fdiv(blockIdx.x, div_segs), (uint32_t)p.cap - 1u);
    int n = indices[3 * b], by = indices[3 * b + 1], bx = indices[3 * b + 2];
    const uint32_t items = nact * (uint32_t)segs;
    const int ovh = p.g.bsize_h - p.g.bstride_h, ovw = p.g.bsize_w - p.g.bstride_w;
    for (uint32_t item = blockIdx.x; item < items; item += gridDim.x) {
        if (item != blockIdx.x) {
            b = fdiv(item, div_segs);
            n = indices[3 * b]; by = indices[3 * b + 1]; bx = indices[3 * b + 2];
        }
        const uint32_t seg = item - b * (uint32_t)segs;
        if (n < 0 || n >= p.N || by < 0 || by >= p.g.bcount_h || bx < 0 || bx >= p.g.bcount_w) continue;
        int nb[9];                                                // list positions of the 3 x 3 blocks around b, -1: none
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int y = by + t / 3 - 1, x = bx + t % 3 - 1;
            const bool ok = y >= 0 && y < p.g.bcount_h && x >= 0 && x < p.g.bcount_w;
            const int e = map[(n * p.g.bcount_h + min(max(y, 0), p.g.bcount_h - 1)) * p.g.bcount_w + min(max(x, 0), p.g.bcount_w - 1)];
            nb[t] = ok ? e : -1;
        }
        const int py0 = p.g.boffset_h + by * p.g.bstride_h, px0 = p.g.boffset_w + bx * p.g.bstride_w;
        const uint32_t v_hi = min((seg + 1) * piece, p.tile_vecs);
        for (uint32_t v0 = seg * piece + threadIdx.x; v0 < v_hi; v0 += kGbThreads * U) {
            V own[U], old[U], more[U][3];
            size_t o[U];
            uint32_t use[U];                                          // bit 3: owned; bits 0..2: more[u][0..2] adds
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t v = v0 + u * kGbThreads;
                const uint32_t i = fdiv(v, div_tr), rem = v - i * p.tile_row_vecs;
                const uint32_t j = fdiv(rem, p.div_pv), k = rem - j * p.pix_vecs;
                const int yy = py0 + (int)i, xx = px0 + (int)j;
                const bool live = v < v_hi && yy >= 0 && yy < p.H && xx >= 0 && xx < p.W;
                // the other tile row / column over this pixel: -1 the one before, +1 the one after, 0 none
                const int dy = (int)i < ovh ? -1 : (int)i >= p.g.bstride_h ? 1 : 0;
                const int dxc = (int)j < ovw ? -1 : (int)j >= p.g.bstride_w ? 1 : 0;
                const int th = dxc < 0 ? nb[3] : dxc > 0 ? nb[5] : -1;
                const int tv = dy < 0 ? nb[1] : dy > 0 ? nb[7] : -1;
                const int td = dy < 0 ? (dxc < 0 ? nb[0] : dxc > 0 ? nb[2] : -1) : dy > 0 ? (dxc < 0 ? nb[6] : dxc > 0 ? nb[8] : -1) : -1;
                // a tile in front of b owns the pixel: left in the same row, anything in the row before
                const bool mine = live && !(dxc < 0 && th >= 0) && !(dy < 0 && (tv >= 0 || td >= 0));
                o[u] = (((size_t)n * p.H + yy) * p.W + xx) * p.pix_vecs + k;
                const int oh = -dxc * p.g.bstride_w * (int)p.pix_vecs, ov = -dy * p.g.bstride_h * (int)p.tile_row_vecs;
                // the row after: the tile further left first
                const bool left = dxc < 0;
                const int t1 = left ? td : tv, t2 = left ? tv : td, o1 = left ? oh + ov : ov, o2 = left ? ov : oh + ov;
                use[u] = mine ? 8u | (th >= 0 ? 1u : 0u) | (t1 >= 0 ? 2u : 0u) | (t2 >= 0 ? 4u : 0u) : 0u;
                if (mine) {
                    own[u] = dtiles[(size_t)b * p.tile_vecs + v];
                    old[u] = dx[o[u]];
                    if (th >= 0) more[u][0] = dtiles[(size_t)th * p.tile_vecs + (v + oh)];
                    if (t1 >= 0) more[u][1] = dtiles[(size_t)t1 * p.tile_vecs + (v + o1)];
                    if (t2 >= 0) more[u][2] = dtiles[(size_t)t2 * p.tile_vecs + (v + o2)];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!use[u]) continue;
                float acc[NW * NA];
#pragma unroll
                for (int i = 0; i < NW * NA; ++i) acc[i] = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) Acc<DT>::add(acc + w * NA, word_of(own[u], w));
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    if (use[u] >> t & 1) {
#pragma unroll
                        for (int w = 0; w < NW; ++w) Acc<DT>::add(acc + w * NA, word_of(more[u][t], w));
                    }
                uint32_t out[NW];
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    Acc<DT>::add(acc + w * NA, word_of(old[u], w));
                    out[w] = Acc<DT>::pack(acc + w * NA);
                }
                V res;
                make_vec(res, out);
                dx[o[u]] = res;
            }
        }
    }
}

// Both ways in one launch: cell by cell from `cells_from` active blocks, tile by tile below (gb_cells_from).  Seven workgroups
// per CU: three vectors per thread in flight on five were slower both ways (800 x 704 x 64, blocks of 16 x 16, 35 % of them
// by tiles: 22.3 against 20.0 us; 8 x 8 all of them by cells: 49.4 against 47.0).
template <typename V, int DT, int U>
__global__ __launch_bounds__(kGbThreads, 7) void gb_either(V *__restrict__ dx, const V *__restrict__ dtiles,
                                                        const int32_t *__restrict__ map, const int32_t *__restrict__ indices,
                                                        const int32_t *__restrict__ count, int cells_from, int segs, uint32_t piece,
                                                        FastDiv div_segs, FastDiv div_tr, GbParams p) {
    const int nact = max(min(*count, p.cap), 0);
    if (nact >= cells_from) gb_cells<V, DT, 1, 2>(dx, dtiles, map, p);
    else gb_tiles<V, DT, U>(dx, dtiles, map, indices, (uint32_t)nact, segs, piece, div_segs, div_tr, p);
}

template <typename V, int DT>
__global__ __launch_bounds__(kGbThreads) void gb_near(V *__restrict__ dx, const V *__restrict__ dtiles,
                                                      const int32_t *__restrict__ map, GbParams p) {
    gb_cells<V, DT, 1, 2>(dx, dtiles, map, p);
}

template <typename V, int DT>
__global__ __launch_bounds__(kGbThreads) void gb_far(V *__restrict__ dx, const V *__restrict__ dtiles,
                                                     const int32_t *__restrict__ map, GbParams p) {
    gb_cells<V, DT, kGbMaxR, 2>(dx, dtiles, map, p);
}

// From how many active blocks on a launch runs cell by cell, for tiles that reach over one following block at most.  By tiles a
// launch has work for every workgroup whatever the list, but pixels of a halo are visited by each of their tiles; by cells
// no pixel is visited twice.  bf16, by cells against by tiles:
//   halos of at least half a cell (8 x 8 blocks): where the active tiles do not fit the caches, 75 MB of them:
//     800 x 704 x 64   65 % (73 MB) 35.3 and 35.4 us, 100 % 46.6 and 48.3;  800 x 704 x 128   20 % 32.5 and 26.1, 35 % (79 MB) 39.9
//     and 42.6, 100 % 89.7 and 126;  200 x 176 x 256   100 % 18.6 and 16.4
//   narrower halos: nearly full lists, where there are cells enough for the device and they are not large:
//     16 x 16 blocks, 800 x 704 x 64   80 % 38.2 and 36.6, 100 % 43.1 and 44.1;  x 96   80 % 54.9 and 53.7, 100 % 62.5 and 64.8;
//     x 256   100 % 215 and 204;  400 x 352 x 64   100 % 17.7 and 14.9;  24 x 24, 800 x 704 x 48   80 % 29.0 and 27.6, 100 % 32.6 and 33.7
static int gb_cells_from(const GbParams &p, long long ncells, int vec_bytes) {
    const long long nblocks = (long long)p.N * p.g.bcount_h * p.g.bcount_w;
    if (2ull * p.tile_vecs >= 3ull * p.cell_vecs) return (int)(75000000 / ((long long)p.tile_vecs * vec_bytes)) + 1;
    return ncells >= 1024 && p.cell_vecs <= 4096 ? (int)((nblocks * 7 + 7) / 8) : 0x7fffffff;
}

template <typename V, int DT>
static void launch_gb(void *dx, const void *dtiles, const int32_t *map, const int32_t *indices, const int32_t *count,
                      const GbParams &p, hipStream_t s) {
    constexpr int U = 2;                                         // vectors per thread in flight
    const long long ncells = (long long)p.N * p.cells_h * p.cells_w;
    // pieces of a tile: one step of a workgroup each, a tile that is little more than one step whole
    const int segs = p.tile_vecs <= 4 * kGbThreads ? 1 : (int)((p.tile_vecs + kGbThreads * U - 1) / (kGbThreads * U));
    const uint32_t piece = (p.tile_vecs + segs - 1) / segs;
    const long long items = (long long)p.cap * segs;
    const int grid = (int)(ncells < 16384 ? ncells : 16384);
    if (p.R_h > 1 || p.R_w > 1) {
        hipLaunchKernelGGL((gb_far<V, DT>), dim3(grid), dim3(kGbThreads), 0, s, (V *)dx, (const V *)dtiles, map, p);
        return;
    }
    // cells that are one step of a workgroup each, all of them resident at once, need no list: one memory round trip less
    // (200 x 176 x 64, 8 x 8 blocks, a tenth of them: 6.6 us against 8.0 by tiles)
    if ((p.cell_vecs <= 2 * kGbThreads && ncells <= 1024) || items >= (1LL << 31)) {
        hipLaunchKernelGGL((gb_near<V, DT>), dim3(grid), dim3(kGbThreads), 0, s, (V *)dx, (const V *)dtiles, map, p);
        return;
    }
    const int cells_from = gb_cells_from(p, ncells, (int)sizeof(V));
    const int gt = (int)(items < 4096 ? items : 4096), gc = p.cap >= cells_from ? grid : 1;
    hipLaunchKernelGGL((gb_either<V, DT, U>), dim3(gt > gc ? gt : gc), dim3(kGbThreads), 0, s, (V *)dx, (const V *)dtiles, map,
                       indices, count, cells_from, segs, piece, make_fastdiv(segs), make_fastdiv(p.tile_row_vecs), p);
}

template <int DT>
static sbnet_status dispatch_gb(int vec_bytes, void *dx, const void *dtiles, const int32_t *map, const int32_t *indices,
                                const int32_t *count, const GbParams &p, hipStream_t s) {
    switch (vec_bytes) {
        case 16: launch_gb<uint4, DT>(dx, dtiles, map, indices, count, p, s); break;
        case 8: launch_gb<uint2, DT>(dx, dtiles, map, indices, count, p, s); break;
        case 4: launch_gb<uint32_t, DT>(dx, dtiles, map, indices, count, p, s); break;
        default: return fail(SBNET_EUNSUPPORTED, "sbnet_sparse_gather_backward: a pixel's channels must fill 4-byte words");
    }
    return launch_status("sbnet_sparse_gather_backward");
}

}  // namespace sbnet

using namespace sbnet;

extern "C" size_t sbnet_gather_backward_workspace_bytes(int N, const sbnet_geom *g) {
    if (N <= 0 || !geom_ok(g)) return 0;
    return (size_t)N * g->bcount_h * g->bcount_w * sizeof(int32_t);
}

extern "C" sbnet_status sbnet_sparse_gather_backward(const void *dtiles, sbnet_dtype dtype, const int32_t *indices,
                                                     const int32_t *count, int cap, const sbnet_geom *g, void *dx,
                                                     int N, int H, int W, int C, void *workspace,
                                                     size_t workspace_bytes, void *stream) {
    const char *who = "sbnet_sparse_gather_backward";
    if (!dtiles || !indices || !count || !dx || !workspace) return fail(SBNET_EINVAL, "%s: null pointer", who);
    if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || cap < 0) return fail(SBNET_EINVAL, "%s: bad sizes", who);
    if (!geom_ok(g)) return fail(SBNET_EINVAL, "%s: bad geometry", who);
    if (!is_float_dtype(dtype)) return fail(SBNET_EUNSUPPORTED, "%s: dtype must be f32, bf16 or f16", who);
    if (((uintptr_t)dx | (uintptr_t)dtiles) & 15 || ((uintptr_t)workspace & 3))
        return fail(SBNET_EINVAL, "%s: pointers must be 16-byte aligned (workspace: 4)", who);
    if (workspace_bytes < sbnet_gather_backward_workspace_bytes(N, g)) return fail(SBNET_EINVAL, "%s: workspace too small", who);
    const int R_h = g->bsize_h > g->bstride_h ? (g->bsize_h - g->bstride_h + g->bstride_h - 1) / g->bstride_h : 0;
    const int R_w = g->bsize_w > g->bstride_w ? (g->bsize_w - g->bstride_w + g->bstride_w - 1) / g->bstride_w : 0;
    if (R_h > kGbMaxR || R_w > kGbMaxR)
        return fail(SBNET_EUNSUPPORTED, "%s: tiles may overlap at most three following blocks per axis", who);
    if (cap == 0) return SBNET_OK;
    const long long pix_bytes = (long long)C * elem_bytes(dtype);
    int vec = 16;
    while (vec > 4 && pix_bytes % vec) vec >>= 1;
    if (pix_bytes % vec) return fail(SBNET_EUNSUPPORTED, "%s: a pixel's channels must fill 4-byte words", who);
    const long long cells = (long long)N * (g->bcount_h + R_h) * (g->bcount_w + R_w);
    const long long tile_vecs = (long long)g->bsize_h * g->bsize_w * (pix_bytes / vec);
    if (cells >= (1LL << 31) || tile_vecs >= (1LL << 31) || (long long)N * g->bcount_h * g->bcount_w >= (1LL << 31) ||
        (long long)g->bstride_h * g->bstride_w * (pix_bytes / vec) >= (1LL << 31))
        return fail(SBNET_EUNSUPPORTED, "%s: tensor too large", who);

    GbParams p;
    p.g = *g;
    p.N = N; p.H = H; p.W = W; p.cap = cap;
    p.R_h = R_h; p.R_w = R_w;
    p.cells_h = g->bcount_h + R_h;
    p.cells_w = g->bcount_w + R_w;
    p.pix_vecs = (uint32_t)(pix_bytes / vec);
    p.row_vecs = (uint32_t)g->bstride_w * p.pix_vecs;
    p.cell_vecs = (uint32_t)g->bstride_h * p.row_vecs;
    p.tile_row_vecs = (uint32_t)g->bsize_w * p.pix_vecs;
    p.tile_vecs = (uint32_t)tile_vecs;
    p.div_cells = make_fastdiv((uint32_t)(p.cells_h * p.cells_w));
    p.div_cw = make_fastdiv((uint32_t)p.cells_w);
    p.div_row = make_fastdiv(p.row_vecs);
    p.div_pv = make_fastdiv(p.pix_vecs);
    hipStream_t s = (hipStream_t)stream;
    int32_t *map = (int32_t *)workspace;
    const int nmap = N * g->bcount_h * g->bcount_w;
    if (nmap <= 32768 && cap <= 32768) {
        hipLaunchKernelGGL(gb_map_build, dim3(1), dim3(1024), 0, s, map, nmap, indices, count, cap, N, g->bcount_h, g->bcount_w);
    } else {
        hipLaunchKernelGGL(gb_map_clear, dim3((nmap + 255) / 256 > 1024 ? 1024 : (nmap + 255) / 256), dim3(256), 0, s, map, nmap);
        hipLaunchKernelGGL(gb_map_fill, dim3((cap + 255) / 256 > 1024 ? 1024 : (cap + 255) / 256), dim3(256), 0, s, map, indices,
                           count, cap, N, g->bcount_h, g->bcount_w);
    }
    if (dtype == SBNET_F32) return dispatch_gb<SBNET_F32>(vec, dx, dtiles, map, indices, count, p, s);
    if (dtype == SBNET_BF16) return dispatch_gb<SBNET_BF16>(vec, dx, dtiles, map, indices, count, p, s);
    return dispatch_gb<SBNET_F16>(vec, dx, dtiles, map, indices, count, p, s);
}
