// Data-layout conversion kernels: NCHW <-> 16-channel-blocked, and the filter re-layouts.
// Pure permutations of bit patterns (paper Abstract / Sec. 2: data layout abstraction).
// HBM bound: 1 read + 1 write per element.  The fast 2-byte path transposes a
// 16(channel) x 256(pixel) tile through LDS so that both the NCHW side (contiguous in
// pixels) and the blocked side (contiguous in channels, then pixels) move as full lines.
#include "common.h"

namespace ngc {

constexpr int LT_PIX = 256;          // pixels per tile
constexpr int LT_PITCH = LT_PIX + 2; // LDS row pitch in elements (odd dword count: 129 dwords)

// ---- NCHW -> blocked, 2-byte elements.  grid = (ceil(HW/256), CB, N), block = 256.
// V = pixels per global read (1, 2, 4 or 8), chosen by the host from the alignment of HW.
// stream: the copy is written past the memory-side cache.  The next kernel reads it, so only copies that would not stay
// there are (launch_layout_convert).
template <int V>
__global__ __launch_bounds__(256) void nchw_to_blocked16_b16(const uint16_t *__restrict__ src,
                                                             uint16_t *__restrict__ dst, int C, int HW, int stream)
{
    __shared__ __align__(16) uint16_t tile[16 * LT_PITCH];
    const int tid = threadIdx.x;
    const int px0 = blockIdx.x * LT_PIX;
    const int cb = blockIdx.y;
    const int n = blockIdx.z;
    const int CB = gridDim.y;

    // read phase: 16 channel rows x 256 pixels, V pixels per access
    constexpr int ACC_PER_ROW = LT_PIX / V;
    constexpr int ITERS = 16 * ACC_PER_ROW / 256;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int a = tid + 256 * it;
        const int ci = a / ACC_PER_ROW;
        const int px = (a % ACC_PER_ROW) * V;
        const int c = cb * 16 + ci;
        uint16_t v[V];
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = 0;
        if (c < C && px0 + px < HW) {                     // HW % V == 0 so a vector is all-in or all-out
            const uint16_t *g = src + ((size_t)n * C + c) * HW + px0 + px;
            if constexpr (V == 8) {
                uint4 q = *reinterpret_cast<const uint4 *>(g);
                v[0] = q.x & 0xFFFF; v[1] = q.x >> 16; v[2] = q.y & 0xFFFF; v[3] = q.y >> 16;
                v[4] = q.z & 0xFFFF; v[5] = q.z >> 16; v[6] = q.w & 0xFFFF; v[7] = q.w >> 16;
            } else if constexpr (V == 4) {
                uint2 q = *reinterpret_cast<const uint2 *>(g);
                v[0] = q.x & 0xFFFF; v[1] = q.x >> 16; v[2] = q.y & 0xFFFF; v[3] = q.y >> 16;
            } else if constexpr (V == 2) {
                uint32_t q = *reinterpret_cast<const uint32_t *>(g);
                v[0] = q & 0xFFFF; v[1] = q >> 16;
            } else {
                v[0] = *g;
            }
        }
#pragma unroll
        for (int e = 0; e < V; ++e) tile[ci * LT_PITCH + px + e] = v[e];
    }
    __syncthreads();

    // write phase: per pixel 16 channels = 32 B; each thread writes 16 B (8 channels)
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int a = tid + 256 * it;
        const int px = a >> 1;
        const int half = a & 1;
        if (px0 + px < HW) {
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t lo = tile[(half * 8 + 2 * e) * LT_PITCH + px];
                const uint32_t hi = tile[(half * 8 + 2 * e + 1) * LT_PITCH + px];
                w[e] = lo | (hi << 16);
            }
            uint16_t *g = dst + (((size_t)n * CB + cb) * HW + px0 + px) * 16 + half * 8;
            store16_result(g, make_uint4(w[0], w[1], w[2], w[3]), stream != 0);
        }
    }
}

// ---- blocked -> NCHW, 2-byte elements.  Same tiling, phases swapped.
template <int V>
__global__ __launch_bounds__(256) void blocked16_to_nchw_b16(const uint16_t *__restrict__ src,
                                                             uint16_t *__restrict__ dst, int C, int HW)
{
    __shared__ __align__(16) uint16_t tile[16 * LT_PITCH];
    const int tid = threadIdx.x;
    const int px0 = blockIdx.x * LT_PIX;
    const int cb = blockIdx.y;
    const int n = blockIdx.z;
    const int CB = gridDim.y;

#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int a = tid + 256 * it;
        const int px = a >> 1;
        const int half = a & 1;
        uint4 q = make_uint4(0, 0, 0, 0);
        if (px0 + px < HW)
            q = *reinterpret_cast<const uint4 *>(src + (((size_t)n * CB + cb) * HW + px0 + px) * 16 + half * 8);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            tile[(half * 8 + 2 * e) * LT_PITCH + px] = (uint16_t)(w[e] & 0xFFFF);
            tile[(half * 8 + 2 * e + 1) * LT_PITCH + px] = (uint16_t)(w[e] >> 16);
        }
    }
    __syncthreads();

    constexpr int ACC_PER_ROW = LT_PIX / V;
    constexpr int ITERS = 16 * ACC_PER_ROW / 256;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int a = tid + 256 * it;
        const int ci = a / ACC_PER_ROW;
        const int px = (a % ACC_PER_ROW) * V;
        const int c = cb * 16 + ci;
        if (c < C && px0 + px < HW) {
            uint16_t v[V];
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = tile[ci * LT_PITCH + px + e];
            uint16_t *g = dst + ((size_t)n * C + c) * HW + px0 + px;
            if constexpr (V == 8) {
                *reinterpret_cast<uint4 *>(g) = make_uint4(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16),
                                                           v[4] | ((uint32_t)v[5] << 16), v[6] | ((uint32_t)v[7] << 16));
            } else if constexpr (V == 4) {
                *reinterpret_cast<uint2 *>(g) = make_uint2(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16));
            } else if constexpr (V == 2) {
                *reinterpret_cast<uint32_t *>(g) = v[0] | ((uint32_t)v[1] << 16);
            } else {
                *g = v[0];
            }
        }
    }
}

// ---- generic element-wise permutation (any element size, any direction): one thread per
// destination element.  Used for 4-byte elements and same-layout copies.
template <typename E>
__global__ __launch_bounds__(256) void layout_generic(const E *__restrict__ src, E *__restrict__ dst, int N, int C,
                                                      int H, int W, int src_layout, int dst_layout, size_t total)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    int n, c, h, w;
    size_t t = i;
    if (dst_layout == NGC_NCHW) {
        w = t % W; t /= W; h = t % H; t /= H; c = t % C; n = (int)(t / C);
    } else {
        const int CB = (C + 15) >> 4;
        const int ci = t % 16; t /= 16; w = t % W; t /= W; h = t % H; t /= H;
        const int cb = t % CB; n = (int)(t / CB);
        c = cb * 16 + ci;
    }
    E v = 0;
    if (c < C) v = src[data_index(src_layout, C, H, W, n, c, h, w)];
    dst[i] = v;
}

// ---- filter re-layout KCRS -> blocked, 2-byte elements, C a multiple of 16: tiles of 16 x G filters through LDS.
// A destination run of 16 channels gathers elements that are R S apart in KCRS (and whole filters apart for the
// backprop-data form), so one thread per destination element reads 2 bytes of a different line per lane, and the tile
// below is what keeps the traffic at one read and one write.  A workgroup reads the filters of 16 lanes (the blocked axis)
// x G rows (the other channel axis) as runs of whole 16-byte pieces, then writes, tap by tap, G runs of 32 bytes.
// Bound: launch and load latency below a few MB, then HBM.  512 x 512 x 3 x 3 (4.7 MB): a thread per element 8.1 us, tiles 5.2 us.
// FWD: lanes = c, rows = k, source run of a row = 16 R S elements; else lanes = k, rows = c, run of a lane = G R S.
template <bool FWD>
__global__ __launch_bounds__(256) void filter_tiles_b16(const uint16_t *__restrict__ src, uint16_t *__restrict__ dst, int K, int C,
                                                        int RS, int lg, FastDiv div_run)
{
    extern __shared__ __align__(16) uint16_t ft[];
    const int G = 1 << lg, b = blockIdx.y, g0 = blockIdx.x << lg;
    const int rows = FWD ? K : C, live = rows - g0 < G ? rows - g0 : G;
    const int pitch = (FWD ? 16 : G) * RS + 8;                          // elements; whole 16-byte pieces
    const int nrun = FWD ? live : 16, run = (FWD ? 16 : live) * RS / 8; // source runs, 16-byte pieces of a run
    for (int i = threadIdx.x; i < nrun * run; i += 256) {
        const int r = (int)(live == G || FWD ? fd_div((uint32_t)i, div_run) : (uint32_t)i / (uint32_t)run), o = i - r * run;
        uint4 v = make_uint4(0, 0, 0, 0);
        const int k = FWD ? g0 + r : b * 16 + r, c = FWD ? b * 16 : g0;
        if (k < K) v = *reinterpret_cast<const uint4 *>(src + ((size_t)k * C + c) * RS + o * 8);
        *reinterpret_cast<uint4 *>(ft + r * pitch + o * 8) = v;
    }
    __syncthreads();
    const int nb = gridDim.y, n = RS * G * 2;
    for (int i = threadIdx.x; i < n; i += 256) {
        const int h = i & 1, g = (i >> 1) & (G - 1), t = i >> (lg + 1);
        if (g >= live) continue;
        uint32_t e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = FWD ? ft[g * pitch + (h * 8 + j) * RS + t] : ft[(h * 8 + j) * pitch + g * RS + t];
        *reinterpret_cast<uint4 *>(dst + (((size_t)t * nb + b) * rows + g0 + g) * 16 + h * 8) =
            make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
    }
}

// ---- the same for what the tiles refuse (4-byte elements, C no multiple of 16, long windows); one thread per
// destination element, padded lanes written as +0.
template <typename E>
__global__ __launch_bounds__(256) void filter_to_blocked(const E *__restrict__ src, E *__restrict__ dst, int K, int C,
                                                         int R, int S, int dst_layout, size_t total)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    size_t t = i;
    const int lane = t % 16; t /= 16;
    int k, c;
    if (dst_layout == NGC_BLOCKED_FWD) {                // [r][s][cb][k][ci]
        const int CB = (C + 15) >> 4;
        k = t % K; t /= K;
        const int cb = t % CB; t /= CB;
        c = cb * 16 + lane;
    } else {                                            // [r][s][kb][c][ki]
        const int KB = (K + 15) >> 4;
        c = t % C; t /= C;
        const int kb = t % KB; t /= KB;
        k = kb * 16 + lane;
    }
    const int s = t % S;
    const int r = (int)(t / S);
    E v = 0;
    if (k < K && c < C) v = src[(((size_t)k * C + c) * R + r) * S + s];
    dst[i] = v;
}

// Combined filter of a stride-2 backprop-data written as a stride-1 convolution over 2x2 output
// blocks: wu[ut][k/16][col][k%16], col = (2a+b)*C + c (64 columns, the rest zero), union tap
// ut = (dr - dr_min)*nds + (ds - ds_min); entry = w[k][c][r][s] with r = a + pad_h - 2 dr,
// s = b + pad_w - 2 ds when that tap exists, else 0.
__global__ __launch_bounds__(256) void subpixel_filter(const uint16_t *__restrict__ w, uint16_t *__restrict__ wu, int K,
                                                       int C, int R, int S, int pbh, int pbw, int dr_min, int ds_min,
                                                       int nds, int BH, int BW, int sh, int sw, size_t total)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    size_t t = i;
    const int ki = t % 16; t /= 16;
    const int col = t % 64; t /= 64;
    const int KB = K >> 4;
    const int kb = t % KB; t /= KB;
    const int ut = (int)t;
    const int dr = dr_min + ut / nds, ds = ds_min + ut % nds;
    uint16_t v = 0;
    if (col < BH * BW * C) {
        const int ab = col / C, c = col - ab * C;
        const int a = ab / BW, b = ab - a * BW;
        const int r = a + pbh - sh * dr, s = b + pbw - sw * ds;
        if (r >= 0 && r < R && s >= 0 && s < S) v = w[(((size_t)(kb * 16 + ki) * C + c) * R + r) * S + s];
    }
    wu[i] = v;
}

hipError_t launch_subpixel_filter(int K, int C, int R, int S, int pbh, int pbw, int dr_min, int ndr, int ds_min, int nds,
                                  int BH, int BW, int sh, int sw, const uint16_t *w_kcrs, uint16_t *wu, hipStream_t st)
{
    const size_t total = (size_t)ndr * nds * K * 64;
    NGC_LAUNCH(subpixel_filter, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, w_kcrs, wu, K, C, R, S, pbh, pbw,
               dr_min, ds_min, nds, BH, BW, sh, sw, total);
    return ngc::launch_result();
}

static bool aligned_to(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

hipError_t launch_layout_convert(int elem_bytes, int n, int c, int h, int w, const void *src, int src_layout,
                                 void *dst, int dst_layout, hipStream_t st)
{
    const int HW = h * w;
    const int CB = (c + 15) / 16;
    const bool fast = elem_bytes == 2 && src_layout != dst_layout && CB <= 65535 && n <= 65535 &&
                      aligned_to(src, 16) && aligned_to(dst, 16);
    if (fast) {
        dim3 grid((HW + LT_PIX - 1) / LT_PIX, CB, n), block(256);
        const uint16_t *s = static_cast<const uint16_t *>(src);
        uint16_t *d = static_cast<uint16_t *>(dst);
        const int v = (HW % 8 == 0) ? 8 : (HW % 4 == 0) ? 4 : (HW % 2 == 0) ? 2 : 1;
        if (src_layout == NGC_NCHW) {
            // Ordinary stores leave the copy in the memory-side cache (256 MB) for the kernel that reads it.  Streaming / ordinary,
            // us, a graph of conversions of tensors in memory, alone, with a forward 1x1 convolution to 64 channels behind each, and
            // with all three calls of that layer:
            //   0.1 MB  2.3 /  2.3,   6.3 /   6.0,   17.5 /  17.2        26 MB  12.7 / 11.4,   21.7 /  18.4,   44.7 /  41.6
            //   0.8 MB  2.8 /  2.7,   7.4 /   6.7,   19.4 /  18.5       103 MB  42.3 / 36.5,   69.8 /  59.8,  123.7 / 114.3
            //   6.4 MB  4.1 /  4.5,  11.0 /   9.7,   27.1 /  25.9       206 MB  81.1 / 71.3,  126.6 / 120.5,  225.9 / 214.9
            // Copies that do not stay there: a conversion and a read 257 MB 149.5 / 149.0, 411 MB 234.1 / 239.2.
            const int stream = (size_t)n * CB * HW * 32 > ((size_t)240 << 20);
            if (v == 8) NGC_LAUNCH(nchw_to_blocked16_b16<8>, grid, block, 0, st, s, d, c, HW, stream);
            else if (v == 4) NGC_LAUNCH(nchw_to_blocked16_b16<4>, grid, block, 0, st, s, d, c, HW, stream);
            else if (v == 2) NGC_LAUNCH(nchw_to_blocked16_b16<2>, grid, block, 0, st, s, d, c, HW, stream);
            else NGC_LAUNCH(nchw_to_blocked16_b16<1>, grid, block, 0, st, s, d, c, HW, stream);
        } else {
            if (v == 8) NGC_LAUNCH(blocked16_to_nchw_b16<8>, grid, block, 0, st, s, d, c, HW);
            else if (v == 4) NGC_LAUNCH(blocked16_to_nchw_b16<4>, grid, block, 0, st, s, d, c, HW);
            else if (v == 2) NGC_LAUNCH(blocked16_to_nchw_b16<2>, grid, block, 0, st, s, d, c, HW);
            else NGC_LAUNCH(blocked16_to_nchw_b16<1>, grid, block, 0, st, s, d, c, HW);
        }
        return ngc::launch_result();
    }
    const size_t total = (dst_layout == NGC_NCHW) ? (size_t)n * c * HW : (size_t)n * CB * HW * 16;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (elem_bytes == 2)
        NGC_LAUNCH(layout_generic<uint16_t>, dim3(blocks), dim3(256), 0, st, static_cast<const uint16_t *>(src),
                           static_cast<uint16_t *>(dst), n, c, h, w, src_layout, dst_layout, total);
    else
        NGC_LAUNCH(layout_generic<uint32_t>, dim3(blocks), dim3(256), 0, st, static_cast<const uint32_t *>(src),
                           static_cast<uint32_t *>(dst), n, c, h, w, src_layout, dst_layout, total);
    return ngc::launch_result();
}

hipError_t launch_filter_convert(int elem_bytes, int K, int C, int R, int S, const void *w_kcrs, void *dst,
                                 int dst_layout, hipStream_t st)
{
    const size_t total = (dst_layout == NGC_BLOCKED_FWD) ? (size_t)R * S * ((C + 15) / 16) * K * 16
                                                         : (size_t)R * S * ((K + 15) / 16) * C * 16;
    // Tiles: whole 16-byte pieces in every source run (C % 16, both pointers aligned), grid and LDS within limits (64 KB: 16
    // filters of up to 120 taps).  32 rows a tile where that leaves a workgroup for every compute unit.  Below 2^17 filter
    // elements a thread per element is as fast or faster, one round trip to memory instead of one and one through LDS: 192 -> 32
    // channels, 3x3 2.5 / 3.2 us (tiles); 80 -> 416, 1x7 (233 k) 4.7 / 3.7 and 2.9 / 3.3 us; 32 -> 416, 3x3 (120 k) 4.8 / 3.6 and 4.6 / 4.6.
    const int RS = R * S, nb = dst_layout == NGC_BLOCKED_FWD ? C / 16 : (K + 15) / 16;
    if (elem_bytes == 2 && C % 16 == 0 && RS <= 120 && nb <= 65535 && total > ((size_t)1 << 17) && aligned_to(w_kcrs, 16) && aligned_to(dst, 16)) {
        const bool fwd = dst_layout == NGC_BLOCKED_FWD;
        const int rows = fwd ? K : C;
        const int lg = RS <= 16 && (size_t)((rows + 31) / 32) * nb >= 256 ? 5 : 4;
        const int G = 1 << lg;
        const size_t lds = (size_t)(fwd ? G : 16) * ((fwd ? 16 : G) * RS + 8) * 2;
        const dim3 grid((unsigned)((rows + G - 1) >> lg), (unsigned)nb);
        const FastDiv div_run = make_fastdiv((uint32_t)((fwd ? 16 : G) * RS / 8));
        const uint16_t *s = static_cast<const uint16_t *>(w_kcrs);
        uint16_t *d = static_cast<uint16_t *>(dst);
        if (fwd) NGC_LAUNCH(filter_tiles_b16<true>, grid, dim3(256), lds, st, s, d, K, C, RS, lg, div_run);
        else NGC_LAUNCH(filter_tiles_b16<false>, grid, dim3(256), lds, st, s, d, K, C, RS, lg, div_run);
        return ngc::launch_result();
    }
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (elem_bytes == 2)
        NGC_LAUNCH(filter_to_blocked<uint16_t>, dim3(blocks), dim3(256), 0, st,
                           static_cast<const uint16_t *>(w_kcrs), static_cast<uint16_t *>(dst), K, C, R, S, dst_layout,
                           total);
    else
        NGC_LAUNCH(filter_to_blocked<uint32_t>, dim3(blocks), dim3(256), 0, st,
                           static_cast<const uint32_t *>(w_kcrs), static_cast<uint32_t *>(dst), K, C, R, S, dst_layout,
                           total);
    return ngc::launch_result();
}

}  // namespace ngc
