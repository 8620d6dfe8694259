// Forward (any stride) and stride-1 backprop-data of multi-tap nodes with many input channels on small images: blocked bf16 tensors,
// bf16 MFMA (gfx950).  A workgroup of 8 waves has two position tiles of up to 112 positions x 64 output channels; four waves share a
// tile by splitting its reduction.
//
// The strip kernel gives each of its waves a part of the positions, so every wave reads every filter operand from LDS: with 256
// positions in a workgroup that is 3 LDS reads per 2 matrix instructions, more than the LDS delivers, and a barrier a stage holds the
// waves together.  Here every wave multiplies its whole tile over its own quarter of the (32-channel chunk, tap) steps, and nothing in
// the loop is shared: a filter operand goes straight from memory to the registers of the wave that needs it (and of the wave with the
// other tile, out of the same cache lines), the activations of a chunk lie in the wave's own two LDS buffers.  No barrier, 11 operand
// reads for 28 instructions.  The four tiles are added at the end through LDS, half of what a wave holds at a time, in a fixed order;
// a wave ends up with 16 channels of all its positions, one block of the blocked layout.
//
// Zeros around the images are shared: the columns between two rows serve as the right halo of one and the left halo of the other, and
// so do the rows between two images of a tile.  Two 7x7 images then take 137 pixels instead of 162.
//
// What bounds it: the issue of a wave (4 waves of 13 position groups, one a SIMD, took 33.9 us where these take 31.3), the LDS, and some
// 4 us of start, sum and stores per round of workgroups: of the cycles that the compute units are busy the matrix pipes work 0.54, the LDS
// 0.59, 0.18 of it bank conflicts (512 -> 512 at 7x7).  Strip kernel / here, us, the same operands again and again: 512 -> 512 at 7x7,
// 128 images 41.8 / 31.1; 512 -> 512 at 14x14, 32 images 36.9 / 29.4; 256 -> 256 at 14x14, 64 images 21.0 / 18.0; 464 -> 368 at 14x9, 2x2
// stride 2, 75 images 27.9 / 17.7.
#include "common.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

namespace ngc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned WV_OOB = 0x80000000u;
constexpr int WV_NBLK = 5;                       // 32-pixel blocks of a patch
constexpr int WV_MAXPATCH = 143;                 // patch pixels; one more is always zero
constexpr int WV_PLANE = (WV_MAXPATCH + 1) * 16; // bytes of 8 channels of a patch in LDS: whole turns of the banks
constexpr int WV_BUF = 4 * WV_PLANE, WV_WAVE = 2 * WV_BUF;
constexpr int WV_TAB = (WV_NBLK + 1) * 64;       // words of a table of pixel offsets, the last line past every patch
constexpr size_t WV_LDS = 2 * WV_TAB * 4 + 8 * WV_WAVE;

// n / d for n < 160, d < 160 with r = 65536 / d + 1: n (r d - 65536) <= n d < 65536
__device__ __forceinline__ int small_div(int n, int r) { return (int)(__umul24(n, r) >> 16); }

// The accumulators have to be the accumulation registers: left to the compiler, part of the 208 live in vector registers and are
// copied there and back in every step.  What reads a result has to wait for it by itself: mfma_drain.
__device__ __forceinline__ void mfma_acc(f32x4 &acc, const bf16x8 &a, const bf16x8 &b)
{
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_drain() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// NP position groups of 16 a tile
template <int NP, bool BWD>
__global__ __launch_bounds__(512) void conv_waves_bf16(const ConvWavesParams p)
{
    extern __shared__ __align__(16) unsigned char smem[];
    preload_kernargs(p);
    const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    // workgroup ids go round-robin to the 8 XCDs: tile numbers run on within one, the channel tiles of a strip are neighbours
    const int tile = (int)(blockIdx.x & 7) * p.per_xcd + (int)(blockIdx.x >> 3);
    if (tile >= p.tiles) return;
    const int bw = (int)fd_div((uint32_t)tile, p.div_nk), k0 = (tile - bw * (int)p.div_nk.d) * 64;
    const int split = wave & 3, bx = 2 * bw + (wave >> 2);              // quarter of the steps, position tile (the last may not exist)
    const int grp = (int)fd_div((uint32_t)bx, p.div_strips);
    const int n0 = grp * p.TN, p0 = (bx - grp * (int)p.div_strips.d) * p.TP;
    const int TN = p.N - n0 < p.TN ? p.N - n0 : p.TN;                    // images of the tile that exist (none: 0 or less)

    const int CB = p.Cin >> 4, HWin = p.Hin * p.Win;
    unsigned *const xtab = reinterpret_cast<unsigned *>(smem) + (wave >> 2) * WV_TAB + lane;     // [block][64]: this lane's offset in it
    unsigned char *const mine = smem + 2 * WV_TAB * 4 + wave * WV_WAVE;

    // this wave's steps: [first, last) of the (chunk, tap) pairs, tap fastest
    const int ntaps = p.ntaps, all = ((CB + 1) >> 1) * ntaps;
    const int first = (all * split) >> 2, last = (all * (split + 1)) >> 2;
    const int c_first = (int)fd_div((uint32_t)first, p.div_taps), t_first = first - c_first * ntaps;
    const int c_last = (int)fd_div((uint32_t)(last - 1), p.div_taps);
    const int n_steps = last - first;

    const __amdgpu_buffer_rsrc_t rs_in = __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)p.in_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_wt = __builtin_amdgcn_make_buffer_rsrc((void *)p.wt, 0, (int)p.wt_bytes, 0x00020000);

    // ---- activations: block i of 32 patch pixels, a lane 8 of 16 channels; two 16-channel blocks make a chunk.  A pixel that does not
    // exist reads as zero; pixels past the patch are written to one place behind it.
    unsigned x_soff = (unsigned)(2 * c_first * HWin * 32), x_none = 2 * c_first + 1 < CB ? 0u : WV_OOB;      // an odd last 16-channel block
    auto load_x = [&](unsigned v, int u) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_in, (int)(u == 0 ? v : v | x_none),
                                                                               (int)(u == 0 ? x_soff : (x_soff + (unsigned)(HWin * 32)) & ~x_none), 0));
    };
    auto place = [&](int i) {
        const int px = i * 32 + (lane >> 1);
        return mine + (lane & 1) * WV_PLANE + (px < WV_MAXPATCH ? px : WV_MAXPATCH) * 16;
    };
    const int h_top = p0 * p.sh + p.h0;
    const unsigned x_image = (unsigned)(CB * HWin) * 32u, x_tile = (unsigned)n0 * x_image;
    bf16x8 x0[WV_NBLK][2];
#pragma unroll
    for (int i = 0; i < WV_NBLK; ++i) {
        const int pi = i * 32 + (lane >> 1), row = small_div(pi, p.rcp_pc), ti = small_div(row, p.rcp_pr);
        const int h = h_top + row - __umul24(ti, p.PR), w = pi - __umul24(row, p.PC) + p.w0;
        const bool ok = (ti < TN) & ((unsigned)h < (unsigned)p.Hin) & ((unsigned)w < (unsigned)p.Win) & (pi < p.npatch);
        const unsigned at = x_tile + (unsigned)ti * x_image + (unsigned)(__umul24(h, p.Win) + w) * 32u + (unsigned)(lane & 1) * 16u;
        const unsigned off = ok ? at : WV_OOB;
        if ((i & 3) == split) xtab[i * 64] = off;
#pragma unroll
        for (int u = 0; u < 2; ++u) x0[i][u] = load_x(off, u);
    }
    if (split == 1) xtab[WV_NBLK * 64] = WV_OOB;

    // ---- filters.  Accumulator block a of this wave holds the channels of block a ^ split, so that every wave sends the same
    // registers in the sum at the end.
    unsigned woff[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int k = k0 + (a ^ split) * 16 + l16;
        const bool none = k >= p.Cout || (2 * c_first + 1 >= CB && g >= 2);
        woff[a] = none ? WV_OOB : (unsigned)(k * 32 + (g & 1) * 16 + (g >> 1) * p.Cout * 32);
    }
    const int tap_r = small_div(lane, p.rcp_s), tap_s = lane - __umul24(tap_r, p.S);      // lane l holds tap l
    const int toffv = p.tap0 + tap_r * p.tap_dr + tap_s * p.tap_ds, slabv = (int)((unsigned)lane * (unsigned)(CB * p.Cout * 32));      // past the last tap: any value
    const int w_chunk = 2 * p.Cout * 32;
    int w_soff = c_first * w_chunk, wt = t_first, wc = c_first, wleft = n_steps;       // the step whose filters are requested next
    auto load_w = [&](int i) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_wt, (int)woff[i], w_soff + __builtin_amdgcn_readlane(slabv, wt), 0));
    };
    auto next_w = [&]() {                                                // past the end: the last step's again
        if (--wleft > 0 && ++wt == ntaps) {
            wt = 0;
            w_soff += w_chunk;
            if (2 * ++wc + 1 >= CB) {                                    // an odd last 16-channel block
#pragma unroll
                for (int a = 0; a < 4; ++a) woff[a] = g >= 2 ? WV_OOB : woff[a];
            }
        }
    };

    bf16x8 wa[2][4];
    wa[0][0] = load_w(0);
    wa[0][1] = load_w(1);
    __builtin_amdgcn_sched_barrier(0);

    // ---- positions of this lane, and where they are stored (in the shadow of the first loads)
    const int CBout = p.Cout >> 4, HWout = p.Hout * p.Wout;
    const int kq = k0 + split * 16 + 4 * g;                               // the lane's channels in the end: kq .. kq + 3
    const unsigned o_image = (unsigned)(CBout * HWout) * 32u, o_tile = (unsigned)n0 * o_image + (unsigned)((kq >> 4) * HWout + p0 * p.Wout) * 32u + 8u * g;
    int pbase[NP];
    unsigned ooff[NP];
#pragma unroll
    for (int f = 0; f < NP; ++f) {
        const int m = f * 16 + l16, row = small_div(m, p.rcp_q), q = m - __umul24(row, p.Wout);
        const int ti = small_div(row, p.rcp_tp), tp = row - __umul24(ti, p.TP);
        const bool in = m < p.npix, ok = in & (ti < TN) & (p0 + tp < p.Hout) & (kq < p.Cout);
        const int px = __umul24(__umul24(ti, p.PR) + __umul24(tp, p.sh), p.PC) + __umul24(q, p.sw);
        const unsigned at = o_tile + (unsigned)ti * o_image + (unsigned)(__umul24(tp, p.Wout) + q) * 32u;
        pbase[f] = (in ? px * 16 : 0) + g * WV_PLANE;
        ooff[f] = ok ? at : WV_OOB;
    }
    f32x4 bias4 = {0.f, 0.f, 0.f, 0.f};
    if (!BWD && p.bias && kq < p.Cout) bias4 = *reinterpret_cast<const f32x4 *>(p.bias + kq);

    f32x4 acc[NP][4];
#pragma unroll
    for (int f = 0; f < NP; ++f)
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[f][a][v] = 0.f;
#pragma unroll
    for (int f = 0; f < NP; ++f)
#pragma unroll
        for (int a = 0; a < 4; ++a) asm volatile("" : "+a"(acc[f][a]));  // written here, well before the first instruction that reads them

    // ---- the loop.  A step multiplies channel blocks 0, 1 by all positions, then 2, 3.  Everything else is issued between the matrix
    // instructions, a fixed piece of it behind each pair: the filters of the step after next, into the registers of the half before;
    // the activations of the next step, behind their last use; a block of the next chunk's activations, which goes through registers
    // to the other LDS buffer two steps later.  The loads are made in every step, wanted or not (a block past the patch loads
    // nothing): the counts of loads in flight, for which the compiler waits, are constants then.
    int c = c_first, t = t_first, buf = 0, left = n_steps, t_end = c == c_last ? last - c * ntaps : ntaps;
    int blk = 0;                                                         // blocks of the next chunk requested
    // the first chunk has been on its way behind all of the above
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < WV_NBLK; ++i)
#pragma unroll
        for (int u = 0; u < 2; ++u) *reinterpret_cast<bf16x8 *>(place(i) + u * 2 * WV_PLANE) = x0[i][u];
    __syncthreads();                                                     // the table
    struct Stage {
        bf16x8 v[2];
        unsigned char *to;
        bool live;                                                       // not past the patch: lanes without a pixel all write to one place, slowly
    } stage[2];
    bf16x8 b[NP];
    unsigned xv = c_first < c_last ? xtab[0] : WV_OOB;
    auto next_chunk = [&]() {                                            // x_soff, x_none: of the chunk that is requested
        x_soff += (unsigned)(2 * HWin * 32);
        x_none = (int)(x_soff + (unsigned)(HWin * 32)) < CB * HWin * 32 ? 0u : WV_OOB;
    };
    if (c_first < c_last) next_chunk();
    auto next_block = [&]() {
        ++blk;
        return xtab[(c < c_last && blk < WV_NBLK ? blk : WV_NBLK) * 64];
    };
    // in the order of the loop, so that its counts hold in the first round as well
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        __builtin_amdgcn_sched_barrier(0);
        if (u == 1) {
            wa[u][0] = load_w(0);
            wa[u][1] = load_w(1);
        }
        __builtin_amdgcn_sched_barrier(0);
        stage[u].to = place(blk) + WV_BUF;
        stage[u].live = c < c_last && blk * 32 < p.npatch;
#pragma unroll
        for (int q = 0; q < 2; ++q) stage[u].v[q] = load_x(xv, q);
        xv = next_block();
        __builtin_amdgcn_sched_barrier(0);
        if (u == 0) {
            wa[u][2] = load_w(2);
            wa[u][3] = load_w(3);
            next_w();
        }
    }
    {
        const int off = __builtin_amdgcn_readlane(toffv, t);
#pragma unroll
        for (int f = 0; f < NP; ++f) b[f] = *reinterpret_cast<const bf16x8 *>(mine + pbase[f] + off);
    }
    __builtin_amdgcn_sched_barrier(0);
    auto step = [&](bf16x8 (&a)[4], bf16x8 (&a_prev)[4], Stage &sg) {
        int off = 0;
#pragma unroll
        for (int f = 0; f < NP; ++f) {
            mfma_acc(acc[f][0], a[0], b[f]);
            mfma_acc(acc[f][1], a[1], b[f]);
            if (f == 0) a_prev[2] = load_w(2);
            if (f == 1) a_prev[3] = load_w(3);
            if (f == 2) next_w();
            if (f == 3 && sg.live) {
                *reinterpret_cast<bf16x8 *>(sg.to) = sg.v[0];
                *reinterpret_cast<bf16x8 *>(sg.to + 2 * WV_PLANE) = sg.v[1];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        --left;
        if (++t == t_end && left > 0) {                                  // the next step is the next chunk's first
            for (int i = blk > 2 ? blk - 2 : 0; i * 32 < p.npatch; ++i) {    // few steps: what is not there yet
                const unsigned v = xtab[i * 64];
#pragma unroll
                for (int u = 0; u < 2; ++u) *reinterpret_cast<bf16x8 *>(place(i) + (buf ^ 1) * WV_BUF + u * 2 * WV_PLANE) = load_x(v, u);
            }
            t = 0;
            buf ^= 1;
            ++c;
            t_end = c == c_last ? last - c * ntaps : ntaps;
            blk = 0;
            xv = WV_OOB;
            if (c < c_last) {
                next_chunk();
                xv = xtab[0];
            }
        }
        off = buf * WV_BUF + __builtin_amdgcn_readlane(toffv, t < ntaps ? t : 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < NP; ++f) {
            mfma_acc(acc[f][2], a[2], b[f]);
            mfma_acc(acc[f][3], a[3], b[f]);
            b[f] = *reinterpret_cast<const bf16x8 *>(mine + (pbase[f] + off));
            if (f == 0) a[0] = load_w(0);
            if (f == 1) a[1] = load_w(1);
            if (f == 2) {
                sg.to = place(blk) + (buf ^ 1) * WV_BUF;
                sg.live = c < c_last && blk * 32 < p.npatch;
            }
            if (f >= 3 && f < 5) sg.v[f - 3] = load_x(xv, f - 3);
            if (f == 5) xv = next_block();
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int u = n_steps >> 1; u > 0; --u) {
        step(wa[0], wa[1], stage[0]);
        step(wa[1], wa[0], stage[1]);
    }
    if (n_steps & 1) step(wa[0], wa[1], stage[0]);
    mfma_drain();
#pragma unroll
    for (int f = 0; f < NP; ++f)
#pragma unroll
        for (int a = 0; a < 4; ++a) asm volatile("" : "+a"(acc[f][a]));

    // the mask arrives under the sum (512 -> 512 at 7x7 backwards, ReLU and channel sums 35.1 us with the loads behind it, 32.5 here)
    const bool has_mask = BWD && p.mask != nullptr;
    const __amdgpu_buffer_rsrc_t rs_mask = __builtin_amdgcn_make_buffer_rsrc((void *)p.mask, 0, has_mask ? (int)p.out_bytes : 0, 0x00020000);
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 mk[BWD ? NP : 1];
    if (has_mask) {
#pragma unroll
        for (int f = 0; f < NP; ++f) mk[BWD ? f : 0] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs_mask, (int)ooff[f], 0, 0));
    }

    // ---- sum of the four tiles: blocks 2 and 3 go to the wave of split ^ 2, block 1 of what that leaves to split ^ 1; a wave writes to
    // its own region, whose buffers nobody reads any more
    f32x4 *const box = reinterpret_cast<f32x4 *>(mine) + lane;
#pragma unroll
    for (int f = 0; f < NP; ++f)
#pragma unroll
        for (int a = 0; a < 2; ++a) box[(f * 2 + a) * 64] = acc[f][2 + a];
    __syncthreads();
    const f32x4 *const in1 = reinterpret_cast<const f32x4 *>(smem + 2 * WV_TAB * 4 + (wave ^ 2) * WV_WAVE) + lane;
#pragma unroll
    for (int f = 0; f < NP; ++f)
#pragma unroll
        for (int a = 0; a < 2; ++a) acc[f][a] += in1[(f * 2 + a) * 64];
    __syncthreads();
#pragma unroll
    for (int f = 0; f < NP; ++f) box[f * 64] = acc[f][1];
    __syncthreads();
    const f32x4 *const in2 = reinterpret_cast<const f32x4 *>(smem + 2 * WV_TAB * 4 + (wave ^ 1) * WV_WAVE) + lane;
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc((void *)p.out, 0, (int)p.out_bytes, 0x00020000);
    float cs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int f = 0; f < NP; ++f) {
        const f32x4 r = acc[f][0] + in2[f * 64] + bias4;
        u32x2 o = {pack_bf16x2_hw(r[0], r[1]), pack_bf16x2_hw(r[2], r[3])};
        if (BWD) {
            if (has_mask) {
                o[0] = relu_keep2(o[0], mk[f][0]);
                o[1] = relu_keep2(o[1], mk[f][1]);
            }
            if (p.dbp && ooff[f] != WV_OOB) {                            // the rounded, masked values as stored
                cs[0] += __uint_as_float(o[0] << 16);
                cs[1] += __uint_as_float(o[0] & 0xFFFF0000u);
                cs[2] += __uint_as_float(o[1] << 16);
                cs[3] += __uint_as_float(o[1] & 0xFFFF0000u);
            }
        } else {
            o[0] = relu_bf16x2(o[0], p.relu != 0);
            o[1] = relu_bf16x2(o[1], p.relu != 0);
        }
        __builtin_amdgcn_raw_buffer_store_b64(o, rs_out, (int)ooff[f], 0, NGC_ST_AUX);
    }
    if (BWD && p.dbp) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int x = 8; x > 0; x >>= 1) cs[v] += __shfl_xor(cs[v], x, 64);       // the 16 lanes of the same channels
        if (l16 == 0 && kq < p.Cout) *reinterpret_cast<float4 *>(p.dbp + (size_t)bx * p.dbp_ld + kq) = make_float4(cs[0], cs[1], cs[2], cs[3]);
    }
}

template <int NP, bool BWD>
static hipError_t launch_waves_t(const ConvWavesParams &p, hipStream_t st)
{
    static_assert(2 * NP * 1024 <= WV_WAVE && WV_LDS <= 160 * 1024, "LDS");
    static LdsLimitOnce lds_limit;                  // per template instantiation
    {
        const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&conv_waves_bf16<NP, BWD>));
        if (e != hipSuccess) return e;
    }
    NGC_LAUNCH((conv_waves_bf16<NP, BWD>), dim3(8 * p.per_xcd), dim3(512), WV_LDS, st, p);
    return launch_result();
}

hipError_t launch_conv_waves(const ConvWavesParams &p, hipStream_t st)
{
    return p.bwd ? launch_waves_t<7, true>(p, st) : launch_waves_t<7, false>(p, st);
}

// The tile of a node: whole images, or rows of one, up to 16 NP positions and WV_NBLK blocks of patch pixels
static bool waves_geometry(ConvWavesParams &q, int np, int max_dh, int max_dw, int min_dh, int min_dw)
{
    const int L = min_dw < 0 ? -min_dw : 0, T = min_dh < 0 ? -min_dh : 0;
    const int over_w = (q.Wout - 1) * q.sw + max_dw - (q.Win - 1), over_h = (q.Hout - 1) * q.sh + max_dh - (q.Hin - 1);
    const int R = over_w > 0 ? over_w : 0, B = over_h > 0 ? over_h : 0;
    const int maxpix = 16 * np, maxpatch = WV_MAXPATCH;
    // patch column c is image column c - L; the columns behind the image are the next row's left halo
    q.PC = q.Win + (L > R ? L : R);
    q.w0 = -L;
    if (q.PC > maxpatch || q.Wout > maxpix) return false;
    const int pr_img = q.Hin + (T > B ? T : B);                          // rows of an image, the halo between two shared
    // the last row needs R columns behind it, of which the row has PC - Win - L; the last image B rows and its row has pr_img - Hin - T
    const int tail_c = R - (q.PC - q.Win - L), tail_r = B - (pr_img - q.Hin - T);
    auto patch = [&](int rows, int tail_rows) { return (rows + (tail_rows > 0 ? tail_rows : 0)) * q.PC + (tail_c > 0 ? tail_c : 0); };
    int tn = maxpix / (q.Hout * q.Wout);
    while (tn > 1 && patch(tn * pr_img, tail_r) > maxpatch) --tn;
    if (tn >= 1 && patch(tn * pr_img, tail_r) <= maxpatch) {
        // as many images a workgroup as leaves no workgroup much emptier than the others
        const int groups = (q.N + tn - 1) / tn;
        q.TN = (q.N + groups - 1) / groups;
        q.TP = q.Hout;
        q.PR = pr_img;
        q.h0 = -T;
        q.row_base = 0;
        q.npatch = patch(q.TN * pr_img, tail_r);
    } else {
        const int span = max_dh - min_dh;
        int rows = maxpix / q.Wout;
        while (rows >= 1 && patch((rows - 1) * q.sh + span + 1, 0) > maxpatch) --rows;
        if (rows < 1) return false;
        const int strips = (q.Hout + rows - 1) / rows;
        q.TN = 1;
        q.TP = (q.Hout + strips - 1) / strips;
        q.PR = (q.TP - 1) * q.sh + span + 1;
        q.h0 = min_dh;
        q.row_base = min_dh + T;                                         // tap offsets count from row -T
        q.npatch = patch(q.PR, 0);
    }
    return true;
}

// Forward (op 0), or backprop-data with stride 1; tdh / tdw: input offset of the taps
bool conv_waves_plan(const ngc_conv_desc *d, int op, int P, int Q, double staged_us, ConvWavesParams *out)
{
    const char *force = env_switch(SW_WAVES);            // tests / benchmarks only: 0 = never, 1 = wherever it can
    const int fv = force ? atoi(force) : -1;
    if (fv == 0) return false;
    const bool fwd = op == NGC_OP_FWD;
    if (!fwd && (d->stride_h != 1 || d->stride_w != 1)) return false;
    const int ntaps = d->r * d->s, Cin = fwd ? d->c : d->k, Cout = fwd ? d->k : d->c;
    if (ntaps < 2 || ntaps > STRIP_MAX_TAPS || Cin % 16 || Cout % 16) return false;
    ConvWavesParams q;
    memset(&q, 0, sizeof(q));
    q.N = d->n; q.Cin = Cin; q.Cout = Cout;
    q.Hin = fwd ? d->h : P; q.Win = fwd ? d->w : Q;
    q.Hout = fwd ? P : d->h; q.Wout = fwd ? Q : d->w;
    q.sh = fwd ? d->stride_h : 1; q.sw = fwd ? d->stride_w : 1;
    q.bwd = !fwd;
    const size_t lim = (size_t)1 << 31, in_bytes = (size_t)d->n * Cin * q.Hin * q.Win * 2, wt_bytes = (size_t)ntaps * Cin * Cout * 2,
                 out_bytes = (size_t)d->n * Cout * q.Hout * q.Wout * 2;
    if (in_bytes >= lim || wt_bytes >= lim || out_bytes >= lim) return false;
    q.in_bytes = (uint32_t)in_bytes; q.wt_bytes = (uint32_t)wt_bytes; q.out_bytes = (uint32_t)out_bytes;
    int tdh[STRIP_MAX_TAPS], tdw[STRIP_MAX_TAPS], lo_h = 0, hi_h = 0, lo_w = 0, hi_w = 0;
    for (int t = 0; t < ntaps; ++t) {
        const int r = t / d->s, s = t % d->s;
        tdh[t] = fwd ? r * d->dil_h - d->pad_below_h : d->pad_below_h - r * d->dil_h;
        tdw[t] = fwd ? s * d->dil_w - d->pad_below_w : d->pad_below_w - s * d->dil_w;
        if (t == 0 || tdh[t] < lo_h) lo_h = tdh[t];
        if (t == 0 || tdh[t] > hi_h) hi_h = tdh[t];
        if (t == 0 || tdw[t] < lo_w) lo_w = tdw[t];
        if (t == 0 || tdw[t] > hi_w) hi_w = tdw[t];
    }
    q.ntaps = ntaps;
    const int steps = (Cin + 31) / 32 * ntaps;
    if (steps < 8) return false;                         // every wave has at least two steps
    if (!waves_geometry(q, 7, hi_h, hi_w, lo_h, lo_w)) return false;
    q.strips = (q.Hout + q.TP - 1) / q.TP;
    q.groups = (q.N + q.TN - 1) / q.TN;
    q.npix = q.TN * q.TP * q.Wout;
    const int nk = (Cout + 63) / 64;
    if ((size_t)q.strips * q.groups * nk > (1u << 24)) return false;
    q.tiles = (q.strips * q.groups + 1) / 2 * nk;
    q.per_xcd = (q.tiles + 7) / 8;
    if (fv < 0 && staged_us >= 0) {
        // A switch that shapes the strip kernel, or rules out another one in its favour, asks for it
        for (Switch sw : {SW_STRIP_NF, SW_STRIP_ROWS, SW_STRIP_BW, SW_STRIP_XCD, SW_STRIP_TAIL, SW_STRIP_SPLIT, SW_STRIP_CPS, SW_STRIP_STRIDED, SW_ROWS, SW_FWD_FEW})
            if (env_switch(sw)) return false;
        // Expected time, us: a start and, per round of workgroups, start, sum and stores and the steps of a wave; the bytes: patches
        // loaded, tensors read and written.  Fitted as strip_node_us, nine tenths within 8 % below and 16 % above.  The strip kernel gains
        // with the size of its strips and of a launch, this one with the length of the reduction: 3351 of 31617 drawn
        // launches are taken, 120622 -> 102889 us, 51 above 1.05 of the strip kernel's time; of 10569 others 1170, 41996 -> 35491, 14 above,
        // 1.15 at worst.
        const double rounds = (q.tiles + 255) / 256, patch_mb = 4e-6 * q.tiles * q.npatch * Cin;
        const double us = 2.99 + rounds * (4.2 + 0.538 * ((steps + 3) / 4)) + 0.051 * patch_mb + 0.0494e-6 * in_bytes + 0.0295e-6 * out_bytes;
        if (us >= 0.97 * staged_us) return false;            // no estimate (0): never
    }
    const int L = lo_w < 0 ? -lo_w : 0, T = lo_h < 0 ? -lo_h : 0;
    // LDS offset of tap (r, s): tap0 + r tap_dr + s tap_ds
    q.S = d->s;
    q.tap0 = ((tdh[0] + T - q.row_base) * q.PC + tdw[0] + L) * 16;
    q.tap_dr = (fwd ? d->dil_h : -d->dil_h) * q.PC * 16;
    q.tap_ds = (fwd ? d->dil_w : -d->dil_w) * 16;
    q.div_nk = make_fastdiv((uint32_t)nk);
    q.div_strips = make_fastdiv((uint32_t)q.strips);
    q.div_taps = make_fastdiv((uint32_t)ntaps);
    auto rcp = [](int v) { return 65536 / v + 1; };
    q.rcp_pc = rcp(q.PC); q.rcp_pr = rcp(q.PR); q.rcp_q = rcp(q.Wout); q.rcp_tp = rcp(q.TP); q.rcp_s = rcp(q.S);
    if (out) *out = q;
    return true;
}

int conv_waves_dbp_rows(const ConvWavesParams &p) { return (p.groups * p.strips + 1) / 2 * 2; }

}  // namespace ngc
