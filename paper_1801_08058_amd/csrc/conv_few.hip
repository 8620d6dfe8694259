// Forward of blocked bf16 nodes with few output tiles (gfx950): one image, or a few small ones.
//
// The strip kernel and the 1x1 GEMM give such a node a handful of workgroups, each of which walks all channels and taps in a
// chain of stages through LDS at some 0.4 us a stage, while most compute units idle.  Here a workgroup takes a tile of 32
// output channels x 32 positions and its waves split the reduction: the (tap, 16-channel block) units are dealt to NW waves,
// whose operands go straight from memory to the registers - both blocked layouts hold the 8 consecutive channels of an MFMA
// lane as 16 bytes, a wave reads 1 KB of each - eight units of loads in flight at a time.  No LDS ring, no barrier but the one in
// front of the sum of the waves' tiles.
//
// One image, staged kernels / this one, us: 1x1 1024 -> 256 at 14x14 13.4 / 3.6 (16 workgroups / 56), 2048 -> 512 at 7x7 21.9 / 4.1,
// 3x3 256 -> 256 at 14x14 18.0 / 6.2 (4 workgroups / 56), 512 -> 512 at 7x7 30.1 / 7.8.
//
// Bound: the latency of U / (8 NW) batches of loads and of the sum; many tiles: the L2 reads, 2 KB per MFMA, which is why the
// staged kernels keep the larger nodes (conv_few_plan).  Elements in the padding and channels past the end read as zeros
// through out-of-range offsets.
#include "common.h"

#include <stdlib.h>
#include <string.h>

namespace ngc {

typedef __bf16 fbf16x8 __attribute__((ext_vector_type(8)));
typedef float ff32x16 __attribute__((ext_vector_type(16)));

constexpr unsigned FEW_OOB = 0x80000000u;              // past the end of every descriptor below 2 GiB

template <int NW>
__global__ __launch_bounds__(64 * NW) void conv_few_bf16(const ConvFewParams p)
{
    constexpr int B = 8;                               // units in flight
    __shared__ float4 red[NW][4][64];
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int k0 = blockIdx.y * 32;
    const uint32_t pos = blockIdx.x * 32 + (lane & 31);
    const bool live = pos < p.M;
    const uint32_t n = fd_div(pos, p.div_pq), pq = pos - n * p.div_pq.d;
    const int op = (int)fd_div(pq, p.div_q), oq = (int)(pq - (uint32_t)op * p.div_q.d);
    const int ih0 = op * p.sh - p.pbh, iw0 = oq * p.sw - p.pbw;
    const unsigned plane = (unsigned)(p.H * p.W * 32);
    const unsigned x_base = n * (unsigned)p.CB * plane + half * 16;
    const bool krow = k0 + (lane & 31) < p.K;
    const unsigned w_base = (unsigned)(k0 + (lane & 31)) * 32 + half * 16;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.in), 0, (int)p.in_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.wt), 0, (int)p.wt_bytes, 0x00020000);

    ff32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    // unit = tap * CB + cb; this wave's units are wave, wave + NW, ..
    const int U = p.R * p.S * p.CB;
    int cb = wave, r = 0, s = 0;
    for (int u0 = wave; u0 < U; u0 += NW * B) {
        __uint128_t xv[B], wv[B];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const int u = u0 + j * NW;
            while (cb >= p.CB) {                       // next tap: at most NW times, CB >= 1
                cb -= p.CB;
                if (++s == p.S) {
                    s = 0;
                    ++r;
                }
            }
            const int ih = ih0 + r * p.dil_h, iw = iw0 + s * p.dil_w;
            const bool okx = live && u < U && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
            const unsigned xo = x_base + (unsigned)cb * plane + (unsigned)(ih * p.W + iw) * 32;
            const unsigned wo = w_base + (unsigned)u * (unsigned)p.K * 32;
            xv[j] = __builtin_bit_cast(__uint128_t, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(okx ? xo : FEW_OOB), 0, 0));
            wv[j] = __builtin_bit_cast(__uint128_t, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(krow && u < U ? wo : FEW_OOB), 0, 0));
            cb += NW;
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(fbf16x8, wv[j]), __builtin_bit_cast(fbf16x8, xv[j]), acc, 0, 0, 0);
    }
    // acc[4 q + v]: channel k0 + 8 q + 4 half + v of position lane % 32
#pragma unroll
    for (int q = 0; q < 4; ++q) red[wave][q][lane] = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
    __syncthreads();
    if (wave >= 4) return;                             // wave q sums the quads q
    const int k = k0 + 8 * wave + 4 * half;
    if (!live || k >= p.K) return;
    float f[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias) {
#pragma unroll
        for (int v = 0; v < 4; ++v) f[v] = p.bias[k + v];
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {                     // fixed order
        const float4 t = red[w][wave][lane];
        f[0] += t.x; f[1] += t.y; f[2] += t.z; f[3] += t.w;
    }
    uint2 o = make_uint2(pack_bf16x2_hw(f[0], f[1]), pack_bf16x2_hw(f[2], f[3]));
    o.x = relu_bf16x2(o.x, p.relu);
    o.y = relu_bf16x2(o.y, p.relu);
    const size_t at = (((size_t)n * (p.K >> 4) + (k >> 4)) * p.div_pq.d + pq) * 16 + (k & 15);
    *reinterpret_cast<uint2 *>(p.out + at) = o;
}

bool conv_few_plan(const ngc_conv_desc *d, int P, int Q, ConvFewParams *q)
{
    const char *force = env_switch(SW_FWD_FEW);        // tests / benchmarks only: 0 = never, 1 = wherever it can
    const int fv = force ? atoi(force) : -1;
    if (fv == 0 || d->c % 16 || d->k % 16) return false;
    // a switch that shapes the staged kernels asks for them
    for (Switch sw : {SW_STRIP_NF, SW_STRIP_ROWS, SW_STRIP_BW, SW_STRIP_XCD, SW_STRIP_TAIL, SW_STRIP_SPLIT, SW_STRIP_CPS, SW_STRIP_STRIDED, SW_G1_VARIANT, SW_ROWS})
        if (env_switch(sw)) return false;
    const size_t in_bytes = (size_t)d->n * d->c * d->h * d->w * 2, wt_bytes = (size_t)d->r * d->s * d->c * d->k * 2;
    const size_t M = (size_t)d->n * P * Q;
    if (in_bytes >= ((size_t)1 << 31) || wt_bytes >= ((size_t)1 << 31) || M * d->k * 2 >= ((size_t)1 << 31) || M >= ((size_t)1 << 24) || d->k > 32 * 65535) return false;
    const size_t tiles = (M + 31) / 32 * ((d->k + 31) / 32), units = (size_t)d->r * d->s * (d->c / 16);
    // One round of workgroups (256 compute units) and a reduction worth dealing out, or most of two rounds and a long one.  Staged
    // kernel / this one, us: 224 tiles of 16 units (256 -> 1024 at 14x14) 5.4 / 3.5, 98 of 8 4.4 / 3.3, 4 of 18 4.4 / 3.9, 104 of 4
    // 3.6 / 3.6; 392 tiles of 36 7.3 / 4.5, 448 of 32 8.0 / 4.4, 400 of 288 35.1 / 17.0, but 392 of 18 5.3 / 5.5 and 400 of 8 4.3 / 4.4;
    // 784 tiles of 144 18.4 / 19.5, of 16 6.0 / 6.7.
    if (fv != 1 && !(tiles <= 256 && units >= 8) && !(tiles <= 448 && units >= 32)) return false;
    if (!q) return true;
    memset(q, 0, sizeof(*q));
    q->in_bytes = (uint32_t)in_bytes;
    q->wt_bytes = (uint32_t)wt_bytes;
    q->M = (uint32_t)M;
    q->CB = d->c / 16; q->K = d->k;
    q->H = d->h; q->W = d->w; q->R = d->r; q->S = d->s;
    q->sh = d->stride_h; q->sw = d->stride_w; q->dil_h = d->dil_h; q->dil_w = d->dil_w;
    q->pbh = d->pad_below_h; q->pbw = d->pad_below_w;
    q->div_pq = make_fastdiv((uint32_t)(P * Q));
    q->div_q = make_fastdiv((uint32_t)Q);
    return true;
}

hipError_t launch_conv_few(const ConvFewParams &p, hipStream_t st)
{
    const dim3 grid((p.M + 31) / 32, (unsigned)(p.K + 31) / 32);
    if (p.R * p.S * p.CB > 64) NGC_LAUNCH((conv_few_bf16<16>), grid, dim3(1024), 0, st, p);
    else NGC_LAUNCH((conv_few_bf16<8>), grid, dim3(512), 0, st, p);
    return launch_result();
}

}  // namespace ngc
