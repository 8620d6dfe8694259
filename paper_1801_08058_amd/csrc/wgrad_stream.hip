// Backprop-filters of the nodes of conv_gather.hip whose tensors are NCHW, operands straight from memory to registers
// (gfx950): fp32 tensors and bf16 ones with channel counts that are no multiple of 16.
//
//   dw[k][c, r, s] = sum over positions of dy[k][pos] * x[c][pos * stride + (r, s) * dilation - padding]
//
// As conv_stream.hip for the other two ops: no operand goes through LDS.  The reduction runs along the rows of dy in units of
// U consecutive positions (4 fp32, 8 bf16: 16 bytes), a step is two units, one for each half of a wave.  A lane loads the unit
// of its k from dy as it lies in memory, and for its column (c, r, s) the same positions of x, 16 bytes at any element
// where the column stride is 1; elements in the padding or past the end of a row are masked in the units at the edges of
// rows.  A workgroup takes 32 k x 32 columns for a part of the positions, its four waves take turns with the steps, the next
// step's loads in flight.
//
// What bounds it: see stream_conv; a load whose lanes lie in 32 rows is served a row at a time.
//
// Sums: fp32 a step's products in a chain of 8 positions, every other step (bf16: those in one chain), for few parts 4 of
// these at a time.  Relative 2-norm error against 64 bits over 26 drawn nodes of each type: 0.97 to 0.98 of the gather GEMM's.
//
// Gather GEMM / now, with the second launch of split reductions, us: fp32 3x3 64 -> 96, 8 x 45 x 37 46.4 / 37.9, 16 -> 32, 2 x 16 x 16
// 8.8 / 6.4, 5x5 45 -> 29, 4 x 42 x 43 31.0 / 19.1; bf16 3x3 40 -> 72, 8 x 28 x 28 17.6 / 12.3, 1x1 94 -> 9, 37 x 18 10.7 / 5.6.  Two
// fragments of either operand a wave measured 1 to 1.6 times the time: fewer waves to cover the loads with.
#include "conv_gather.h"

#include <limits.h>
#include <stdlib.h>

namespace ngc {

struct WgradStreamParams {
    const void *x, *dy;
    float *out;                    // [parts][pitch] partial sums, or dw itself (one part)
    uint32_t x_bytes, dy_bytes;    // bf16: in whole dwords
    int32_t C, H, W, K, P, Q, R, S;
    int32_t sh, sw, dil_h, dil_w, pb_h, pb_w;
    int32_t ctiles;
    uint32_t units, chunk;         // units of all rows; of a part (a multiple of 2)
    uint32_t pitch;                // floats between the parts
    FastDiv div_qu, div_p;         // units of a row, rows of an image
};

// U elements from byte offset off on, any element alignment; nothing past the end of the descriptor
template <typename T> __device__ __forceinline__ uint4 load_unit(__amdgpu_buffer_rsrc_t rs, unsigned off);
template <> __device__ __forceinline__ uint4 load_unit<float>(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}
template <> __device__ __forceinline__ uint4 load_unit<uint16_t>(__amdgpu_buffer_rsrc_t rs, unsigned off) { return load_bf16x8(rs, off); }

// elements lo .. hi - 1 of a unit, zeros elsewhere
template <typename T>
__device__ __forceinline__ uint4 unit_mask(uint4 v, int lo, int hi)
{
    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (sizeof(T) == 4) w[i] = i >= lo && i < hi ? w[i] : 0;
        else w[i] &= (2 * i >= lo && 2 * i < hi ? 0xFFFFu : 0u) | (2 * i + 1 >= lo && 2 * i + 1 < hi ? 0xFFFF0000u : 0u);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// the unit moved up by n elements (what comes in below is masked by the caller)
template <typename T>
__device__ __forceinline__ uint4 unit_shift(uint4 v, int n)
{
#pragma unroll 1
    for (int i = 0; i < n && i < GElem<T>::U; ++i) {
        if constexpr (sizeof(T) == 4) v = make_uint4(v.x, v.x, v.y, v.z);
        else v = make_uint4(v.x << 16, __builtin_amdgcn_alignbit(v.y, v.x, 16), __builtin_amdgcn_alignbit(v.z, v.y, 16), __builtin_amdgcn_alignbit(v.w, v.z, 16));
    }
    return v;
}

template <typename T, bool SW1, bool LONG>
__global__ __launch_bounds__(256) void wgrad_stream(const WgradStreamParams p)
{
    preload_kernargs(p);
    constexpr int U = GElem<T>::U, KS = 4;
    constexpr unsigned SZ = sizeof(T);
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int slice = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int kt = (int)blockIdx.y / p.ctiles, ct = (int)blockIdx.y - kt * p.ctiles;
    const int k0 = kt * 32, RS = p.R * p.S, CRS = p.C * RS, PQ = p.P * p.Q, HW = p.H * p.W;
    const unsigned u0 = blockIdx.x * p.chunk, u1 = u0 + p.chunk < p.units ? u0 + p.chunk : p.units;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc((void *)p.dy, 0, (int)p.dy_bytes, 0x00020000);

    // this lane's rows of both operands
    const int krow = k0 + l32, koff = krow < p.K ? krow * PQ : -1;
    const int col = ct * 32 + l32, c = col / RS, tap = col - c * RS, r = tap / p.S;
    const int xdh = r * p.dil_h - p.pb_h, xdw = (tap - r * p.S) * p.dil_w - p.pb_w;
    const int xoff = c * HW + xdh * p.W + xdw;
    const bool cok = col < CRS;

    // columns that are inside for every lane when a unit starts at column q: q sw >= edge_lo and q sw <= edge_hi
    const int edge_lo = p.pb_w, edge_hi = p.W - 1 - (U - 1) * p.sw - ((p.S - 1) * p.dil_w - p.pb_w);

    uint4 kv[2], xv[2];
    uint32_t xe[2][U];
    int klive[2];                                                        // live positions of this half's unit
    int q_of[2];                                                         // its first column
    int up[2];                                             // elements by which x has to be moved up
    auto request = [&](int set, unsigned step) {
        const unsigned u = u0 + 2 * step + half;
        const bool live = u < u1;
        const unsigned row = fd_div(u, p.div_qu);
        const int q = (int)(u - row * p.div_qu.d) * U;
        const int n = (int)fd_div(row, p.div_p), pp = (int)(row - (unsigned)n * p.div_p.d);
        klive[set] = live ? p.Q - q : 0;
        q_of[set] = q;
        const int ybase = n * p.K * PQ + pp * p.Q + q;
        kv[set] = load_unit<T>(rs_dy, live && koff >= 0 ? (unsigned)(ybase + koff) * SZ : GATHER_OOB);
        const int at = n * p.C * HW + pp * p.sh * p.W + q * p.sw + xoff;
        const bool in = live && cok && (unsigned)(pp * p.sh + xdh) < (unsigned)p.H;
        if constexpr (SW1) {
            // a unit that starts in the padding in front of the tensor is loaded from element 0 on and moved into place below
            up[set] = in && at < 0 ? -at : 0;
            xv[set] = load_unit<T>(rs_x, in ? (unsigned)(at < 0 ? 0 : at) * SZ : GATHER_OOB);
        } else {
#pragma unroll
            for (int e = 0; e < U; ++e)
                xe[set][e] = GElem<T>::load(rs_x, in && (unsigned)((q + e) * p.sw + xdw) < (unsigned)p.W ? (unsigned)(at + e * p.sw) * SZ : GATHER_OOB);
        }
    };

    constexpr gf32x16 ZERO = {};
    gf32x16 acc[2] = {ZERO, ZERO}, total = ZERO;                         // every other step, and 8 steps at a time
    auto multiply = [&](int set, unsigned step) {
        uint4 a = kv[set], b = xv[set];
        if constexpr (!SW1) {
            keep_raw(xe[set]);
            b = GElem<T>::pack(xe[set]);
        }
        // units at the edge of a row: positions past its end, columns in the padding (uniform branches)
        const bool tail = __builtin_amdgcn_ballot_w64(klive[set] < U) != 0;
        if (tail) a = unit_mask<T>(a, 0, klive[set]);
        if constexpr (SW1) {
            const int q = q_of[set];
            if (tail || __builtin_amdgcn_ballot_w64(q < edge_lo || q > edge_hi) != 0) {
                if (__builtin_amdgcn_ballot_w64(up[set] > 0) != 0) b = unit_shift<T>(b, up[set]);
                const int w = q + xdw;                                   // image column of the unit's first element
                b = unit_mask<T>(b, -w, p.W - w);
            }
        }
        if constexpr (sizeof(T) == 4) acc[set] += mma_pair<T>(a, b, ZERO);
        else acc[set] = mma_pair<T>(a, b, acc[set]);
        if (LONG && set == 1 && ((step / KS) & 7) == 7) {
            total += acc[0] + acc[1];
            acc[0] = acc[1] = ZERO;
        }
    };
    const unsigned nsteps = (u1 - u0 + 1) >> 1;
    request(0, slice);
    for (unsigned step = slice; step < nsteps; step += 2 * KS) {
        request(1, step + KS);                                           // past the end: out of range, zeros
        multiply(0, step);
        request(0, step + 2 * KS);
        multiply(1, step + KS);
    }
    acc[0] += acc[1];
    if (LONG) acc[0] += total;
    // slice z adds up the register group (4 rows) z over all slices
    float *red = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int v = 0; v < 16; ++v) red[(slice * 16 + v) * 64 + lane] = acc[0][v];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier_nofence();
    float sum[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sum[e] = 0.f;
#pragma unroll
        for (int z = 0; z < KS; ++z) sum[e] += red[(z * 16 + slice * 4 + e) * 64 + lane];
    }
    if (!cok) return;
    const int k = k0 + 8 * slice + 4 * half;
    // Positions past the end of a row and taps in the padding are no part of the sum; the zeros in their place give NaN against
    // an infinite or NaN factor.  Sums that came out as NaN are added up again without them.
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(__builtin_isunordered(sum[0], sum[1]) || __builtin_isunordered(sum[2], sum[3])) != 0, 0)) {
        float again[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (unsigned u = u0; u < u1; ++u) {
            const unsigned row = fd_div(u, p.div_qu);
            const int q0 = (int)(u - row * p.div_qu.d) * U, n = (int)fd_div(row, p.div_p), pp = (int)(row - (unsigned)n * p.div_p.d);
            if ((unsigned)(pp * p.sh + xdh) >= (unsigned)p.H) continue;
#pragma unroll 1
            for (int q = q0; q < q0 + U && q < p.Q; ++q) {
                if ((unsigned)(q * p.sw + xdw) >= (unsigned)p.W) continue;
                const float x = load_value<T>(rs_x, (unsigned)(n * p.C * HW + pp * p.sh * p.W + q * p.sw + xoff) * SZ);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    again[e] = fmaf(load_value<T>(rs_dy, k + e < p.K ? (unsigned)((n * p.K + k + e) * PQ + pp * p.Q + q) * SZ : GATHER_OOB), x, again[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] = sum[e] != sum[e] ? again[e] : sum[e];
    }
    float *out = p.out + (size_t)blockIdx.x * p.pitch;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (k + e < p.K) out[(size_t)(k + e) * CRS + col] = sum[e];
}

// ---------------------------------------------------------------------------------------------- host side

struct StreamWgradPlan {
    int parts, P, Q, H, W;                             // the node's rows, or all of an image as one row
    uint32_t units, chunk;
};

static bool stream_wgrad_plan(const ngc_conv_desc &d, int P, int Q, StreamWgradPlan *pl)
{
    const char *force = env_switch(SW_WGRAD_STREAM);                     // tests only: 0 = never, else that many parts
    const int fv = force ? atoi(force) : -1;
    if (fv == 0 || env_switch(SW_GATHER_WGRAD)) return false;            // a switch that shapes the gather kernel asks for it
    if (d.x_layout != NGC_NCHW || d.y_layout != NGC_NCHW) return false;
    // bf16, one tap, many channels on both sides: the gather GEMM's 64 x 64 tiles read less (130 -> 219 at 4 x 56x35 11.1 / 13.4 us here,
    // 233 -> 192 at 8 x 52x57, stride 2 22.6 / 26.0; 155 -> 90 at 22 x 24x22 10.0 / 9.5)
    if (fv < 0 && d.dtype == NGC_BF16 && d.r * d.s == 1 && d.c >= 128 && d.k >= 128) return false;
    pl->P = P; pl->Q = Q; pl->H = d.h; pl->W = d.w;
    if (d.r == 1 && d.s == 1 && d.stride_h == 1 && d.stride_w == 1 && P == d.h && Q == d.w && d.pad_below_h == 0 && d.pad_below_w == 0) {
        pl->Q = pl->W = P * Q;
        pl->P = pl->H = 1;
    }
    const int U = d.dtype == NGC_F32 ? 4 : 8;
    const size_t CRS = (size_t)d.c * d.r * d.s, tiles = (size_t)((d.k + 31) / 32) * ((CRS + 31) / 32);
    pl->units = (uint32_t)((size_t)d.n * pl->P * ((pl->Q + U - 1) / U));
    if (tiles > 65535) return false;
    // Parts of the positions by expected time, fitted to 23 drawn nodes in 1 to 64 parts each (within 7 % fp32, 17 % bf16): steps of a
    // wave, a second launch to add up the parts and its bytes.  Over 297 others the choice costs 4 % over the best count of 1 to 128 on
    // average, a sixth of them 10 % and more, 43 % at most.  A term in the workgroups per compute unit fitted to those halves that, but
    // 400 further nodes take 0.997 of the time with it, three of them 1.12 to 1.2.
    const bool f32 = d.dtype == NGC_F32;
    const size_t most = pl->units / 16 ? pl->units / 16 : 1, cap = ((size_t)16 << 20) / ((d.k * CRS + 15) / 16 * 64);
    double best = 0;
    pl->parts = 0;
    for (int i = 0; i < 17; ++i) {                                       // 1, 2, 3, 4, 6, 8, 12 .. 256
        size_t parts = i == 0 ? 1 : (i & 1) ? (size_t)2 << (i >> 1) : (size_t)3 << ((i >> 1) - 1);
        if (fv > 0) parts = (size_t)fv;
        if (parts > most) parts = most;
        if (parts > cap) parts = cap;
        if (parts > 256) parts = 256;
        if (parts < 1) parts = 1;
        const uint32_t chunk = (uint32_t)((pl->units + parts - 1) / parts + 1) / 2 * 2;
        const int n = (int)((pl->units + chunk - 1) / chunk);
        const double t = (f32 ? 0.418 : 0.392) * ((chunk / 2 + 3) / 4) + (n > 1 ? (f32 ? 2.65 : 2.97) + (f32 ? 1.23e-6 : 1.31e-6) * n * (double)(d.k * CRS) * 4 : 0);
        if (!pl->parts || t < best) {
            best = t;
            pl->parts = n;
            pl->chunk = chunk;
        }
    }
    return true;
}

static uint32_t stream_wgrad_pitch(const ngc_conv_desc &d) { return (uint32_t)(((size_t)d.k * d.c * d.r * d.s + 15) / 16 * 16); }

size_t wgrad_stream_workspace(const ngc_conv_desc &d, int P, int Q, bool *takes)
{
    StreamWgradPlan pl;
    *takes = stream_wgrad_plan(d, P, Q, &pl);
    return *takes && pl.parts > 1 ? (size_t)pl.parts * stream_wgrad_pitch(d) * sizeof(float) : 0;
}

template <typename T, bool SW1>
static hipError_t launch_wgrad_stream_t(const WgradStreamParams &p, const StreamWgradPlan &pl, bool longsum, hipStream_t st)
{
    const dim3 grid((unsigned)pl.parts, (unsigned)((p.K + 31) / 32) * p.ctiles);
    if (longsum) NGC_LAUNCH((wgrad_stream<T, SW1, true>), grid, dim3(256), 4 * 4096, st, p);
    else NGC_LAUNCH((wgrad_stream<T, SW1, false>), grid, dim3(256), 4 * 4096, st, p);
    return launch_result();
}

bool launch_wgrad_stream(const ngc_conv_desc &d, int P, int Q, const void *x, const void *dy, float *dw, void *ws, size_t ws_bytes, hipStream_t st, hipError_t *e)
{
    StreamWgradPlan pl;
    if (!stream_wgrad_plan(d, P, Q, &pl)) return false;
    WgradStreamParams p = {};
    p.pitch = stream_wgrad_pitch(d);
    if (pl.parts > 1 && (!ws || ws_bytes < (size_t)pl.parts * p.pitch * sizeof(float))) return false;
    const uint32_t sz = d.dtype == NGC_F32 ? 4 : 2, U = 16 / sz;
    p.x = x; p.dy = dy;
    p.out = pl.parts > 1 ? static_cast<float *>(ws) : dw;
    // an odd last bf16 element is in range with its dword (tensors start on 16 bytes)
    p.x_bytes = (uint32_t)(((size_t)d.n * d.c * d.h * d.w * sz + 3) & ~(size_t)3);
    p.dy_bytes = (uint32_t)(((size_t)d.n * d.k * P * Q * sz + 3) & ~(size_t)3);
    p.C = d.c; p.H = pl.H; p.W = pl.W; p.K = d.k; p.P = pl.P; p.Q = pl.Q; p.R = d.r; p.S = d.s;
    p.sh = d.stride_h; p.sw = d.stride_w; p.dil_h = d.dil_h; p.dil_w = d.dil_w; p.pb_h = d.pad_below_h; p.pb_w = d.pad_below_w;
    p.ctiles = (d.c * d.r * d.s + 31) / 32;
    p.units = pl.units;
    p.chunk = pl.chunk;
    p.div_qu = make_fastdiv((uint32_t)((pl.Q + (int)U - 1) / (int)U));
    p.div_p = make_fastdiv((uint32_t)pl.P);
    const bool longsum = pl.chunk > 2 * 4 * 32;                          // more than 32 steps a wave
    if (d.dtype == NGC_F32) *e = d.stride_w == 1 ? launch_wgrad_stream_t<float, true>(p, pl, longsum, st) : launch_wgrad_stream_t<float, false>(p, pl, longsum, st);
    else *e = d.stride_w == 1 ? launch_wgrad_stream_t<uint16_t, true>(p, pl, longsum, st) : launch_wgrad_stream_t<uint16_t, false>(p, pl, longsum, st);
    if (*e == hipSuccess && pl.parts > 1) *e = launch_bias_grad_reduce(p.out, dw, pl.parts, d.k * d.c * d.r * d.s, (int)p.pitch, st);
    return true;
}

}  // namespace ngc
