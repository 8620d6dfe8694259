// Shared by the two kernels of the nodes that the blocked bf16 kernels do not take (conv_gather.hip: operands gathered
// element by element through LDS; conv_stream.hip: straight to registers): the arguments of forward and
// backprop-data, element types, epilogue.
#pragma once
#include "common.h"

namespace ngc {

typedef __bf16 gbf16x8 __attribute__((ext_vector_type(8)));
typedef float gf32x4 __attribute__((ext_vector_type(4)));
typedef float gf32x16 __attribute__((ext_vector_type(16)));

constexpr unsigned GATHER_OOB = 0x80000000u;           // past the end of every descriptor below 2 GiB: reads as zero

constexpr int GATHER_CLASSES = 4;

struct GatherConvParams {
    const void *in, *wt;
    void *out;
    const float *bias;             // may be null
    const void *mask;              // may be null; else shaped like out: out = (mask > 0) ? out : 0
    uint32_t in_bytes, wt_bytes;
    int32_t N, Cin, Cout, Hin, Win, Hout, Wout;
    int32_t in_n, in_c, in_px;     // elements between images, channels (blocked: 16-channel blocks), pixels
    int32_t in_blocked, out_blocked;
    int32_t w_row, w_chan;         // filter elements between output channels and between reduction channels
    int32_t S;                     // filter columns
    int32_t is_h, is_w;            // input pixels per lattice step (forward: the stride)
    int32_t os_h, os_w;            // output pixels per lattice step (backprop-data: the stride, at most GATHER_CLASSES)
    int32_t rst_h, rst_w;          // filter rows / columns between the taps of a class (forward: 1)
    int32_t step_h, step_w;        // input rows / columns between the taps of a class (forward: dilation; backprop-data: negative)
    // residue classes of the output rows / columns modulo os: first tap, number of taps (at most 31), input row / column of
    // the first tap at lattice row / column 0, lattice extent
    int32_t r0[GATHER_CLASSES], nr[GATHER_CLASSES], base_h[GATHER_CLASSES], oph[GATHER_CLASSES];
    int32_t s0[GATHER_CLASSES], ns[GATHER_CLASSES], base_w[GATHER_CLASSES], opw[GATHER_CLASSES];
    FastDiv div_pq[4], div_q[2];   // by the lattice extents: index 2 * (oph != oph[0]) + (opw != opw[0]), and the latter
    int32_t relu;
    int32_t wvec;                  // gather GEMM: a filter row is whole 16-byte pieces in the order of the reduction
};

template <typename T> struct GElem;
template <> struct GElem<float> {
    static constexpr int U = 4;
    __device__ static uint32_t load(__amdgpu_buffer_rsrc_t rs, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0); }
    __device__ static uint4 pack(const uint32_t (&v)[4]) { return make_uint4(v[0], v[1], v[2], v[3]); }
    __device__ static float widen(float v) { return v; }
};
template <> struct GElem<uint16_t> {
    static constexpr int U = 8;
    __device__ static uint32_t load(__amdgpu_buffer_rsrc_t rs, unsigned off) { return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)off, 0, 0); }
    __device__ static uint4 pack(const uint32_t (&v)[8]) { return make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16); }
    __device__ static float widen(uint16_t v) { return bf16_bits_to_float(v); }
};

// Elements in flight stay as they were loaded until they are staged: without this the compiler packs the pairs of a step as
// soon as it has requested them, in front of the barrier, and every step waits for its own loads.
template <int N> __device__ __forceinline__ void keep_raw(uint32_t (&v)[N])
{
#pragma unroll
    for (int e = 0; e < N; ++e) asm volatile("" : "+v"(v[e]));
}

template <typename T>
__device__ __forceinline__ float load_value(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    const uint32_t v = GElem<T>::load(rs, off);
    if constexpr (sizeof(T) == 4) return __uint_as_float(v);
    else return GElem<T>::widen((uint16_t)v);
}

__device__ __forceinline__ unsigned bit_mask(unsigned bits, unsigned i) { return (unsigned)__builtin_amdgcn_sbfe((int)bits, i, 1); }   // bit i % 32: 0 or ~0

// acc += A (32 rows) * B (32 columns) over the 2 U reduction indices of a plane pair; a, b: this lane's 16-byte units
template <typename T>
__device__ __forceinline__ gf32x16 mma_pair(uint4 a, uint4 b, gf32x16 acc)
{
    if constexpr (sizeof(T) == 4) {
        const gf32x4 fa = __builtin_bit_cast(gf32x4, a), fb = __builtin_bit_cast(gf32x4, b);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], acc, 0, 0, 0);
        return acc;
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(gbf16x8, a), __builtin_bit_cast(gbf16x8, b), acc, 0, 0, 0);
    }
}

__device__ __forceinline__ bool any_nan(const gf32x16 &v)
{
    bool u = false;
#pragma unroll
    for (int i = 0; i < 16; i += 2) u |= __builtin_isunordered(v[i], v[i + 1]);
    return u;
}

// Taps in the padding are no part of the sum; a GEMM multiplies zeros there, which is NaN where the filter is infinite or NaN.
// Sums that came out as NaN are added up again without those taps, if the position has any.  acc[4 g + e]: channel
// cw + 8 g + e of lattice position (n, i, j) of residue class (ca, cb).
template <typename T>
__device__ __forceinline__ void gather_redo(const GatherConvParams &p, int ca, int cb, int n, int i, int j, int cw, gf32x16 &acc)
{
    constexpr unsigned SZ = sizeof(T);
    const __amdgpu_buffer_rsrc_t rs_in = __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)p.in_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_wt = __builtin_amdgcn_make_buffer_rsrc((void *)p.wt, 0, (int)p.wt_bytes, 0x00020000);
    const int nr = p.nr[ca], ns = p.ns[cb];
    const int ih0 = i * p.is_h + p.base_h[ca], iw0 = j * p.is_w + p.base_w[cb];
    const int ih1 = ih0 + (nr - 1) * p.step_h, iw1 = iw0 + (ns - 1) * p.step_w;
    auto in_h = [&](int ih) { return (unsigned)ih < (unsigned)p.Hin; };
    auto in_w = [&](int iw) { return (unsigned)iw < (unsigned)p.Win; };
    if (in_h(ih0) && in_h(ih1) && in_w(iw0) && in_w(iw1)) return;
#pragma unroll
    for (int g = 0; g < 4; ++g) {                            // four channels at a time: sixteen would cost the GEMM waves
        const int co = cw + 8 * g;
        float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int c = 0; c < p.Cin; ++c) {
            const int chan = p.in_blocked ? (c >> 4) * p.in_c + (c & 15) : c * p.in_c;
#pragma unroll 1
            for (int t = 0; t < nr * ns; ++t) {
                const int r = t / ns, s = t - r * ns, ih = ih0 + r * p.step_h, iw = iw0 + s * p.step_w;
                if (!in_h(ih) || !in_w(iw)) continue;
                const float x = load_value<T>(rs_in, (unsigned)(n * p.in_n + chan + (ih * p.Win + iw) * p.in_px) * SZ);
                const int tap = c * p.w_chan + (p.r0[ca] + r * p.rst_h) * p.S + p.s0[cb] + s * p.rst_w;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    sum[e] = fmaf(x, load_value<T>(rs_wt, co + e < p.Cout ? (unsigned)((co + e) * p.w_row + tap) * SZ : GATHER_OOB), sum[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = acc[4 * g + e];
            acc[4 * g + e] = v != v ? sum[e] : v;
        }
    }
}

// bias of the channels cw + 8 j + e: reads past the end (or of no bias at all) give zero
__device__ __forceinline__ void gather_bias(const GatherConvParams &p, int cw, float (&bias)[4][4])
{
    const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc((void *)p.bias, 0, p.bias ? p.Cout * 4 : 0, 0x00020000);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) bias[j][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs_b, (cw + 8 * j + e) * 4, 0, 0));
}

// Epilogue: bias, ReLU, mask, one rounding; a lane holds 4 consecutive output channels of a position per group.  With KS
// slices a slice stores the groups g0 + j that are its own.
template <typename T, int KS>
__device__ __forceinline__ void gather_store(const GatherConvParams &p, int ca, int cb, int n, int i, int jj, int cw, int g0, int slice,
                                             const float (&bias)[4][4], const gf32x16 &acc)
{
    const size_t HW = (size_t)p.Hout * p.Wout;
    const int cend = p.out_blocked ? (p.Cout + 15) & ~15 : p.Cout;
    T *out = static_cast<T *>(p.out);
    const T *mask = static_cast<const T *>(p.mask);
    const size_t step = p.out_blocked ? 1 : HW;
    const size_t opix = (size_t)(i * p.os_h + ca) * p.Wout + jj * p.os_w + cb;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int co = cw + 8 * j;
        if (KS > 1 && (g0 + j) % KS != slice) continue;      // another slice's group
        if (co >= cend) continue;
        const size_t base = p.out_blocked ? (((size_t)n * (cend >> 4) + (co >> 4)) * HW + opix) * 16 + (co & 15)
                                          : ((size_t)n * p.Cout + co) * HW + opix;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = acc[4 * j + e] + bias[j][e];
            v[e] = p.relu ? fmaxf(v[e], 0.f) : v[e];
            if (co + e >= p.Cout) v[e] = 0.f;                // padding lanes of a blocked result (0 * infinity before)
        }
        if (mask) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (co + e < p.Cout && !(GElem<T>::widen(mask[base + e * step]) > 0.f)) v[e] = 0.f;
        }
        if (p.out_blocked) {
            if constexpr (sizeof(T) == 4) *reinterpret_cast<float4 *>(out + base) = make_float4(v[0], v[1], v[2], v[3]);
            else *reinterpret_cast<uint2 *>(out + base) = make_uint2(pack_bf16x2_hw(v[0], v[1]), pack_bf16x2_hw(v[2], v[3]));
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (co + e < p.Cout) {
                    if constexpr (sizeof(T) == 4) out[base + e * step] = v[e];
                    else out[base + e * step] = (uint16_t)(pack_bf16x2_hw(v[e], 0.f) & 0xFFFFu);
                }
        }
    }
}

// 8 bf16 at a 2-byte aligned offset: whole dwords around them, shifted
__device__ __forceinline__ uint4 load_bf16x8(__amdgpu_buffer_rsrc_t rs, unsigned off)
{
    const unsigned a = off & ~3u, sh = (off & 2u) * 8;
    const uint4 v = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)a, 0, 0));
    const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(a + 16), 0, 0);
    return make_uint4(__builtin_amdgcn_alignbit(v.y, v.x, sh), __builtin_amdgcn_alignbit(v.z, v.y, sh), __builtin_amdgcn_alignbit(v.w, v.z, sh),
                      __builtin_amdgcn_alignbit(w, v.w, sh));
}

// element strides of images, channels (blocked: 16-channel blocks) and pixels
inline void gather_strides(int layout, int C, int HW, int32_t *n, int32_t *c, int32_t *px)
{
    const bool b = layout == NGC_NCHW16C;
    *n = (b ? (C + 15) / 16 * 16 : C) * HW;
    *c = b ? 16 * HW : HW;
    *px = b ? 16 : 1;
}

// conv_stream.hip; max_m: positions of the largest class
struct StreamChoice {
    bool take, sliced, wrow;       // the node is its own; slices of the reduction (else positions); filter rows in the order of the indices
    size_t lds;                    // of the index table
};
double gather_f32_bwd_us(const GatherConvParams &p, unsigned max_m);    // conv_gather.hip: what the gather GEMM would take
StreamChoice stream_conv_choice(const GatherConvParams &p, int dtype, unsigned max_m, int classes);
hipError_t launch_stream_conv(const GatherConvParams &p, int dtype, unsigned max_m, int classes, const StreamChoice &c, hipStream_t st);
// wgrad_stream.hip: the same for backprop-filters (false also where the workspace is too small); bytes of partial sums
bool launch_wgrad_stream(const ngc_conv_desc &d, int P, int Q, const void *x, const void *dy, float *dw, void *ws, size_t ws_bytes, hipStream_t st, hipError_t *e);
size_t wgrad_stream_workspace(const ngc_conv_desc &d, int P, int Q, bool *takes);

}  // namespace ngc
