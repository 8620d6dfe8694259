// Softmax over the last axis of a [rows, cols] tensor and its backprop (gfx950).  The paper names
// softmax next to convolution as a kernel a backend supplies (Sec. 4); backward graphs come from
// autodiff of the forward ops (Sec. 3).
//
//   y[i][j]  = exp(x[i][j] - m_i) / sum_k exp(x[i][k] - m_i),  m_i = max_k x[i][k]
//   dx[i][j] = y[i][j] * (dy[i][j] - sum_k dy[i][k] y[i][k])
//
// Bound: HBM (each tensor once).  A row lives in registers as vectors of 16 bytes, all of its loads in flight at once.  It
// belongs to a group of GL lanes: 8, 16, 32 or 64 lanes of a wave (butterfly reductions) or a workgroup of 256 or 1024
// (through LDS); a group of the row's own size keeps the lanes busy (rows of 100 elements with a wave each ran at 0.43 TB/s).
// Results leave as 16-byte stores - one read and one write of the row, fp32 arithmetic, one rounding.
//
// Row lengths that are no multiple of 16 bytes use the same kernel: the rows then start anywhere and the vectors are read
// and written unaligned; the last one is the last 16 bytes of the row, and its elements that the vector before it also holds
// are left out of the sums (both lanes store the same values).  Rows beyond the registers are walked twice: the maximum and
// the sum of a thread's part in one pass (rescaled when the maximum grows), the results in the second.  Rows below 16 bytes
// take one thread each.
#include "common.h"

#include <math.h>

namespace ngc {

template <typename T> struct SmElem;
template <> struct SmElem<uint16_t> {                  // bf16 bit patterns, 8 per 16 bytes
    static constexpr int E = 8;
    __device__ static void unpack(const uint4 &v, float (&f)[8])
    {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            f[2 * j] = __uint_as_float(w[j] << 16);
            f[2 * j + 1] = __uint_as_float(w[j] & 0xFFFF0000u);
        }
    }
    __device__ static uint4 pack(const float (&f)[8])
    {
        return make_uint4(pack_bf16x2_hw(f[0], f[1]), pack_bf16x2_hw(f[2], f[3]), pack_bf16x2_hw(f[4], f[5]),
                          pack_bf16x2_hw(f[6], f[7]));
    }
    __device__ static float load(const uint16_t *p) { return bf16_bits_to_float(*p); }
    __device__ static void store(uint16_t *p, float v) { *p = (uint16_t)(pack_bf16x2_hw(v, 0.f) & 0xFFFFu); }
    // bf16 results carry 8 bits: the hardware exp2 (1 ulp of fp32) is far inside the rounding
    __device__ static float exp_of(float d) { return __builtin_amdgcn_exp2f(d * 1.44269504088896341f); }
};
template <> struct SmElem<float> {
    static constexpr int E = 4;
    __device__ static void unpack(const uint4 &v, float (&f)[4])
    {
        f[0] = __uint_as_float(v.x); f[1] = __uint_as_float(v.y); f[2] = __uint_as_float(v.z); f[3] = __uint_as_float(v.w);
    }
    __device__ static uint4 pack(const float (&f)[4])
    {
        return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    }
    __device__ static float load(const float *p) { return *p; }
    __device__ static void store(float *p, float v) { *p = v; }
    __device__ static float exp_of(float d) { return expf(d); }
};

template <int GL>
__device__ __forceinline__ float group_max(float v)
{
#pragma unroll
    for (int o = GL / 2; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
template <int GL>
__device__ __forceinline__ float group_sum(float v)
{
#pragma unroll
    for (int o = GL / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);   // butterfly: every lane ends with the same sum
    return v;
}

// reduction over the NW waves of a workgroup (fixed order); sm holds NW floats
template <int NW>
__device__ __forceinline__ float block_reduce(float v, bool is_max, float *sm)
{
    v = is_max ? group_max<64>(v) : group_sum<64>(v);
    const int wave = threadIdx.x >> 6;
    __syncthreads();                                                     // sm may still be read from the last call
    if ((threadIdx.x & 63) == 0) sm[wave] = v;
    __syncthreads();
    float r = sm[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) r = is_max ? fmaxf(r, sm[w]) : r + sm[w];
    return r;
}

// 16 bytes at any element address
template <typename T>
__device__ __forceinline__ uint4 load16_any(const T *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}
template <typename T>
__device__ __forceinline__ void store16_any(T *p, uint4 v)
{
    typedef unsigned u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
    const u32x4_any w = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4_any *>(p));
}

// A long bf16 row stays packed between the passes over it: unpacked (and its exponentials taken) again instead of kept as
// floats, so that twice as many rows are in flight on a compute unit (1047 x 32029: 36.2 -> 30.3 us).  fp32 exponentials
// replace the elements; of a short bf16 row they are kept (32768 x 1000: 20.1 us against 21.6 us).
template <int N> __device__ __forceinline__ void keep_packed(uint4 (&v)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) asm volatile("" : "+v"(v[j].x), "+v"(v[j].y), "+v"(v[j].z), "+v"(v[j].w));
}

// The row in registers: V vectors per lane of a group of GL lanes: E <= cols <= GL * E * V.  TAIL: cols is no multiple of E
// or the tensors are off the 16-byte grid.  BWD: a = y, b = dy, out = dx; else a = x, out = y (b unused).
template <typename T, int V, bool BWD, int GL, bool TAIL>
__global__ __launch_bounds__(GL <= 64 ? 256 : GL) void softmax_rows_reg(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ out,
                                                        uint32_t rows, int cols)
{
    constexpr int E = SmElem<T>::E;
    constexpr int NW = GL <= 64 ? 1 : GL / 64;
    __shared__ float sm[NW];
    const int lane = threadIdx.x & (GL - 1);
    const uint32_t row = GL <= 64 ? blockIdx.x * (256 / GL) + threadIdx.x / GL : blockIdx.x;
    const bool live = row < rows;                                        // groups past the end stay for the lane exchanges
    const size_t base = (size_t)(live ? row : 0) * cols;
    const int nvec = TAIL ? (cols + E - 1) / E : cols / E;
    auto first = [&](int vi) { return TAIL && vi * E + E > cols ? cols - E : vi * E; };     // first element of a vector
    uint4 va[V], vb[BWD ? V : 1];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int vi = j * GL + lane;
        va[j] = make_uint4(0, 0, 0, 0);
        if (BWD) vb[BWD ? j : 0] = va[j];
        if (vi < nvec) {
            va[j] = load16_any(a + base + first(vi));
            if (BWD) vb[BWD ? j : 0] = load16_any(b + base + first(vi));
        }
    }
    auto counts = [&](int vi, int e) { return vi < nvec && (!TAIL || e >= vi * E + E - cols); };   // not held by the vector before
    auto group = [&](float v, bool is_max) {
        if constexpr (GL <= 64) return is_max ? group_max<GL>(v) : group_sum<GL>(v);
        else return block_reduce<NW>(v, is_max, sm);
    };
    constexpr bool PACKED = sizeof(T) == 2 && V > 2, KEEP = !BWD && !PACKED;
    float m = -INFINITY, s = 0.f, ex[KEEP ? V : 1][E];
    if (BWD) {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float fa[E], fb[E];
            SmElem<T>::unpack(va[j], fa);
            SmElem<T>::unpack(vb[BWD ? j : 0], fb);
#pragma unroll
            for (int e = 0; e < E; ++e) s += !TAIL || counts(j * GL + lane, e) ? fa[e] * fb[e] : 0.f;   // zeros past the end
        }
        if (PACKED) {
            keep_packed(va);
            keep_packed(vb);
        }
        s = group(s, false);
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float f[E];
            SmElem<T>::unpack(va[j], f);
#pragma unroll
            for (int e = 0; e < E; ++e) m = fmaxf(m, j * GL + lane < nvec ? f[e] : -INFINITY);
        }
        if (PACKED) keep_packed(va);
        m = group(m, true);
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float f[E];
            SmElem<T>::unpack(va[j], f);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float v = SmElem<T>::exp_of(f[e] - m);
                if (KEEP) ex[KEEP ? j : 0][e] = v;
                s += counts(j * GL + lane, e) ? v : 0.f;
            }
        }
        if (PACKED) keep_packed(va);
        s = group(s, false);
    }
    if (!live) return;
    const float inv = 1.0f / s;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int vi = j * GL + lane;
        if (vi >= nvec) continue;
        float f[E], fb[E];
        SmElem<T>::unpack(va[j], f);
        if (BWD) SmElem<T>::unpack(vb[BWD ? j : 0], fb);
#pragma unroll
        for (int e = 0; e < E; ++e) f[e] = BWD ? f[e] * (fb[e] - s) : (KEEP ? ex[KEEP ? j : 0][e] : SmElem<T>::exp_of(f[e] - m)) * inv;
        if (TAIL) store16_any(out + base + first(vi), SmElem<T>::pack(f));
        else store16_result(out + base + (size_t)vi * E, SmElem<T>::pack(f), true);
    }
}

// Rows of any length >= E: one workgroup of 1024 threads per row, two passes over it.
template <typename T, bool BWD>
__global__ __launch_bounds__(1024) void softmax_rows_long(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ out,
                                                          uint32_t rows, int cols)
{
    constexpr int E = SmElem<T>::E;
    __shared__ float sm[16];
    const size_t base = (size_t)blockIdx.x * cols;
    const int nvec = (cols + E - 1) / E;
    auto first = [&](int vi) { return vi * E + E > cols ? cols - E : vi * E; };
    float m = -INFINITY, s = 0.f;
#pragma unroll 4
    for (int vi = threadIdx.x; vi < nvec; vi += 1024) {
        float f[E], fb[E];
        SmElem<T>::unpack(load16_any(a + base + first(vi)), f);
        if (BWD) {
            SmElem<T>::unpack(load16_any(b + base + first(vi)), fb);
#pragma unroll
            for (int e = 0; e < E; ++e) s += e >= vi * E + E - cols ? f[e] * fb[e] : 0.f;
        } else {
            float top = f[0];
#pragma unroll
            for (int e = 1; e < E; ++e) top = fmaxf(top, f[e]);
            if (top > m) {
                s *= SmElem<T>::exp_of(m - top);                         // exp(-inf) = 0 the first time
                m = top;
            }
#pragma unroll
            for (int e = 0; e < E; ++e)                                  // a masked element counts nothing, also while all so far were
                s += e >= vi * E + E - cols && f[e] != -INFINITY ? SmElem<T>::exp_of(f[e] - m) : 0.f;
        }
    }
    if (!BWD) {
        const float mine = m;
        m = block_reduce<16>(m, true, sm);
        s *= mine > -INFINITY ? SmElem<T>::exp_of(mine - m) : 0.f;
    }
    s = block_reduce<16>(s, false, sm);
    const float inv = 1.0f / s;
    // The last vector may overlap the one before it, which another thread writes: where out is one of the inputs
    // (in place), its elements are stored one by one, only those that are its own.
#pragma unroll 4
    for (int vi = threadIdx.x; vi < nvec; vi += 1024) {
        const int own = vi * E;
        float f[E], fb[E];
        if (own + E <= cols) {
            SmElem<T>::unpack(load16_any(a + base + own), f);
            if (BWD) SmElem<T>::unpack(load16_any(b + base + own), fb);
#pragma unroll
            for (int e = 0; e < E; ++e) f[e] = BWD ? f[e] * (fb[e] - s) : SmElem<T>::exp_of(f[e] - m) * inv;
            store16_any(out + base + own, SmElem<T>::pack(f));
        } else {
            for (int j = own; j < cols; ++j) {
                const float v = SmElem<T>::load(a + base + j);
                SmElem<T>::store(out + base + j, BWD ? v * (SmElem<T>::load(b + base + j) - s) : SmElem<T>::exp_of(v - m) * inv);
            }
        }
    }
}

// Rows below one vector: a thread per row.
template <typename T, bool BWD>
__global__ __launch_bounds__(256) void softmax_rows_tiny(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ out,
                                                         uint32_t rows, int cols)
{
    constexpr int E = SmElem<T>::E;
    const uint32_t row = blockIdx.x * 256 + threadIdx.x;
    if (row >= rows) return;
    const size_t base = (size_t)row * cols;
    float f[E], fb[E], m = -INFINITY, s = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        f[e] = e < cols ? SmElem<T>::load(a + base + e) : BWD ? 0.f : -INFINITY;
        fb[e] = BWD && e < cols ? SmElem<T>::load(b + base + e) : 0.f;
        m = fmaxf(m, f[e]);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        if (!BWD) f[e] = SmElem<T>::exp_of(f[e] - m);
        s += BWD ? f[e] * fb[e] : f[e];
    }
    const float inv = 1.0f / s;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e < cols) SmElem<T>::store(out + base + e, BWD ? f[e] * (fb[e] - s) : f[e] * inv);
}

// Kernel of a row length: below one vector a thread per row; else the smallest group of lanes and the fewest vectors per lane
// that hold the row; else two passes.
SoftmaxPlan softmax_plan(int dtype, int cols, bool bwd)
{
    const int E = dtype == NGC_BF16 ? 8 : 4, nvec = (cols + E - 1) / E;
    if (cols < E) return {SM_TINY, 1, 1};
    static const SoftmaxPlan groups[] = {{SM_WAVE, 1, 8}, {SM_WAVE, 1, 16}, {SM_WAVE, 1, 32}, {SM_WAVE, 1, 64}, {SM_WAVE, 2, 64}, {SM_WAVE, 4, 64},
                                         {SM_WG, 2, 256}, {SM_WG, 4, 256}, {SM_WG, 2, 1024}, {SM_WG, 4, 1024}, {SM_WG, 8, 1024}};
    for (const SoftmaxPlan &g : groups)
        if (nvec <= g.V * g.GL && !(g.V == 8 && bwd && dtype == NGC_BF16)) return g;     // bf16 backprop: two tensors unpacked do not fit
    return {SM_LONG, 1, 1024};
}

template <typename T, bool BWD, bool TAIL>
static hipError_t launch_softmax_t(const T *a, const T *b, T *out, uint32_t rows, int cols, hipStream_t st)
{
    const SoftmaxPlan pl = softmax_plan(sizeof(T) == 2 ? NGC_BF16 : NGC_F32, cols, BWD);
#define NGC_SM_WAVE(V, GL) NGC_LAUNCH((softmax_rows_reg<T, V, BWD, GL, TAIL>), dim3((rows + 256 / (GL) - 1) / (256 / (GL))), dim3(256), 0, st, a, b, out, rows, cols)
#define NGC_SM_WG(V, GL) NGC_LAUNCH((softmax_rows_reg<T, V, BWD, GL, TAIL>), dim3(rows), dim3(GL), 0, st, a, b, out, rows, cols)
    switch (pl.kernel == SM_TINY ? 0 : pl.kernel == SM_LONG ? 1 : pl.GL * 16 + pl.V) {
    case 0: NGC_LAUNCH((softmax_rows_tiny<T, BWD>), dim3((rows + 255) / 256), dim3(256), 0, st, a, b, out, rows, cols); break;
    case 1: NGC_LAUNCH((softmax_rows_long<T, BWD>), dim3(rows), dim3(1024), 0, st, a, b, out, rows, cols); break;
    case 8 * 16 + 1: NGC_SM_WAVE(1, 8); break;
    case 16 * 16 + 1: NGC_SM_WAVE(1, 16); break;
    case 32 * 16 + 1: NGC_SM_WAVE(1, 32); break;
    case 64 * 16 + 1: NGC_SM_WAVE(1, 64); break;
    case 64 * 16 + 2: NGC_SM_WAVE(2, 64); break;
    case 64 * 16 + 4: NGC_SM_WAVE(4, 64); break;
    case 256 * 16 + 2: NGC_SM_WG(2, 256); break;
    case 256 * 16 + 4: NGC_SM_WG(4, 256); break;
    case 1024 * 16 + 2: NGC_SM_WG(2, 1024); break;
    case 1024 * 16 + 4: NGC_SM_WG(4, 1024); break;
    case 1024 * 16 + 8:
        if constexpr (!(BWD && sizeof(T) == 2)) NGC_SM_WG(8, 1024);
        break;
    default: return hipErrorInvalidValue;
    }
#undef NGC_SM_WAVE
#undef NGC_SM_WG
    return ngc::launch_result();
}

template <typename T>
static hipError_t launch_softmax_e(bool bwd, const void *a, const void *b, void *out, uint32_t rows, int cols, bool grid16, hipStream_t st)
{
    const T *pa = static_cast<const T *>(a), *pb = static_cast<const T *>(b);
    T *po = static_cast<T *>(out);
    if (bwd) return grid16 ? launch_softmax_t<T, true, false>(pa, pb, po, rows, cols, st) : launch_softmax_t<T, true, true>(pa, pb, po, rows, cols, st);
    return grid16 ? launch_softmax_t<T, false, false>(pa, pb, po, rows, cols, st) : launch_softmax_t<T, false, true>(pa, pb, po, rows, cols, st);
}

hipError_t launch_softmax(int dtype, bool bwd, const void *a, const void *b, void *out, uint32_t rows, int cols, bool aligned, hipStream_t st)
{
    const bool grid16 = aligned && cols % (dtype == NGC_BF16 ? 8 : 4) == 0;
    // a grid holds fewer than 2^32 threads: more rows than that take several launches
    const uint32_t most = 0xFFFFFFFFu / (uint32_t)softmax_plan(dtype, cols, bwd).GL / 256 * 256;
    for (uint32_t r0 = 0; r0 < rows;) {
        const uint32_t n = rows - r0 < most ? rows - r0 : most;
        const size_t at = (size_t)r0 * cols * (dtype == NGC_BF16 ? 2 : 4);
        const char *pa = static_cast<const char *>(a) + at, *pb = b ? static_cast<const char *>(b) + at : nullptr;
        char *po = static_cast<char *>(out) + at;
        const hipError_t e = dtype == NGC_BF16 ? launch_softmax_e<uint16_t>(bwd, pa, pb, po, n, cols, grid16, st)
                                               : launch_softmax_e<float>(bwd, pa, pb, po, n, cols, grid16, st);
        if (e != hipSuccess) return e;
        r0 += n;
    }
    return hipSuccess;
}

}  // namespace ngc
