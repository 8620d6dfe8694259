// ConvolutionBackpropFilters on bf16 MFMA (gfx950) for windows of several taps: any strides, dilations, padding and
// window size, any multiple of 16 channels, rank 2 and rank 3.
//
//   dw[k,c,tap] = sum_{m=(n,o,p,q)} dy[m][k] * X[m @ tap][c]
//
// A per-tap GEMM reads both tensors once per tap and pays a load latency per 64 positions; here a workgroup holds a
// block of NKB x 16 k, ncq x 16 c and NT taps of dw in registers and takes its positions through LDS once for all of
// these taps: a stage is SR rows of dy (or G whole small images) plus the patch of x their taps touch, both in their
// natural channel-contiguous form (32-byte pixels, global->LDS loads, out-of-range lanes deliver the zeros of the
// padding).  The transposing LDS read gives a lane 8 positions of one channel, every group of 4 lanes at an address of
// its own, so a tap is an offset and a stride is a pitch: x offsets of the positions of a stage are tabled in LDS once.
//
// Workgroup = 8 waves = ncq channel groups x 8 / ncq interleaved streams of 32-position steps, two waves per SIMD so
// that one's LDS latency hides behind the other's MFMAs; x operands run one step ahead of the MFMAs, stages run
// nring - 1 ahead of both.  NT and NKB are template parameters (accumulators, operands and the step are straight-line
// code): a window splits into groups of at most 9 taps, as equal as the instantiated counts allow, and narrow k
// (NKB < 4) does not multiply padding.
//
// A step costs NKB * NT MFMAs of 16 cycles and 2 (NKB + NT) transposing reads of 512 bytes: the matrix cores bound it
// from NKB = 3, NT = 5 on, the LDS below; small layers are bound by set-up, the latency of a stage and the sum of the
// streams.  Against the per-tap GEMM (us): 51 x 272 x 44 x 87 -> 16, 1x7 287 -> 41; 29 x 352 x 104 x 31 -> 64, 3x3 stride 2
// 63 -> 39; 3 x 304 x 82 x 47 -> 480, 3x3 83 -> 56; 56 x 16 x 71 x 48 -> 80, 5x5 stride 2 68 -> 21; 3x3x3, 3 x 144 x 7 x 24 x
// 29 -> 64 49 -> 26; the geometric mean of 30 layers over the range of window and video layers 21.2 -> 15.0.
#include "common.h"

#include <stdlib.h>
#include <type_traits>

namespace ngc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr unsigned WT_OOB = 0x80000000u;
constexpr int WT_POS = 256;                        // positions per stage, at most: 8 blocks of 32, one per wave
constexpr int WT_RED_KB = 152;                     // stream copies of the tile in LDS, KB
constexpr int WT_XB = 5;                           // 32-pixel blocks of a patch plane per wave, at most

__device__ __forceinline__ bf16x8 wt_frag(const unsigned char *lo, const unsigned char *hi)
{
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)lo);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)hi);
    const s16x8 r = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// Zeros the elements of the operands whose positions are not below `rem`: a lane holds positions 0 .. 3 and 16 .. 19
template <int N> __device__ __forceinline__ void keep_first(bf16x8 (&b)[N], int rem)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    u32x4 keep;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = rem - (i >> 1) * 16 - (i & 1) * 2;
        keep[i] = n >= 2 ? 0xFFFFFFFFu : n == 1 ? 0xFFFFu : 0u;
    }
#pragma unroll
    for (int t = 0; t < N; ++t) b[t] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, b[t]) & keep);
}

// Quotients of the set-up, in a handful of vector operations each (the compiler's 32-bit division is a chain of some
// thirty scalar ones; two dozen of those cost a small launch half its time).
// n / d for n < 65536, inv = 1 / d to one unit in the last place: n + 0.5 is at least 0.5 / d away from a multiple, the
// error of the product below n / d * 2^-22
__device__ __forceinline__ int small_div(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }
// wave-uniform n / d for 0 <= n < 2^24, 0 < d: one correction step makes the rounded quotient exact
__device__ __forceinline__ int uniform_div(int n, int d)
{
    int q = (int)((float)n * __builtin_amdgcn_rcpf((float)d));
    const int r = n - q * d;
    q += (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
    return __builtin_amdgcn_readfirstlane(q);
}

// Largest of 0 .. 12 outstanding loads not above n: a short tree of compares
__device__ __forceinline__ void wait_loads(int n)
{
#define NGC_WT_CASE(N) case N: __builtin_amdgcn_s_waitcnt(0x0F70 | (N)); break;
    switch (n < 12 ? n : 12) {
        NGC_WT_CASE(1) NGC_WT_CASE(2) NGC_WT_CASE(3) NGC_WT_CASE(4) NGC_WT_CASE(5) NGC_WT_CASE(6)
        NGC_WT_CASE(7) NGC_WT_CASE(8) NGC_WT_CASE(9) NGC_WT_CASE(10) NGC_WT_CASE(11) NGC_WT_CASE(12)
    default: __builtin_amdgcn_s_waitcnt(0x0F70); break;
    }
#undef NGC_WT_CASE
}

// The end of a workgroup: the accumulators of its NH = 8 / ncq step streams become its partial, or with one part dw.  LDS is free.
template <int NT, int NKB>
__device__ __forceinline__ void wgrad_taps_finish(const WgradTapsParams &p, f32x4 (&acc)[NKB][NT], unsigned char *smem, const int part,
                                                  const int tile, const int tiles, const int kb0, const int cb0, const int nk, const int nc,
                                                  const int td, const int tap0, const int ntap)
{
    constexpr int NW = 8;
    const int lane = threadIdx.x & 63, L = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncq = p.ncq, lcq = ncq >> 1, NH = NW >> lcq, cq = wave & (ncq - 1), wh = wave >> lcq;
    // ---- the sum of the NH step streams.  While all copies (and, with one part, dw on its way out) do not fit the LDS
    // together, the upper half of the streams publishes and the lower half adds.
    constexpr int UNITS = NKB * NT;                        // 1 KB pieces (16 k x 16 c of a tap) of a wave
    f32x4 *red = reinterpret_cast<f32x4 *>(smem) + lane;
    int nh = NH;
    while (nh > 1 && (nh + 1) * ncq * UNITS > WT_RED_KB) {
        nh >>= 1;
        if (wh >= nh && wh < 2 * nh) {
            f32x4 *d = red + ((wh - nh) * ncq + cq) * (UNITS * 64);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int t = 0; t < NT; ++t) d[(kb * NT + t) * 64] = acc[kb][t];
        }
        __syncthreads();
        if (wh < nh) {
            const f32x4 *src = red + (wh * ncq + cq) * (UNITS * 64);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[kb][t] += src[(kb * NT + t) * 64];
        }
        __syncthreads();
    }
    // dw of one part leaves through LDS so that the stores are contiguous ([k][c][tap] as in memory): accumulator element
    // v of unit (kb, t) is k = 16 kb + 4 grp + v, c = 16 cq + L; the row pitch spreads the four groups over the banks
    const int pitch = 16 * ncq * NT + 4;
    float *tl = reinterpret_cast<float *>(smem) + (nh > 1 ? nh * ncq * UNITS * 256 : 0);
    f32x4 *out = reinterpret_cast<f32x4 *>(p.partial) + ((size_t)part * tiles + tile) * ncq * (UNITS * 64) + lane;
    if (nh == 1) {
        if (wh == 0) {
            if (p.nparts > 1) {
                out += cq * (UNITS * 64);
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int t = 0; t < NT; ++t) out[(kb * NT + t) * 64] = acc[kb][t];
            } else {
                float *d = tl + (4 * grp) * pitch + (16 * cq + L) * NT;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int t = 0; t < NT; ++t) d[(kb * 16 + v) * pitch + t] = acc[kb][t][v];
            }
        }
    } else {
        // the remaining copies fit: every wave adds a share of the units over all of them, in stream order
        if (wh < nh) {
            f32x4 *d = red + (wh * ncq + cq) * (UNITS * 64);
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int t = 0; t < NT; ++t) d[(kb * NT + t) * 64] = acc[kb][t];
        }
        __syncthreads();
        for (int u = wave; u < ncq * UNITS; u += NW) {
            f32x4 r = red[u * 64];
            for (int h = 1; h < nh; ++h) r += red[(h * ncq * UNITS + u) * 64];
            if (p.nparts > 1) {
                out[u * 64] = r;
            } else {
                const int q = (int)(((float)u + 0.5f) * (1.0f / UNITS)), w = u - q * UNITS, kb = w / NT, t = w - kb * NT;
                float *d = tl + (kb * 16 + 4 * grp) * pitch + (16 * q + L) * NT + t;
#pragma unroll
                for (int v = 0; v < 4; ++v) d[v * pitch] = r[v];
            }
        }
    }
    if (p.nparts > 1) return;
    __syncthreads();
    const int taps = p.T * p.RS, C = p.CB * 16, rowlen = 16 * nc * NT;
    float *dst = p.dw + ((size_t)kb0 * 16 * C + cb0 * 16) * taps + td * p.RS + tap0;
    for (int k = wave; k < 16 * nk; k += NW)
        for (int j = lane; j < rowlen; j += 64) {
            const int c = j / NT, t = j - c * NT;
            if (t < ntap) dst[((size_t)k * C + c) * taps + t] = tl[k * pitch + j];
        }
}

// A launch starts with a cold instruction cache (every 64-byte line of code a round trip to the L2 or beyond), so code
// that runs once is kept short: one copy of the stage loads and of the MFMA steps, geometry that does not depend on the
// workgroup in the arguments.  The first version, 1600 instructions before its first load, took 9.9 us for a layer of
// 5 MFLOP that takes 6.5 now.
template <int NT, int NKB>
__global__ __launch_bounds__(512) void wgrad_taps_bf16(const WgradTapsParams p)
{
    constexpr int NW = 8;
    extern __shared__ __align__(16) unsigned char smem[];
    preload_kernargs(p);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ncq = p.ncq, lcq = ncq >> 1;                  // ncq is 1, 2 or 4; lcq its logarithm
    const int NH = NW >> lcq;
    const int cq = wave & (ncq - 1);
    const int wh = wave >> lcq;
    const int L = lane & 15, grp = lane >> 4;

    // ---- part, tile, tap group.  Where the parts deal evenly to the 8 XCDs (blockIdx % 8), the tiles and tap groups of a
    // part run one after the other on one of them and share its rows through its L2.
    const int ngroups = p.T * p.gpt, tiles = p.ktiles * p.ctiles * ngroups;
    int part = 0, tile = blockIdx.x;
    if (p.xcd) {
        const int j = blockIdx.x >> 3, pl = uniform_div(j, tiles);
        tile = j - pl * tiles;
        part = pl * 8 + (blockIdx.x & 7);
        if (part >= p.nparts) return;                      // uniform per workgroup
    } else if (p.nparts > 1) {
        tile = uniform_div(blockIdx.x, p.nparts);
        part = blockIdx.x - tile * p.nparts;
    }
    int kt = tile, ct = 0, td = 0, tap0 = 0, r0 = 0;
    if (ngroups > 1) {
        kt = uniform_div(tile, ngroups);
        td = tile - kt * ngroups;
        if (p.gpt > 1) {
            const int group = td;
            td = uniform_div(group, p.gpt);
            tap0 = (group - td * p.gpt) * NT;
            r0 = uniform_div(tap0, p.S);
        }
    }
    if (p.ctiles > 1) {
        const int kc = kt;
        kt = uniform_div(kc, p.ctiles);
        ct = kc - kt * p.ctiles;
    }
    const int s0 = tap0 - r0 * p.S;
    const int ntap = p.RS - tap0 < NT ? p.RS - tap0 : NT;

    const int PQ = p.P * p.Q, HW = p.H * p.W;
    const int kb0 = kt * NKB, cb0 = ct * ncq;
    // planes of the tile that exist: the others are not loaded, what the LDS holds there only reaches rows and columns
    // of dw that are not stored
    const int nk = p.KB - kb0 < NKB ? p.KB - kb0 : NKB, nc = p.CB - cb0 < ncq ? p.CB - cb0 : ncq;
    const int G = p.G;
    const bool multi = G > 1;

    // ---- slices: rank 2 = the images of the batch; rank 3 = the depth slices of an image whose tap is inside x
    const unsigned dy_pl = (unsigned)(p.O * PQ * 32), x_pl = (unsigned)(p.D * HW * 32);          // 16-channel planes
    const unsigned dy_out = (unsigned)p.KB * dy_pl, x_out = (unsigned)p.CB * x_pl;   // images
    unsigned dy_in = dy_out, x_in = x_out;                                                       // slices
    unsigned is_dy = (unsigned)kb0 * dy_pl, is_x = (unsigned)cb0 * x_pl;                         // first slice
    int ninner = p.N, nib = p.nib, per = 0x3fffffff;
    int tq = p.tq, trem = p.trem;                          // stages per part, parts with one more
    const int nrb = p.nrb;
    if (p.r3) {
        const int dd = td * p.dil_d - p.pbd;
        int olo = dd < 0 ? uniform_div(-dd + p.sd - 1, p.sd) : 0;
        int ohi = p.D - 1 - dd < 0 ? 0 : uniform_div(p.D - 1 - dd, p.sd) + 1;
        if (ohi > p.O) ohi = p.O;
        if (olo > ohi) olo = ohi;
        ninner = ohi - olo;
        nib = uniform_div(ninner + G - 1, G);              // blocks of slices
        dy_in = (unsigned)(PQ * 32);
        x_in = (unsigned)(p.sd * HW * 32);
        is_dy += (unsigned)(olo * PQ * 32);
        is_x += (unsigned)((olo * p.sd + dd) * HW * 32);
        per = nib * nrb;
        tq = uniform_div(p.N * per, p.nparts);
        trem = p.N * per - tq * p.nparts;
    }
    const int st_begin = part * tq + (part < trem ? part : trem);
    const int st_count = tq + (part < trem ? 1 : 0);

    const int stage_pos = multi ? G * PQ : p.SR * p.Q;
    const int nblk_dy = (stage_pos + 31) >> 5;             // 32-position steps of a full stage, at most 8
    const int npatch1 = p.PRS * p.PC, npatch = G * npatch1;
    const int nblk_x = (npatch + 31) >> 5;
    const int dyplane = nblk_dy * 1024 + 128, xplane = nblk_x * 1024 + 128;
    const int stage_bytes = NKB * dyplane + ncq * xplane;
    int *xtab = reinterpret_cast<int *>(smem + p.nring * stage_bytes);                            // [WT_POS]

    const int min_dh = r0 * p.dil_h - p.pbh, min_dw = -p.pbw;
    const float inv_pc = __builtin_amdgcn_rcpf((float)p.PC);
    const float inv_pq = __builtin_amdgcn_rcpf((float)PQ), inv_patch = __builtin_amdgcn_rcpf((float)npatch1);

    const ngc_u32x4 rs_dy = make_rsrc_words(p.dy, (unsigned)p.N * dy_out);
    const ngc_u32x4 rs_x = make_rsrc_words(p.x, (unsigned)p.N * x_out);

    // ---- stages are issued in order; the (outer, slice block, row block) of the next one is carried along
    int is_rb = 0, is_ib = st_begin;
    if (p.r3) {
        const int a = per ? uniform_div(st_begin, per) : 0;
        is_ib -= a * per;
        is_dy += (unsigned)a * dy_out;
        is_x += (unsigned)a * x_out;
    }
    if (nrb > 1) {
        const int b = is_ib;
        is_ib = uniform_div(b, nrb);
        is_rb = b - is_ib * nrb;
    }
    int ms_rb = is_rb, ms_ib = is_ib;                      // the stage being multiplied

    // ---- loads of a stage: wave w brings 32-position block w of every dy plane and the 32-pixel blocks w, w + 8, ..
    // of every x plane.  What does not change from stage to stage is computed here, once for all planes.
    const int half = (lane & 1) * 16, lane2 = lane >> 1;
    const int ndy = wave < nblk_dy ? nk : 0, nxb = (nblk_x - wave + NW - 1) >> 3;                // nxb <= 0: none
    const int dy_pos = wave * 32 + lane2;
    unsigned dy_voff = (unsigned)(dy_pos * 32 + half);
    if (multi) dy_voff += (unsigned)small_div(dy_pos, inv_pq) * (dy_in - (unsigned)(PQ * 32));
    int x_row[WT_XB];
    unsigned x_voff[WT_XB];
#pragma unroll
    for (int j = 0; j < WT_XB; ++j) {
        x_row[j] = 0;
        x_voff[j] = 0;
        if (j < nxb) {
            const int px = (wave + NW * j) * 32 + lane2;
            const int g = multi ? small_div(px, inv_patch) : 0;
            const int px1 = px - (int)__umul24(g, npatch1);
            const int pr = small_div(px1, inv_pc), pc = px1 - (int)__umul24(pr, p.PC);
            bool ok = px < npatch && (unsigned)(min_dw + pc) < (unsigned)p.W;
            if (multi) ok = ok && (unsigned)(min_dh + pr) < (unsigned)p.H;
            x_voff[j] = (unsigned)(((int)__umul24(pr, p.W) + pc) * 32 + half);
            if (multi) x_voff[j] += (unsigned)g * x_in;
            x_row[j] = ok ? (multi ? g : pr) : 0x40000000;
        }
    }
    auto issue_loads = [&](int buf) {
        unsigned char *base = smem + buf * stage_bytes + wave * 1024;
        const int row0 = is_rb * p.SR;
        int rows = p.P - row0, gv = ninner - is_ib * G;
        if (rows > p.SR) rows = p.SR;
        if (gv > G) gv = G;
        const int nvalid = multi ? gv * PQ : rows * p.Q;
        const int h0 = row0 * p.sh + min_dh;
        const unsigned dy_org = is_dy + (unsigned)(is_ib * G) * dy_in + (unsigned)(row0 * p.Q * 32);
        const unsigned x_org = is_x + (unsigned)(is_ib * G) * x_in + (unsigned)((h0 * p.W + min_dw) * 32);
        const int radd = multi ? 0 : h0;
        const unsigned rlim = multi ? (unsigned)gv : (unsigned)p.H;
        {
            const unsigned off = dy_pos < nvalid ? dy_org + dy_voff : WT_OOB;
            unsigned soff = 0;
            unsigned char *dst = base;
            for (int i = 0; i < ndy; ++i, soff += dy_pl, dst += dyplane) dma_load_lds16(rs_dy, dst, off, soff);
        }
        base += NKB * dyplane;
#pragma unroll
        for (int j = 0; j < WT_XB; ++j)
            if (j < nxb) {
                const unsigned off = (unsigned)(x_row[j] + radd) < rlim ? x_org + x_voff[j] : WT_OOB;
                unsigned soff = 0;
                unsigned char *dst = base + j * (NW * 1024);
#pragma unroll 1
                for (int i = 0; i < nc; ++i, soff += x_pl, dst += xplane) dma_load_lds16(rs_x, dst, off, soff);
            }
        if (++is_rb == nrb) {
            is_rb = 0;
            if (++is_ib == nib) {
                is_ib = 0;
                is_dy += dy_out;
                is_x += x_out;
            }
        }
    };

    f32x4 acc[NKB][NT];
#pragma unroll
    for (int a = 0; a < NKB; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][t][v] = 0.f;

    const int lane_pos = grp * 4 + (L >> 2), lane_col = (L & 3) * 8;
    const int lpw = ndy + (nxb > 0 ? nxb * nc : 0), ahead = p.nring - 1;
    int tap_off[NT];
    {
        int r = 0, c = s0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            tap_off[t] = t < ntap ? (r * p.dil_h * p.PC + c * p.dil_w) * 32 : 0;
            const bool wrap = ++c == p.S;
            c = wrap ? 0 : c;
            r += wrap ? 1 : 0;
        }
    }
    const bool early = wave >= 4 || p.nring < 3;
    int buf = 0, nbuf = 0, j0 = wh;                        // j0: this stream's first step of the stage
    auto offsets = [&](int step, int (&xo)[2]) {
#pragma unroll
        for (int e = 0; e < 2; ++e) xo[e] = xtab[(step * 32 + e * 16 + lane_pos) & (WT_POS - 1)];
    };
    // Iterations s < 0 fill the ring.  With three buffers waves 0-3, one of each SIMD, issue the loads of a later
    // stage behind their MFMAs, the others before: a wave is held at issue while the memory system takes its loads.
    for (int s = -ahead; s < st_count; ++s) {
        int xo[2] = {0, 0}, xn[2] = {0, 0};                    // x offsets of this stream's first two steps of the stage
        if (s > 0) {                                       // under the wait below; the table is complete from s = 0 on
            offsets(j0, xo);
            offsets(j0 + NH, xn);
        }
        if (s >= 0) {
            const int later = (st_count - 1 - s < ahead - 1) ? st_count - 1 - s : ahead - 1;
            wait_loads(later * lpw);
            wg_barrier_nofence();                          // stage s is complete, buffer of stage s - 1 is free
        }
#pragma unroll 1
        for (int turn = 0; turn < 2; ++turn) {
            if ((turn == 0) == early) {
                if (s + ahead < st_count) issue_loads(nbuf);
                if (++nbuf == p.nring) nbuf = 0;
                if (s == -ahead) {
                    // under the first loads: x offsets of the positions of a stage (dy is zero beyond the last one; keep
                    // x inside the patch) and of the taps
                    if (tid < WT_POS) {
                        const int pos = tid < stage_pos ? tid : stage_pos - 1;
                        const int g = multi ? small_div(pos, inv_pq) : 0;
                        const int pos1 = pos - (int)__umul24(g, PQ);
                        const int row = small_div(pos1, __builtin_amdgcn_rcpf((float)p.Q)), col = pos1 - (int)__umul24(row, p.Q);
                        xtab[tid] = (int)(__umul24(g, npatch1) + __umul24(row, p.sh * p.PC) + __umul24(col, p.sw)) * 32;
                    }
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                }
                continue;
            }
            if (s < 0) continue;
            int rows = p.P - ms_rb * p.SR, gv = ninner - ms_ib * G;
            if (rows > p.SR) rows = p.SR;
            if (gv > G) gv = G;
            const int nvalid = multi ? gv * PQ : rows * p.Q, nsteps = (nvalid + 31) >> 5;
            if (++ms_rb == nrb) {
                ms_rb = 0;
                if (++ms_ib == nib) ms_ib = 0;
            }
            const unsigned char *dys = smem + buf * stage_bytes + lane_col;
            const unsigned char *xs = smem + buf * stage_bytes + NKB * dyplane + cq * xplane + lane_col;
            if (++buf == p.nring) buf = 0;
            auto load_a = [&](int step, bf16x8 (&a)[NKB]) {
                const unsigned char *q = dys + (step * 32 + lane_pos) * 32;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) a[kb] = wt_frag(q + kb * dyplane, q + kb * dyplane + 512);
            };
            auto load_b = [&](const int (&xo)[2], int t) { return wt_frag(xs + xo[0] + tap_off[t], xs + xo[1] + tap_off[t]); };
            int j = j0;
            if (j < nsteps) {
                bf16x8 acur[NKB], b[NT];
                if (s == 0) {
                    offsets(j, xo);
                    offsets(j + NH, xn);
                }
                // the offsets are waited for here and, below, at the end of the step before: at the head of the loop the wait
                // would be for every operand under way
                asm volatile("" : "+v"(xo[0]), "+v"(xo[1]), "+v"(xn[0]), "+v"(xn[1]));
                load_a(j, acur);
#pragma unroll
                for (int t = 0; t < NT; ++t) b[t] = load_b(xo, t);
                auto step_body = [&](auto has_next_tag) {
                    constexpr bool HAS_NEXT = decltype(has_next_tag)::value;
                    bf16x8 anext[NKB];
                    int xnn[2];
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
#pragma unroll
                        for (int kb = 0; kb < NKB; ++kb)
                            acc[kb][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(acur[kb], b[t], acc[kb][t], 0, 0, 0);
                        if (HAS_NEXT && t == 0) offsets(j + 2 * NH, xnn);
                        if (HAS_NEXT) b[t] = load_b(xn, t);
                        if (HAS_NEXT && t == (NT > 2 ? 2 : 0)) load_a(j + NH, anext);
                        // keeps the refills among the MFMAs: collected behind them they are waited for in one piece
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (HAS_NEXT) {
#pragma unroll
                        for (int kb = 0; kb < NKB; ++kb) acur[kb] = anext[kb];
                        asm volatile("" : "+v"(xnn[0]), "+v"(xnn[1]));
                        xn[0] = xnn[0];
                        xn[1] = xnn[1];
                    }
                };
                while (j + NH < nsteps) {
                    step_body(std::true_type{});
                    j += NH;
                }
                // positions past the last one: dy is zero there, x is not and has to be where it is infinite or NaN
                if (j * 32 + 32 > nvalid) keep_first(b, nvalid - j * 32 - grp * 4);
                step_body(std::false_type{});
            }
            // streams continue across stages, so that the remainders even out
            j0 = (j0 - nsteps) & (NH - 1);
        }
    }
    __syncthreads();                                       // all stage buffers are free

    wgrad_taps_finish<NT, NKB>(p, acc, smem, part, tile, tiles, kb0, cb0, nk, nc, td, tap0, ntap);
}

// Bytes from a pixel to the end of what its taps reach (9 taps, one of the rows of a tap group)
__host__ __device__ inline int wgrad_own_zeros(const WgradTapsParams &p)
{
    return (((p.RS / p.S - 1) * p.dil_h * p.PC + (p.S - 1) * p.dil_w) * 32 + 32 + 15) & ~15;
}

// The same for 3x3-class windows (9 taps, any stride and dilation) with one 16-channel group of c per workgroup, rank 2: every wave
// takes stages of its own, SR rows of at most 32 positions - one step - and their patch, through a ring of buffers of its own.  With
// ncq = 1 no wave ever reads what another loaded, so the common stages of the kernel above only make the waves wait for each other,
// 8 steps and a barrier at a time.  Here there is none: while the operands of a stage, already in registers, are multiplied, those of
// the next one are read from LDS and two (NXB = 2) or one more are under way.  Loads past the last stage deliver zeros to buffers that
// nobody reads, so that the wait is always for the same number of loads.
// 512 -> 512 at 7x7, 128 images: 54.6 us with common stages, 41.7 here (42.8 with
// masks on the operands in place of zeros to read and an address addition per tap).  Bound by the LDS, 26 transposing reads of 512 bytes and 6 KB
// of loads for 36 MFMAs: it works 0.69 of the cycles that the compute units are busy, the matrix pipes 0.46.
// U3: three rows of three taps a pixel apart - the taps of a row are constants in the LDS reads.
template <int NXB, bool U3>
__global__ __launch_bounds__(512) void wgrad_taps_own_bf16(const WgradTapsParams p)
{
    constexpr int NT = 9, NKB = 4, NW = 8, RING = NXB == 2 ? 3 : 2, STAGE = (NKB + NXB) * 1024;
    extern __shared__ __align__(16) unsigned char smem[];
    preload_kernargs(p);
    const int lane = threadIdx.x & 63, L = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    const int tiles = p.ktiles * p.ctiles;
    int part = 0, tile = blockIdx.x;
    if (p.xcd) {
        const int j = blockIdx.x >> 3, pl = uniform_div(j, tiles);
        tile = j - pl * tiles;
        part = pl * 8 + (blockIdx.x & 7);
        if (part >= p.nparts) return;                      // uniform per workgroup
    } else if (p.nparts > 1) {
        tile = uniform_div(blockIdx.x, p.nparts);
        part = blockIdx.x - tile * p.nparts;
    }
    const int kt = uniform_div(tile, p.ctiles), cb0 = tile - kt * p.ctiles, kb0 = kt * NKB;
    const int nk = p.KB - kb0 < NKB ? p.KB - kb0 : NKB;    // planes of the tile that exist; zeros for the others

    const int PQ = p.P * p.Q, HW = p.H * p.W, nrb = p.nrb;
    const unsigned dy_pl = (unsigned)(PQ * 32), x_pl = (unsigned)(HW * 32);              // 16-channel planes
    const unsigned dy_img = (unsigned)p.KB * dy_pl, x_img = (unsigned)p.CB * x_pl;
    const int st_begin = part * p.tq + (part < p.trem ? part : p.trem);
    const int st_end = st_begin + p.tq + (part < p.trem ? 1 : 0);
    const ngc_u32x4 rs_dy = make_rsrc_words(p.dy, (unsigned)p.N * dy_img);
    const ngc_u32x4 rs_x = make_rsrc_words(p.x, (unsigned)p.N * x_img);
    unsigned char *const mine = smem + wave * (RING * STAGE);

    // ---- loads: 32 positions of each of the four dy planes, NXB blocks of 32 patch pixels
    const int lane2 = lane >> 1;
    const int min_dh = -p.pbh, min_dw = -p.pbw, npatch = p.PRS * p.PC;
    const float inv_pc = __builtin_amdgcn_rcpf((float)p.PC);
    int x_row[NXB];
    unsigned x_voff[NXB];
#pragma unroll
    for (int j = 0; j < NXB; ++j) {
        const int px = j * 32 + lane2, pr = small_div(px, inv_pc), pc = px - (int)__umul24(pr, p.PC);
        const bool ok = (px < npatch) & ((unsigned)(min_dw + pc) < (unsigned)p.W);
        x_voff[j] = (unsigned)(((int)__umul24(pr, p.W) + pc) * 32 + (lane & 1) * 16);
        x_row[j] = ok ? pr : 0x40000000;
    }
    int st = st_begin + wave, img = uniform_div(st, nrb), rb = st - img * nrb;           // the stage loaded next
    const int img_step = uniform_div(NW, nrb), rb_step = NW - img_step * nrb;
    int ibuf = 0;
    auto issue = [&]() {
        const int row0 = rb * p.SR;
        int nvalid = (p.P - row0 < p.SR ? p.P - row0 : p.SR) * p.Q;
        const bool live = st < st_end;
        nvalid = live ? nvalid : 0;
        const int h0 = row0 * p.sh + min_dh;
        unsigned char *dst = mine + ibuf * STAGE;
        const unsigned dy_org = (unsigned)img * dy_img + (unsigned)kb0 * dy_pl + (unsigned)(row0 * p.Q * 32);
        const unsigned x_org = (unsigned)img * x_img + (unsigned)cb0 * x_pl + (unsigned)((h0 * p.W + min_dw) * 32);
        const unsigned off = lane2 < nvalid ? dy_org + (unsigned)(lane * 16) : WT_OOB;
        unsigned soff = 0;
#pragma unroll
        for (int i = 0; i < NKB; ++i, soff += dy_pl) dma_load_lds16(rs_dy, dst + i * 1024, i < nk ? off : WT_OOB, i < nk ? soff : 0u);
        const unsigned rlim = live ? (unsigned)p.H : 0u;
#pragma unroll
        for (int j = 0; j < NXB; ++j)
            dma_load_lds16(rs_x, dst + (NKB + j) * 1024, (unsigned)(x_row[j] + h0) < rlim ? x_org + x_voff[j] : WT_OOB, 0);
        st += NW;
        img += img_step;
        rb += rb_step;
        if (rb >= nrb) {
            rb -= nrb;
            ++img;
        }
        ibuf = ibuf + 1 == RING ? 0 : ibuf + 1;
    };
#pragma unroll 1
    for (int s = 0; s < RING; ++s) issue();

    // ---- operand addresses: positions 4 grp + L / 4 and 16 further on.  Positions past the last one, where dy is zero but x would be
    // what some pixel holds, infinities and NaN included, read zeros behind the rings, as far as the taps reach.
    const int zeros = NW * RING * STAGE, zero_bytes = wgrad_own_zeros(p);
    for (int i = threadIdx.x * 4; i < zero_bytes; i += 2048) *reinterpret_cast<int *>(smem + zeros + i) = 0;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier_nofence();
    int xo[2], pos_of[2];
    const int lane_pos = grp * 4 + (L >> 2), lane_col = (L & 3) * 8;
    {
        const float inv_q = __builtin_amdgcn_rcpf((float)p.Q);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            pos_of[e] = lane_pos + 16 * e;
            const int row = small_div(pos_of[e], inv_q), col = pos_of[e] - (int)__umul24(row, p.Q);
            xo[e] = (int)(__umul24(row, p.sh * p.PC) + __umul24(col, p.sw)) * 32 + NKB * 1024 + lane_col + wave * (RING * STAGE);
        }
    }
    int tap_off[NT];
    {
        int r = 0, c = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            tap_off[t] = (r * p.dil_h * p.PC + c * p.dil_w) * 32;
            const bool wrap = ++c == p.S;
            c = wrap ? 0 : c;
            r += wrap ? 1 : 0;
        }
    }
    f32x4 acc[NKB][NT];
#pragma unroll
    for (int a = 0; a < NKB; ++a)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][t][v] = 0.f;

    int ms = st_begin + wave, mrb = ms - uniform_div(ms, nrb) * nrb, mbuf = 0;           // the stage whose operands are read next
    auto load_a = [&](const unsigned char *base, bf16x8 (&a)[NKB]) {
        const unsigned char *q = base + lane_pos * 32 + lane_col;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) a[kb] = wt_frag(q + kb * 1024, q + kb * 1024 + 512);
    };
    auto x_at = [&](int (&at)[2]) {
        const int nvalid = (p.P - mrb * p.SR < p.SR ? p.P - mrb * p.SR : p.SR) * p.Q;
#pragma unroll
        for (int e = 0; e < 2; ++e) at[e] = pos_of[e] < nvalid ? xo[e] + mbuf * STAGE : zeros + lane_col;
    };
    auto load_b = [&](const int (&at)[2], int t) {
        const int off = U3 ? (t / 3) * p.dil_h * p.PC * 32 : tap_off[t];
        const unsigned char *q0 = smem + (at[0] + off), *q1 = smem + (at[1] + off);
        return wt_frag(q0 + (U3 ? t % 3 * 32 : 0), q1 + (U3 ? t % 3 * 32 : 0));
    };
    auto next_stage = [&]() {
        ms += NW;
        mrb += rb_step;
        mrb = mrb >= nrb ? mrb - nrb : mrb;
        mbuf = mbuf + 1 == RING ? 0 : mbuf + 1;
    };
    bf16x8 acur[NKB], b[NT];
    __builtin_amdgcn_s_waitcnt(0x0F70 | ((RING - 1) * (NKB + NXB) & 15));                // all but the loads of the other stages
    asm volatile("" ::: "memory");
    if (ms < st_end) {
        int at[2];
        load_a(mine, acur);
        x_at(at);
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = load_b(at, t);
        next_stage();
#pragma unroll 1
        for (;;) {
            const bool more = ms < st_end;
            bf16x8 anext[NKB];
            // the operands in registers were the last reads of their buffer
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue();
            __builtin_amdgcn_s_waitcnt(0x0F70 | ((RING - 1) * (NKB + NXB) & 15));
            asm volatile("" ::: "memory");
            x_at(at);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    acc[kb][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(acur[kb], b[t], acc[kb][t], 0, 0, 0);
                b[t] = load_b(at, t);
                if (t == 2) load_a(mine + mbuf * STAGE, anext);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!more) break;                                            // what was read is a stage of zeros
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) acur[kb] = anext[kb];
            next_stage();
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                     // the loads of zeros are still on their way to the LDS
    __syncthreads();
    wgrad_taps_finish<NT, NKB>(p, acc, smem, part, tile, tiles, kb0, cb0, nk, 1, 0, 0, NT);
}

// dw[k][c][tap] = sum over parts (index order).  256 threads = 256 / SL outputs (float4: four k) x SL interleaved part
// slices, joined in a fixed order.
template <int SL>
__global__ __launch_bounds__(256) void wgrad_taps_reduce(const WgradTapsParams p, int nt, int nkb, unsigned per4)
{
    constexpr int NO = 256 / SL;
    __shared__ f32x4 sm[SL == 1 ? 1 : SL][SL == 1 ? 1 : NO];
    const f32x4 *partial = reinterpret_cast<const f32x4 *>(p.partial);
    const int o = threadIdx.x % NO, sl = threadIdx.x / NO;
    const unsigned i = blockIdx.x * NO + o;                // per4 is a multiple of 64, a block of SL = 1 covers 256
    if (SL == 1 && i >= per4) return;
    f32x4 t0 = {0.f, 0.f, 0.f, 0.f}, t1 = t0;
    int sp = sl;
    for (; sp + SL < p.nparts; sp += 2 * SL) {
        t0 += partial[(size_t)sp * per4 + i];
        t1 += partial[(size_t)(sp + SL) * per4 + i];
    }
    if (sp < p.nparts) t0 += partial[(size_t)sp * per4 + i];
    f32x4 r = t0 + t1;
    if constexpr (SL > 1) {
        sm[sl][o] = r;
        __syncthreads();
        if (sl != 0) return;
        f32x4 q[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            q[a] = sm[a][o];
#pragma unroll
            for (int b = 4; b < SL; b += 4) q[a] += sm[a + b][o];
        }
        r = (q[0] + q[1]) + (q[2] + q[3]);
    }
    const int lane = (int)(i & 63);
    unsigned u = i >> 6;
    const int t = (int)(u % (unsigned)nt); u /= (unsigned)nt;
    const int kb = (int)(u % (unsigned)nkb); u /= (unsigned)nkb;
    const int cq = (int)(u % (unsigned)p.ncq); u /= (unsigned)p.ncq;
    const int ngroups = p.T * p.gpt, group = (int)(u % (unsigned)ngroups), kc = (int)(u / (unsigned)ngroups);
    const int kt = kc / p.ctiles, ct = kc - kt * p.ctiles;
    const int td = group / p.gpt, tap = (group - td * p.gpt) * nt + t;
    const int c = (ct * p.ncq + cq) * 16 + (lane & 15), k = (kt * nkb + kb) * 16 + 4 * (lane >> 4);
    const int C = p.CB * 16, taps = p.T * p.RS;
    if (c >= C || k >= p.KB * 16 || tap >= p.RS) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) p.dw[((size_t)(k + v) * C + c) * taps + td * p.RS + tap] = r[v];
}

// ---- host: shape of the split
//
// Costs in cycles of a compute unit, from the operation counts; only their order matters.  A workgroup has a compute
// unit to itself (registers of two waves per SIMD).
double wgrad_stage_cost(int nkb, int ncq, int nt, int dy_blocks, int x_blocks, int ring, double *fixed)
{
    const double mf = 32.0 * nkb * nt, ld = 70.0 * (nkb + nt);                       // MFMAs, LDS reads of 8 wave steps
    const double loads = (nkb * dy_blocks + ncq * x_blocks) * 1024.0 / 32.0;
    double stage = dy_blocks * ncq / 8.0 * (mf > ld ? mf : ld) + 900.0;              // barrier, first operands
    if (loads > stage) stage = loads;
    if (2400.0 / (ring - 1) > stage) stage = 2400.0 / (ring - 1);                    // a load's latency, over the stages ahead
    // once per workgroup: set-up, first stage, sum of the streams
    const int units = nkb * nt;
    int nh = 8 / ncq;
    *fixed = 4500.0 + loads;
    for (; nh > 1 && (nh + 1) * ncq * units > WT_RED_KB; nh >>= 1) *fixed += 64.0 * units + 400.0;
    *fixed += 16.0 * (nh + 1) * ncq * units;
    return stage;
}

// a second launch; partials out and in
double wgrad_parts_cost(int parts, size_t part_bytes) { return parts > 1 ? 6500.0 + 2.0 * parts * part_bytes / 1600.0 : 0.0; }

// Expected time, to choose between this kernel and the others and between the splits of rank 3: the terms above (2400 cycles a us)
// with the weights that fit 435 measured nodes of the window and video ranges, nine tenths of them within 8 %
static double wgrad_taps_us(long rounds, long per, double stage, double fixed, size_t partial_bytes, size_t dw_elems, long wgs, long blocks)
{
    return 1.2 + (partial_bytes ? 2.8 : 0.0) + rounds * (1.2 + (1.67 * per * stage + 1.63 * fixed) / 2400.0) + 0.29e-6 * partial_bytes +
           0.48e-6 * 4.0 * dw_elems + 1.8e-3 * wgs / 256.0 * per * blocks;
}

// whether the tiles of a part are kept on one XCD
static bool wgrad_taps_xcd(long tiles, long parts) { return tiles > 1 && (parts % 8 == 0 || parts >= 64); }

// Rounds of workgroups, one to a compute unit.  by_xcd (rank 3 and stages of a wave's own): of the fullest XCD where they are ordered by XCD: 84
// parts of 3 tiles are 33 for its 32 compute units (3 x 32 -> 32, 21 x 17 x 43 25.1 us, 42 parts of 6 tiles 19.0; 112 x 48 -> 64 at 105x22, own
// stages, 84 parts 50.7, 78 parts 32.4).
static long wgrad_taps_rounds(long tiles, long parts, bool by_xcd)
{
    return by_xcd && wgrad_taps_xcd(tiles, parts) ? ((parts + 7) / 8 * tiles + 31) / 32 : (tiles * parts + 255) / 256;
}

// Turns a finished plan into one of wgrad_taps_own_bf16 where that is expected to take less time: 64 k, 16 c, 9 taps a workgroup, as
// many parts as one round of workgroups has room for or fewer.  Expected time, us, operands from memory: start and sum of the streams per
// round, the stages of a wave, partials, dw, operands read; fitted to 1206 launches of 350 drawn nodes (0.1 GFLOP and more, images up to 40 x
// 32), nine tenths of them within 6 %, its split 0.4 % above the best of those that were timed.  common_stages: of a part of the plan it is
// compared with, which takes less than its own expectation where there are one or two (0.88 and 0.95 of it at the median of 125 nodes):
// nothing waits for the other waves then (416 -> 528 at 14x4, 3 images, one stage 10.6 / 12.9).  Of 8139 other drawn nodes 2980 are taken, the
// mean of operands from memory and from the caches 105108 -> 88186 us (the best of each 87534), 15 above 1.05 (2 x 16 -> 256 at 45x14 11.3 / 13.1).
static void wgrad_taps_own_plan(WgradTapsPlan *out, int rspan, int pc, long common_stages, int force, bool within)
{
    WgradTapsParams &q = out->p;
    if (q.Q > 32 || env_switch(SW_WGRAD_OWN)) return;         // the switch (any value): common stages, tests / benchmarks only
    int sr = 32 / q.Q < q.P ? 32 / q.Q : q.P;
    const int nb = (q.P + sr - 1) / sr;
    sr = (q.P + nb - 1) / nb;
    const long prs = (long)(sr - 1) * q.sh + rspan + 1, nstages = (long)q.N * nb, tiles = (long)((q.KB + 3) / 4) * q.CB;
    const int nxb = prs * pc <= 64 ? 2 : (int)((prs * pc + 31) / 32);
    if (nxb > 4 || nstages >= (1 << 23) || tiles >= (1 << 20)) return;     // a patch holds what the taps of a position reach: the zeros fit
    const double dw_mb = 36864e-6 * tiles;
    const long most = tiles < 256 ? 256 / tiles : 1;
    double best = 0.0;
    long parts = 0;
    for (long p = 1; p <= most && p <= nstages; ++p) {
        if (force > 0 ? p != force % 1000 && force % 1000 : p > 1 && p * dw_mb * 1e6 > (double)NGC_STATIC_SCRATCH_BYTES) continue;
        if (within && p > 1 && (size_t)p * tiles * 36864 > out->ws) continue;
        const long per = (nstages + p - 1) / p, rounds = wgrad_taps_rounds(tiles, p, true);      // of the fullest XCD
        const double us = 3.76 + rounds * (6.48 + 0.738 * ((per + 7) / 8)) + (p > 1 ? 0.43 + 0.63 * p * dw_mb : 0.0) + 0.32 * dw_mb +
                          0.003 * tiles * p / 256.0 * per * (4 + nxb);
        if (parts == 0 || us < best) {
            best = us;
            parts = p;
        }
    }
    const bool same_tile = q.ncq == 1 && out->nkb == 4;
    if (parts == 0 || (force > 0 ? !same_tile : best >= (common_stages <= 2 ? 0.9 : 1.0) * out->us)) return;
    q.SR = (int16_t)sr;
    q.G = 1;
    q.PRS = (int16_t)prs;
    q.nrb = (int16_t)nb;
    q.nib = q.N;
    q.ncq = 1;
    q.ktiles = (int16_t)((q.KB + 3) / 4);
    q.ctiles = q.CB;
    q.nparts = (int16_t)parts;
    q.xcd = wgrad_taps_xcd(tiles, parts);
    q.tq = (int32_t)(nstages / parts);
    q.trem = (int16_t)(nstages % parts);
    out->own = nxb;
    out->nkb = 4;
    // the rings; the sum: four waves' copies, then two and dw on its way out
    const size_t ring = (size_t)8 * (nxb == 2 ? 3 : 2) * (4 + nxb) * 1024 + wgrad_own_zeros(q), sum = 4 * 36 * 1024;
    out->lds = ring > sum ? ring : sum;
    out->ws = parts > 1 ? (size_t)parts * tiles * 36864 : 0;
    out->us = best;
}

bool wgrad_taps_plan(WgradTapsPlan *out, bool within)
{
    const char *force = env_switch(SW_WGRAD_TAPS);        // tests / benchmarks only: 0 = never, nkb * 10000 + ncq * 1000 + parts
    const int fv = force ? atoi(force) : -1;
    if (fv == 0) return false;
    // a switch that shapes the per-tap GEMM asks for it
    if (env_switch(SW_WGG_SP) || env_switch(SW_WGG_TILE) || env_switch(SW_WGG_SLOTS) || env_switch(SW_WGG_XCD) || env_switch(SW_WGG3_PARTS))
        return false;
    WgradTapsParams q = out->p;
    q.r3 = q.T > 1 || q.D > 1 || q.O > 1 || q.pbd > 0;     // pbd: the one slice of dy may lie in front of x
    const int taps = q.T * q.RS;
    if (taps < 2 || q.Q > 224 || (size_t)q.N * q.CB * q.D * q.H * q.W * 32 >= 0x80000000ull ||
        (size_t)q.N * q.KB * q.O * q.P * q.Q * 32 >= 0x80000000ull) return false;
    // tap groups of a depth slice: as few as 9 taps each allow, then the smallest instantiated count that covers them
    static const int counts[] = {1, 2, 3, 4, 5, 7, 9};
    const int want = (q.RS + (q.RS + 8) / 9 - 1) / ((q.RS + 8) / 9);
    int nt = 9;
    for (int i = 6; i >= 0; --i)
        if (counts[i] >= want)
            nt = counts[i];
    q.gpt = (int8_t)((q.RS + nt - 1) / nt);
    int rspan = 0;                                         // rows a group's taps span, at most
    for (int g = 0; g < q.gpt; ++g) {
        const int a = g * nt, b = (a + nt < q.RS ? a + nt : q.RS) - 1;
        const int span = (b / q.S - a / q.S) * q.dil_h;
        rspan = span > rspan ? span : rspan;
    }
    const long pc = (long)(q.Q - 1) * q.sw + (long)(q.S - 1) * q.dil_w + 1;
    const int KB = q.KB, CB = q.CB, groups = q.T * q.gpt;
    const size_t dw_elems = (size_t)256 * KB * CB * taps;
    double best = 0.0, by_cycles = 0.0, by_cycles_us = 0.0;
    int b_nkb = 0, b_ncq = 0, b_sr = 0, b_g = 0, b_parts = 0, b_ring = 0;
    for (int ncq = 4; ncq >= 1; ncq >>= 1) {
        if (ncq > 1 && ncq / 2 >= CB) continue;
        if (fv > 0 && fv / 1000 % 10 != ncq) continue;
        for (int nkb = 4; nkb >= 1; --nkb) {
            if (nkb > 1 && nkb > KB) continue;
            if (fv > 0 && fv / 10000 % 10 != nkb) continue;
            const int ktiles = (KB + nkb - 1) / nkb, ctiles = (CB + ncq - 1) / ncq;
            const long tiles = (long)ktiles * ctiles * groups;
            int last_sr = 0, last_g = 0;
            for (int target = WT_POS; target >= 32; target >>= 1) {
                // rows (or whole images) of a stage: near `target` positions, evened out, within slots and LDS
                int sr = target / q.Q, g = 1;
                if (sr < 1) sr = 1;
                if (sr > q.P) sr = q.P;
                const bool flat = !q.r3;
                auto fits = [&](int sr_, int g_, int *ring) {
                    const long prs = (long)(sr_ - 1) * q.sh + rspan + 1;
                    const long npos = (long)g_ * sr_ * q.Q, npatch = (long)g_ * prs * pc;
                    const long bx = (npatch + 31) / 32, bd = (npos + 31) / 32;
                    if (npos > WT_POS || bx > 8 * WT_XB || prs > 32767) return false;
                    const long stage = nkb * (bd * 1024 + 128) + ncq * (bx * 1024 + 128);
                    if (3 * stage + WT_POS * 4 <= 160 * 1024) *ring = 3;
                    else if (2 * stage + WT_POS * 4 <= 160 * 1024) *ring = 2;
                    else return false;
                    return true;
                };
                int ring = 0;
                while (sr > 1 && !fits(sr, 1, &ring)) --sr;
                if (!fits(sr, 1, &ring)) continue;
                if (sr == q.P) {
                    const int lim = flat ? q.N : q.O;
                    while (g < lim && (g + 1) * q.P * q.Q <= target && fits(sr, g + 1, &ring)) ++g;
                    g = (lim + (lim + g - 1) / g - 1) / ((lim + g - 1) / g);
                    if (!fits(sr, g, &ring)) continue;
                } else {
                    const int nb = (q.P + sr - 1) / sr;
                    sr = (q.P + nb - 1) / nb;
                    if (!fits(sr, 1, &ring)) continue;
                }
                if (sr == last_sr && g == last_g) continue;
                last_sr = sr;
                last_g = g;
                const long prs = (long)(sr - 1) * q.sh + rspan + 1;
                const long bx = (g * prs * pc + 31) / 32, bd = ((long)g * sr * q.Q + 31) / 32;
                const long total = flat ? (long)((q.N + g - 1) / g) * ((q.P + sr - 1) / sr)
                                        : (long)q.N * ((q.O + g - 1) / g) * ((q.P + sr - 1) / sr);
                if (total >= (1 << 23)) continue;               // uniform_div
                double fixed;
                const double stage = wgrad_stage_cost(nkb, ncq, nt, (int)bd, (int)bx, ring, &fixed);
                const int units = nkb * nt;
                const size_t part_bytes = (size_t)tiles * ncq * units * 1024;
                // Rank 2, large operands, parts whose workgroups lie on several XCDs: each fetches them for itself.
                const double streamed = 0.5 * (bd * nkb + bx * ncq) * 1024.0 * total * tiles > 4e7 ? 1.25 : 1.0;
                auto consider = [&](long parts) {
                    if (parts < 1 || parts > total || parts > 1024) return;
                    if (parts > 1 && parts * part_bytes > ((size_t)NGC_STATIC_SCRATCH_BYTES)) return;
                    const long wgs = tiles * parts, rounds = wgrad_taps_rounds(tiles, parts, q.r3);
                    const long stages = (total + parts - 1) / parts;
                    // Rank 3 by the expected time: the depth taps of a part read the same slices at other times, and parts in multiples
                    // of 8 leave compute units idle.  64 -> 128, 8 x 16 x 56 x 56 206.6 us in cycles as rank 2 (32 parts), 200.8 without the
                    // quarter, 190.2 by time (36); 152 drawn nodes take 0.92 of the time they take in cycles without the quarter up to 8
                    // tiles: 90 are faster by 5 % and more, 7 slower, by 10 % at most.
                    const bool xcd = parts % 8 == 0 || parts >= 64 || tiles == 1;
                    double cost = ((wgs + 255) / 256) * (fixed + stages * stage * (xcd ? 1.0 : streamed)) + wgrad_parts_cost((int)parts, part_bytes) + dw_elems * 4.0 / 1600.0;
                    if (q.r3) {
                        const double us = wgrad_taps_us(rounds, stages, stage, fixed, parts > 1 ? parts * part_bytes : 0, dw_elems, wgs, bx * ncq + bd * nkb);
                        if (by_cycles == 0.0 || cost < by_cycles) {
                            by_cycles = cost;
                            by_cycles_us = us;
                        }
                        cost = us;
                    }
                    if (best == 0.0 || cost < best) {
                        best = cost;
                        b_nkb = nkb; b_ncq = ncq; b_sr = sr; b_g = g; b_parts = (int)parts; b_ring = ring;
                    }
                };
                if (fv > 0 && fv % 1000) {
                    consider(fv % 1000 < total ? fv % 1000 : total);
                } else {
                    consider(1);
                    for (long per = 1; per < total; per = per < 16 ? per + 1 : per + per / 8) consider((total + per - 1) / per);
                    for (long parts = 8; parts <= 256; parts += 8) consider(parts);
                }
            }
        }
    }
    if (best == 0.0) return false;
    q.SR = (int16_t)b_sr;
    q.G = (int16_t)b_g;
    q.PRS = (int16_t)((b_sr - 1) * q.sh + rspan + 1);
    q.PC = (int16_t)pc;
    q.ncq = (int8_t)b_ncq;
    q.nring = (int8_t)b_ring;
    q.ktiles = (int16_t)((KB + b_nkb - 1) / b_nkb);
    q.ctiles = (int16_t)((CB + b_ncq - 1) / b_ncq);
    q.nparts = (int16_t)b_parts;
    const long tiles = (long)q.ktiles * q.ctiles * groups;
    if (tiles * (b_parts + 7) >= (1 << 23)) return false;
    q.xcd = wgrad_taps_xcd(tiles, b_parts);
    q.nrb = (int16_t)((q.P + b_sr - 1) / b_sr);
    q.nib = (q.N + b_g - 1) / b_g;                        // rank 3: these three per depth tap, in the kernel
    q.tq = q.nib * q.nrb / b_parts;
    q.trem = (int16_t)(q.nib * q.nrb % b_parts);
    const long bx = ((long)b_g * q.PRS * pc + 31) / 32, bd = ((long)b_g * b_sr * q.Q + 31) / 32;
    out->p = q;
    out->nt = nt;
    out->nkb = b_nkb;
    const size_t stages = (size_t)b_ring * (b_nkb * (bd * 1024 + 128) + b_ncq * (bx * 1024 + 128)) + WT_POS * 4;
    // the sum of the step streams: either all copies and dw on its way out, or four waves' copies and then dw
    const int units = b_nkb * nt;
    int nh = 8 / b_ncq;
    const bool tree = (nh + 1) * b_ncq * units > WT_RED_KB;
    while (nh > 1 && (nh + 1) * b_ncq * units > WT_RED_KB) nh >>= 1;
    const size_t tile = (size_t)16 * b_nkb * (16 * b_ncq * nt + 4) * sizeof(float);
    size_t red = (size_t)(nh > 1 ? nh : 0) * b_ncq * units * 1024 + tile;
    if (tree && red < (size_t)4 * units * 1024) red = (size_t)4 * units * 1024;
    out->lds = stages > red ? stages : red;
    if (out->lds > 160 * 1024) return false;
    out->ws = b_parts > 1 ? (size_t)b_parts * tiles * b_ncq * b_nkb * nt * 1024 : 0;
    out->own = 0;
    out->cycles = q.r3 ? 0.0 : best;
    double fixed;
    const double stage = wgrad_stage_cost(b_nkb, b_ncq, nt, (int)bd, (int)bx, b_ring, &fixed);
    const long total = (q.r3 ? (long)q.N * ((q.O + b_g - 1) / b_g) : (long)q.nib) * q.nrb, per = (total + b_parts - 1) / b_parts;
    const long wgs = tiles * b_parts, rounds = wgrad_taps_rounds(tiles, b_parts, q.r3);
    out->us = wgrad_taps_us(rounds, per, stage, fixed, out->ws, dw_elems, wgs, bx * b_ncq + bd * b_nkb);
    // Rank 3, against the per-tap GEMM: the smallest of many estimates is a low one, so a node that the split by cycles would leave to
    // the GEMM has to be expected 8 % faster (1 x 80 -> 48, 8 x 22 x 52 /2, expected 12.3 / 13.4, takes 12.3 / 12.5; 40 nodes that change
    // kernels without this margin take 0.76 to 1.07 of the GEMM's time).
    if (q.r3) out->us = by_cycles_us < 1.09 * out->us ? by_cycles_us : 1.09 * out->us;
    else if (nt == 9 && q.RS == 9) wgrad_taps_own_plan(out, rspan, (int)pc, per, fv, within);
    return true;
}

// The same for the per-tap GEMM: rounds of 512 workgroups, its stages of 64 positions by tile width, partials, operands read
// (297 nodes, nine tenths within 14 %)
double wgrad_gemm_us(const WgradGemmParams &q, int taps)
{
    const double wgs = (double)q.ktiles * q.ctiles * taps * q.nparts, stages = (double)q.M / q.nparts / 64.0;
    const double stage = q.wk * q.wc == 1 ? 0.59 : q.wk * q.wc == 2 ? 0.65 : 0.71;
    return 8.0 + (double)(((long)wgs + 511) / 512) * (0.22 + stages * stage) + 0.47e-6 * 16384.0 * wgs * q.wk * q.wc +
           0.054 * wgs / 512.0 * stages * (q.wk + q.wc);
}

template <int NT, int NKB>
static hipError_t launch_wgrad_taps_t(const WgradTapsPlan &pl, hipStream_t st)
{
    static LdsLimitOnce lds_limit;                         // per template instantiation
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&wgrad_taps_bf16<NT, NKB>));
    if (e != hipSuccess) return e;
    const WgradTapsParams &p = pl.p;
    const unsigned tiles = (unsigned)(p.ktiles * p.ctiles * p.T * p.gpt);
    const dim3 grid(p.xcd ? 8u * ((p.nparts + 7) / 8) * tiles : (unsigned)p.nparts * tiles);
    NGC_LAUNCH((wgrad_taps_bf16<NT, NKB>), grid, dim3(512), pl.lds, st, p);
    return launch_result();
}

template <int NXB, bool U3>
static hipError_t launch_wgrad_taps_own(const WgradTapsPlan &pl, hipStream_t st)
{
    static LdsLimitOnce lds_limit;                         // per template instantiation
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&wgrad_taps_own_bf16<NXB, U3>));
    if (e != hipSuccess) return e;
    const WgradTapsParams &p = pl.p;
    const unsigned tiles = (unsigned)(p.ktiles * p.ctiles);
    const dim3 grid(p.xcd ? 8u * ((p.nparts + 7) / 8) * tiles : (unsigned)p.nparts * tiles);
    NGC_LAUNCH((wgrad_taps_own_bf16<NXB, U3>), grid, dim3(512), pl.lds, st, p);
    return launch_result();
}

template <int NT>
static hipError_t launch_wgrad_taps_n(const WgradTapsPlan &pl, hipStream_t st)
{
    switch (pl.nkb) {
    case 1: return launch_wgrad_taps_t<NT, 1>(pl, st);
    case 2: return launch_wgrad_taps_t<NT, 2>(pl, st);
    case 3: return launch_wgrad_taps_t<NT, 3>(pl, st);
    case 4: return launch_wgrad_taps_t<NT, 4>(pl, st);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_wgrad_taps(const WgradTapsPlan &pl, hipStream_t st)
{
    hipError_t e = hipErrorInvalidValue;
    switch (pl.own ? 10 + pl.own : pl.nt) {
    case 12: e = pl.p.S == 3 && pl.p.dil_w == 1 ? launch_wgrad_taps_own<2, true>(pl, st) : launch_wgrad_taps_own<2, false>(pl, st); break;
    case 13: e = pl.p.S == 3 && pl.p.dil_w == 1 ? launch_wgrad_taps_own<3, true>(pl, st) : launch_wgrad_taps_own<3, false>(pl, st); break;
    case 14: e = pl.p.S == 3 && pl.p.dil_w == 1 ? launch_wgrad_taps_own<4, true>(pl, st) : launch_wgrad_taps_own<4, false>(pl, st); break;
    case 1: e = launch_wgrad_taps_n<1>(pl, st); break;     // 3x1x1: three groups of one tap
    case 2: e = launch_wgrad_taps_n<2>(pl, st); break;
    case 3: e = launch_wgrad_taps_n<3>(pl, st); break;
    case 4: e = launch_wgrad_taps_n<4>(pl, st); break;
    case 5: e = launch_wgrad_taps_n<5>(pl, st); break;
    case 7: e = launch_wgrad_taps_n<7>(pl, st); break;
    case 9: e = launch_wgrad_taps_n<9>(pl, st); break;
    }
    const WgradTapsParams &p = pl.p;
    if (e != hipSuccess || p.nparts == 1) return e;
    const unsigned per4 = (unsigned)(p.ktiles * p.ctiles * p.T * p.gpt * p.ncq * pl.nkb * pl.nt) * 64u;
    if (p.nparts >= 16)
        NGC_LAUNCH(wgrad_taps_reduce<16>, dim3(per4 / 16), dim3(256), 0, st, p, pl.nt, pl.nkb, per4);
    else if (p.nparts > 8)
        NGC_LAUNCH(wgrad_taps_reduce<8>, dim3(per4 / 32), dim3(256), 0, st, p, pl.nt, pl.nkb, per4);
    else                                                   // a handful of parts: one thread per output adds them itself
        NGC_LAUNCH(wgrad_taps_reduce<1>, dim3((per4 + 255) / 256), dim3(256), 0, st, p, pl.nt, pl.nkb, per4);
    return launch_result();
}

}  // namespace ngc
