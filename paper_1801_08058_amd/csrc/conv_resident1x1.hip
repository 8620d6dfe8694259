// 1x1 convolution (forward and backprop-data, any stride) whose filters stay in registers while the activations stream past
// them: blocked bf16 tensors, bf16 MFMA (gfx950).
//
//   out[pos][co] = sum_ci in[pos'][ci] * wt[ci/16][co][ci%16]        (one tap)
//
// The GEMM of conv_gemm1x1.hip cuts the output into tiles of 64 to 256 channels; a tile's workgroup starts its ring of loads
// anew, and where several channel tiles share an activation tile their rings hold the same lines, so few of the bytes in flight
// are new ones.  Here a workgroup (8 waves, one a compute unit) holds the filters of all output channels as MFMA operands, at most
// 128 registers a wave, and takes an equal share of the positions: the activations come through LDS once, a ring of 64 KB that
// runs on over the tiles, the results leave straight from the registers.  A wave multiplies 32 FC channels by 32 positions;
// WN waves lie side by side over the channels, 8 / WN over the positions.  Products are added in the order of the GEMM: the
// results are the same bits.
//
// What bounds it: HBM on large nodes (256 -> 512 at 56x56 / 2, 64 images, cold: forward 25.4 us for 103 MB of lines, the GEMM 36.6),
// the start (filters, first tile) on small ones.  Two workgroups a compute unit measured 31 us there.
#include "common.h"

#include <math.h>
#include <stdlib.h>

namespace ngc {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr unsigned R1_OOB = 0x80000000u;

struct Resident1x1Params {
    Gemm1x1Params g;
    uint32_t chunk;                    // positions per workgroup
};

template <int KS, int WN>
struct ResidentTile {
    static constexpr int FC = KS == 32 ? 1 : 2;                          // 32-channel fragments of a wave
    static constexpr int WM = 8 / WN, T = 32 * WM;                       // waves over the positions, positions of a tile
    static constexpr int LPW = (WN == 1 ? 2 : 1) * (KS == 32 && WN <= 2 ? 2 : 1);                          // loads per wave and slice
    static constexpr int KSL = LPW * 8 / WM, NSL = KS / KSL;             // 16-channel steps of a slice, slices of a tile
    static constexpr int SLICE = LPW * 8192, NS = 65536 / SLICE + 1;     // ring buffers
    static constexpr size_t LDS = (size_t)NS * SLICE + 32 * FC * WN * 4, LDS_SIB = LDS + 8 * 1024;      // ring, bias; a block of results per wave
    static_assert(KS % KSL == 0, "slices of a tile");
};

template <int KS, int WN, bool SIB>
__global__ __launch_bounds__(512) void conv1x1_resident(const Resident1x1Params rp)
{
    preload_kernargs(rp);
    typedef ResidentTile<KS, WN> G;
    constexpr int FC = G::FC, WM = G::WM, T = G::T, LPW = G::LPW, KSL = G::KSL, NSL = G::NSL, SLICE = G::SLICE, NS = G::NS;
    const Gemm1x1Params &p = rp.g;
    extern __shared__ __align__(16) unsigned char smem[];
    float *bias_lds = reinterpret_cast<float *>(smem + NS * SLICE);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lg = lane >> 5;
    const int wm = wave % WM, wn = wave / WM;
    const int co0 = wn * 32 * FC;
    const int CBin = p.Cin >> 4, HWin = p.Hin * p.Win, CBout = p.Cout >> 4, HWout = p.Hout * p.Wout;

    const uint32_t first = blockIdx.x * rp.chunk;
    const uint32_t end = p.M - first < rp.chunk ? p.M : first + rp.chunk;     // first < M (host)
    const int ntiles = (int)((end - first + T - 1) / T);
    const int nsl = (CBin + KSL - 1) / KSL, total = ntiles * nsl;            // live slices of a tile, of all

    const ngc_u32x4 rw_in = make_rsrc_words(p.in, p.in_bytes);
    const __amdgpu_buffer_rsrc_t rs_wt = __builtin_amdgcn_make_buffer_rsrc((void *)p.wt, 0, (int)p.wt_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc((void *)p.out, 0, (int)p.out_bytes, 0x00020000);

    // ---- loads: piece q = wave + 8 i of a slice is position group q % WM, 16-channel step q / WM of it; lanes 0 .. 31 bring
    // the first 8 channels of the 32 positions, lanes 32 .. 63 the others, so the wave that multiplies reads them in lane order
    int itile = 0, islice = 0, ibuf = 0;
    unsigned voff = R1_OOB;
    auto issue = [&]() {
        if (islice == 0) {
            const uint32_t m = first + (uint32_t)(itile * T + wm * 32 + l32);
            const uint32_t mm = m < end ? m : first;
            const uint32_t n = fd_div(mm, p.div_pq);
            const uint32_t rem = mm - n * p.div_pq.d;
            const uint32_t i = fd_div(rem, p.div_q);
            const uint32_t j = rem - i * p.div_q.d;
            const int ih = (int)i * p.is_h + p.dh, iw = (int)j * p.is_w + p.dw;
            const bool ok = m < end && (unsigned)ih < (unsigned)p.Hin && (unsigned)iw < (unsigned)p.Win;
            voff = ok ? (unsigned)(((int)n * CBin * HWin + ih * p.Win + iw) * 32 + lg * 16) : R1_OOB;
        }
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const int q = wave + 8 * i;
            const int cb = islice * KSL + q / WM;
            const bool live = cb < CBin;                                 // wave-uniform
            dma_load_lds16(rw_in, smem + ibuf * SLICE + q * 1024, live ? voff : R1_OOB, live ? (unsigned)(cb * HWin * 32) : 0u);
        }
        ibuf = ibuf + 1 == NS ? 0 : ibuf + 1;
        if (++islice == nsl) {
            islice = 0;
            ++itile;
        }
    };
#pragma unroll 1
    for (int s = 0; s < NS - 1 && s < total; ++s) issue();

    // ---- filters: rows = output channels; channels and steps past the end are zero
    bf16x8 wa[FC][KS];
#pragma unroll
    for (int f = 0; f < FC; ++f)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int co = co0 + 32 * f + l32;
            const unsigned off = ks < CBin && co < p.Cout ? (unsigned)(((ks * p.Cout + co) * 16 + lg * 8) * 2) : R1_OOB;
            wa[f][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_wt, (int)off, 0, 0));
        }
    if (tid < 32 * FC * WN) bias_lds[tid] = p.bias && tid < p.Cout ? p.bias[tid] : 0.f;      // seen behind the first barrier
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");

    const bool relu_b = p.relu != 0;
    // Stores per wave and tile, for the waits below.  A store out of range counts: its offset is out of range, there is no branch around
    // it, and as the size of the result is not known at compile time no path can do without the instruction.
    constexpr int ST = 2 * FC * (SIB ? 4 : 1);
    unsigned char *const mine = smem + NS * SLICE + 32 * FC * WN * 4 + wave * 1024;

    int g = 0, buf = 0;
    int since = 0, osl = 0;            // tiles stored since the loads of slice g were issued; slice of the iteration that issued them
    for (int t = 0; t < ntiles; ++t) {
        f32x16 acc[FC];
#pragma unroll
        for (int f = 0; f < FC; ++f)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // bias_lds is written before the first barrier: the first tile takes it behind that one
                if (t == 0 && f == 0 && j == 0) wg_barrier_nofence();
                const float4 b4 = *reinterpret_cast<const float4 *>(bias_lds + co0 + 32 * f + 8 * j + 4 * lg);
                acc[f][4 * j] = b4.x; acc[f][4 * j + 1] = b4.y; acc[f][4 * j + 2] = b4.z; acc[f][4 * j + 3] = b4.w;
            }
#pragma unroll
        for (int sl = 0; sl < NSL; ++sl) {
            if (sl >= nsl) break;                                        // uniform
            // Vector-memory operations of a wave complete in the order they were issued, loads and stores alike: behind the
            // loads of slice g there are those of the slices up to g + NS - 2 and the stores of `since` tiles.
            const int later = total - 1 - g < NS - 2 ? total - 1 - g : NS - 2;
            wait_vmcnt63(later * LPW + since * ST);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wg_barrier_nofence();                                        // slice g complete; the buffer of slice g - 1 is free
            if (g + NS - 1 < total) issue();
            const unsigned char *xs = smem + buf * SLICE + wm * 1024 + lane * 16;
            buf = buf + 1 == NS ? 0 : buf + 1;
#pragma unroll
            for (int kk = 0; kk < KSL; ++kk) {
                const bf16x8 xb = *reinterpret_cast<const bf16x8 *>(xs + kk * WM * 1024);
#pragma unroll
                for (int f = 0; f < FC; ++f) acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wa[f][sl * KSL + kk], xb, acc[f], 0, 0, 0);
            }
            // the next slice's loads were issued in iteration g + 2 - NS (or before the first)
            if (sl == nsl - 1) ++since;
            ++g;
            if (g >= NS - 1) {
                // iteration g - (NS - 1) issued slice g's loads ahead of its own stores; the one before it no longer counts
                if (g > NS - 1) {
                    if (++osl == nsl) {
                        osl = 0;
                        --since;
                    }
                }
            }
        }
        // ---- ReLU (bias is in the accumulators), one RNE rounding, lane-pair exchange, 16-byte stores
        const uint32_t m0 = first + (uint32_t)(t * T + wm * 32);
        // byte offset of the 16-channel block 0 of a position's output pixel
        auto pixel = [&](uint32_t m) {
            const uint32_t mm = m < end ? m : first;
            const uint32_t n = fd_div(mm, p.div_pq);
            const uint32_t rem = mm - n * p.div_pq.d;
            const uint32_t i = fd_div(rem, p.div_q);
            const uint32_t j = rem - i * p.div_q.d;
            const int oh = (int)i * p.os_h + p.oa_h, ow = (int)j * p.os_w + p.oa_w;
            struct { unsigned off; int oh, ow; } r = {(unsigned)((int)n * CBout * HWout + oh * p.Wout + ow) * 32u, oh, ow};
            return r;
        };
        unsigned off0 = R1_OOB;
        SibLanes sib;
        if constexpr (!SIB) {
            if (m0 + l32 < end) off0 = pixel(m0 + l32).off + lg * 16;
        } else {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t m = m0 + 16 * u + (lane >> 2);
                const auto px = pixel(m);
                sib.place(u, lane, m < end, px.off, px.oh, px.ow, p.Hout, p.Wout);
            }
        }
#pragma unroll
        for (int f = 0; f < FC; ++f)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x16 &v = acc[f];
                const uint32_t q0 = relu_bf16x2(pack_bf16x2_hw(v[8 * h], v[8 * h + 1]), relu_b);
                const uint32_t q1 = relu_bf16x2(pack_bf16x2_hw(v[8 * h + 2], v[8 * h + 3]), relu_b);
                const uint32_t q2 = relu_bf16x2(pack_bf16x2_hw(v[8 * h + 4], v[8 * h + 5]), relu_b);
                const uint32_t q3 = relu_bf16x2(pack_bf16x2_hw(v[8 * h + 6], v[8 * h + 7]), relu_b);
                const uint4 o = lane_pair_exchange(q0, q1, q2, q3);
                const int cb = (co0 >> 4) + 2 * f + h;
                const unsigned block = (unsigned)(cb * HWout) * 32u;
                const bool live = cb < CBout;                            // wave-uniform
                if constexpr (SIB) {
                    sib.store(mine, lane, o, rs_out, live, block, false);      // small results (resident1x1_takes)
                } else {
                    const ngc_u32x4 ov = {o.x, o.y, o.z, o.w};
                    __builtin_amdgcn_raw_buffer_store_b128(ov, rs_out, (int)(live && off0 != R1_OOB ? off0 + block : R1_OOB), 0, NGC_ST_AUX);
                }
            }
    }
}

// ---------------------------------------------------------------------------------------------- host side

template <int KS, int WN, bool SIB>
static hipError_t launch_resident(const Gemm1x1Params &p, hipStream_t st)
{
    typedef ResidentTile<KS, WN> G;
    static LdsLimitOnce lds_limit;
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&conv1x1_resident<KS, WN, SIB>));
    if (e != hipSuccess) return e;
    Resident1x1Params rp;
    rp.g = p;
    rp.chunk = ((p.M + 255) / 256 + 7) / 8 * 8;                          // whole lines of a 16-channel block
    NGC_LAUNCH((conv1x1_resident<KS, WN, SIB>), dim3((p.M + rp.chunk - 1) / rp.chunk), dim3(512), (SIB ? G::LDS_SIB : G::LDS), st, rp);
    return launch_result();
}

// Forward with strided columns (rows alone, 496 -> 144 channels, 18496 positions, GEMM / here 11.2 / 13.8: the GEMM reads whole lines there),
// expected times of both, us: here a start, tiles of a workgroup, slices of a tile, bytes, the filters that every workgroup fetches; the GEMM
// rounds of tiles, 32-channel steps, bytes, the activations once per channel tile.  Fitted to the mean of operands from memory and from the
// caches over 26499 drawn nodes, strides up to 3, nine tenths within 8 % and 13 %.  2057 nodes are taken, where 5 % less is
// expected: 30398 -> 24863 us, 28 above 1.05 of the GEMM's time; of 10697 others 823, 12642 -> 10338, 17 above, 1.22 at worst.
static bool resident1x1_faster(const Gemm1x1Params &p)
{
    const bool deep = p.Cin > 256, wide = gemm1x1_wide_tiles(p);
    const int wn = deep ? (p.Cout <= 32 ? 1 : p.Cout <= 64 ? 2 : 8) : p.Cout <= 64 ? 1 : p.Cout <= 256 ? 4 : 8;       // as launch_resident1x1
    const int loads = (wn == 1 ? 2 : 1) * (deep && wn <= 2 ? 2 : 1), slices = (p.Cin / 16 + loads * wn - 1) / (loads * wn);
    const double chunk = ceil(ceil(p.M / 256.0) / 8) * 8, tiles = ceil(chunk / (256 / wn)), wgs = ceil(p.M / chunk);
    const double in_mb = 2e-6 * p.Cin * (p.M / p.div_q.d) * p.Win, out_mb = 2e-6 * p.Cout * p.M, filters_mb = 2e-6 * p.Cin * p.Cout;
    const double here = 4.76 + tiles * (0.462 + 0.329 * slices) + 0.0983 * in_mb + 0.095 * out_mb + filters_mb * (2.92 + 0.0067 * wgs);
    const double across = ceil(p.Cout / (wide ? 128.0 : 64.0)), gt = ceil(p.M / (wide ? 128.0 : 256.0)) * across, steps = (p.Cin + 31) / 32;
    const double rounds = ceil(gt / 256), share = gt > 256 ? gt / 256 : 1.0;
    const double gemm = wide ? 3.54 + rounds * (0.845 + 0.02 * steps) + share * steps * 0.22 + in_mb * (0.0831 + 0.0294 * across)
                             : 3.75 + rounds * (0.428 + 0.1013 * steps) + share * steps * 0.271 + in_mb * (0.0954 + 0.0288 * across) + 0.038 * out_mb;
    return here < 0.95 * gemm;
}

// Nodes it is expected to run faster than the GEMM.  GEMM / here, us, operands from memory; m: positions.  Backprop-data (stride 2 x 2): up to
// 2 million results of lattice positions (256 <- 512, m 3136 13.3 / 7.6; 80 <- 400, m 12240 14.0 / 9.0; above, the GEMM's tiles fill the chip:
// 128 <- 112, m 32129 11.2 / 12.2), of channels whose filters pay for being fetched by every workgroup: more than 64 from more than 64 (48 <- 112,
// m 32490 7.5 / 8.3; 32 <- 208, m 45849 9.6 / 15.1), up to 256 (352 <- 48, m 5236 5.4 / 6.3; 368 <- 176, m 4805 7.1 / 8.0), 512 only from 65 to
// 128.  Of 11893 drawn nodes with an instance 10083 are taken, the mean of operands from memory and from the caches 66148 -> 56358 us, 48 above
// 1.05 of the GEMM's time, 1.16 at worst.
bool resident1x1_takes(const Gemm1x1Params &p)
{
    const char *force = env_switch(SW_RESIDENT);                         // tests only: 0 = never, 1 = all it can
    if (force && atoi(force) == 0) return false;
    if (env_switch(SW_G1_VARIANT)) return false;                         // a switch that shapes the GEMM asks for it
    if (p.in_nchw || p.out_nchw || p.dbp || p.mask || !p.out_bytes) return false;
    const bool sib = gemm1x1_siblings(p);
    if (p.os_h * p.os_w > 1 && !sib) return false;
    if (!(p.Cin <= 256 ? p.Cout <= 512 : p.Cin <= 512 && p.Cout <= 256)) return false;
    if (sib && (p.Cin <= 64 ? p.Cout > 256 : p.Cout <= 64 || (p.Cin > 128 && p.Cout > 256))) return false;
    if (force) return true;
    if (sib) return (uint64_t)p.M * p.Cout < 2000000;
    return p.is_w > 1 && resident1x1_faster(p);
}

// The smallest instance that holds the filters; forward has those its rule reaches, the others run the next larger one
hipError_t launch_resident1x1(const Gemm1x1Params &p, hipStream_t st)
{
    if (p.zero_sib) {
        if (p.Cin <= 64) {
            if (p.Cout <= 64) return launch_resident<4, 1, true>(p, st);
            if (p.Cout <= 128) return launch_resident<4, 2, true>(p, st);
            return launch_resident<4, 4, true>(p, st);
        }
        if (p.Cin <= 128) {
            if (p.Cout <= 128) return launch_resident<8, 2, true>(p, st);
            return p.Cout <= 256 ? launch_resident<8, 4, true>(p, st) : launch_resident<8, 8, true>(p, st);
        }
        if (p.Cin <= 256) return p.Cout <= 128 ? launch_resident<16, 2, true>(p, st) : launch_resident<16, 4, true>(p, st);
        return p.Cout <= 128 ? launch_resident<32, 4, true>(p, st) : launch_resident<32, 8, true>(p, st);
    }
    if (p.Cin <= 256) {
        if (p.Cout <= 64) return launch_resident<16, 1, false>(p, st);
        return p.Cout <= 256 ? launch_resident<16, 4, false>(p, st) : launch_resident<16, 8, false>(p, st);
    }
    if (p.Cout <= 32) return launch_resident<32, 1, false>(p, st);
    return p.Cout <= 64 ? launch_resident<32, 2, false>(p, st) : launch_resident<32, 8, false>(p, st);
}

}  // namespace ngc
