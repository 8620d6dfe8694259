// Forward and backprop-data of the nodes of conv_gather.hip, operands straight from memory to registers (gfx950): fp32
// tensors, channel counts that are no multiple of 16, low-channel first layers, whatever the layout.
//
//   out[co][pos] = sum_kk wt[co][kk] * in[kk][pos],   kk = (reduction channel, tap row, tap column), columns fastest
//
// The gather GEMM stages both operands of a step through LDS; a step is then a chain of load latency, LDS and a barrier,
// 0.45 us however small the tile.  Here a wave takes a tile of 32 output channels x 32 NF positions for its share of the
// reduction: KS slices take turns with groups of B steps of 2 U indices (U = 4 fp32, 8 bf16), a lane loads the U indices of its
// half itself, and the loads of a wave's next group are in flight while it multiplies the one before.  No barrier but the ones
// behind the index table and in front of the sum over the slices.
//
// What bounds it: small nodes launch, table and one or two batches of loads; large ones the L1, which serves a load whose lanes
// lie in different lines (the filter operand: 32 rows) a line at a time: fp32 3x3 64 -> 96, 8 x 45 x 37, 19.7 accesses a load, 0.87 a
// cycle that a compute unit is busy, the matrix pipes busy in half of those cycles (0.4 of the launch).  Two fragments of positions a
// wave (half the filter loads) measured level, eight slices slower.  Gather GEMM / here, forward and backprop-data, us: that layer
// 34.5 / 23.8 and 30.8 / 33.0 (which stays there); fp32 16 -> 32, 2 x 16 x 16 6.8 / 5.2 and 8.9 / 6.4; bf16 40 -> 72, 8 x 28 x 28 9.0 / 8.9 and
// 16.6 / 11.6; bf16 190 -> 12, 4 x 23 x 15 /2 25.3 / 12.9 and 7.3 / 5.0; 1x1 fp32 128 -> 83, 7 x 47 x 53 16.8 / 10.2 and 15.3 / 11.8.
//
// Where the elements of an index lie is worked out once per workgroup into a table in LDS, {input offset, tap} and for
// backprop-data the filter offset; a lane adds its pixel and masks taps in the padding with one bit per tap.
#include "conv_gather.h"

#include <math.h>
#include <stdlib.h>

namespace ngc {

constexpr int STREAM_DEAD = 31;                        // tap bit that is set in every lane: indices past the end

template <typename T> constexpr int STREAM_B = sizeof(T) == 4 ? 2 : 1;      // steps per group

template <typename T, int NF, int KS, int WN, bool WROW>
__global__ __launch_bounds__(64 * KS * WN) void stream_conv(const GatherConvParams p)
{
    preload_kernargs(p);
    constexpr int U = GElem<T>::U, NK = 2 * U, B = STREAM_B<T>, NT = 64 * KS * WN;
    constexpr bool SHORT = sizeof(T) == 4 && KS == 1;
    constexpr unsigned SZ = sizeof(T);
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int slice = wave % KS;

    const int ca = (int)blockIdx.z / p.os_w, cb = (int)blockIdx.z - ca * p.os_w;           // residue class of this grid slice
    const int nr = p.nr[ca], ns = p.ns[cb], OP = p.oph[ca], OQ = p.opw[cb], ntaps = nr * ns;
    const int kred = ntaps * p.Cin;
    const unsigned M = (unsigned)p.N * OP * OQ;
    if (blockIdx.x * (32 * NF * WN) >= M) return;                        // uniform per workgroup
    const unsigned m0 = blockIdx.x * (32 * NF * WN) + wave / KS * (32 * NF);
    const int co0 = blockIdx.y * 32;
    const FastDiv div_pq = p.div_pq[2 * (OP != p.oph[0]) + (OQ != p.opw[0])], div_q = p.div_q[OQ != p.opw[0]];
    auto position = [&](unsigned m, int &n, int &i, int &j) {
        n = (int)fd_div(m, div_pq);
        const unsigned t = m - (unsigned)n * div_pq.d;
        i = (int)fd_div(t, div_q);
        j = (int)(t - (unsigned)i * div_q.d);
    };

    gf32x16 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;

    if (kred > 0) {
        const int ngroups = (kred + NK * B - 1) / (NK * B), kpad = (ngroups + 1) * NK * B;     // the last group is dead
        uint2 *ent = reinterpret_cast<uint2 *>(smem);
        unsigned *wtab = reinterpret_cast<unsigned *>(smem + (size_t)kpad * 8);
        const int row_off = p.step_h * p.Win * p.in_px * (int)SZ, col_off = p.step_w * p.in_px * (int)SZ;
        for (int kk = tid; kk < kpad; kk += NT) {
            const int c = kk / ntaps, t = kk - c * ntaps, r = (int)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)ns)), s = t - r * ns;
            const bool live = kk < kred;
            const unsigned chan = p.in_blocked ? (unsigned)(c >> 4) * p.in_c + (c & 15) : (unsigned)c * p.in_c;
            ent[kk] = make_uint2(live ? (unsigned)(r * row_off + s * col_off) + chan * SZ : 0, live ? t : STREAM_DEAD);
            // past the last index: wt_bytes, out of range on its own and on top of a lane offset that already is
            if (!WROW) wtab[kk] = live ? ((unsigned)c * p.w_chan + r * p.rst_h * p.S + s * p.rst_w) * SZ : p.wt_bytes;
        }
        // this lane's positions: byte offset of tap (0, 0), and one bit per tap that lies outside the image
        unsigned pix[NF], nok[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            pix[f] = 0;
            nok[f] = ~0u;
            if (m0 + 32 * f + l32 < M) {
                int n, i, j;
                position(m0 + 32 * f + l32, n, i, j);
                const int ih = i * p.is_h + p.base_h[ca], iw = j * p.is_w + p.base_w[cb];
                pix[f] = (unsigned)(n * p.in_n + (ih * p.Win + iw) * p.in_px) * SZ;
                unsigned okc = 0, ok = 0;
                for (int s = 0; s < ns; ++s) okc |= (unsigned)((unsigned)(iw + s * p.step_w) < (unsigned)p.Win) << s;
                for (int r = 0; r < nr; ++r) ok |= (unsigned)(ih + r * p.step_h) < (unsigned)p.Hin ? okc << (r * ns) : 0;
                nok[f] = ~ok;
            }
        }
        const bool crow = co0 + l32 < p.Cout;
        const unsigned wrow = crow ? (unsigned)((co0 + l32) * p.w_row + p.r0[ca] * p.S + p.s0[cb] + (WROW ? U * half : 0)) * SZ : GATHER_OOB;
        const __amdgpu_buffer_rsrc_t rs_in = __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)p.in_bytes, 0x00020000);
        // load_bf16x8 reads whole dwords: an odd last element is in range with its dword
        const __amdgpu_buffer_rsrc_t rs_wt = __builtin_amdgcn_make_buffer_rsrc((void *)p.wt, 0, (int)(WROW ? (p.wt_bytes + 3) & ~3u : p.wt_bytes), 0x00020000);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier_nofence();

        uint32_t xr[2][B][NF][U], wr[2][B][WROW ? 1 : U];
        uint4 wv[2][WROW ? B : 1];
        auto request = [&](int set, int grp) {
            const int k0 = (grp < ngroups ? grp : ngroups) * (NK * B);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int kk = k0 + b * NK + half * U;
#pragma unroll
                for (int e = 0; e < U; e += 2) {
                    const uint4 d = *reinterpret_cast<const uint4 *>(ent + kk + e);
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        xr[set][b][f][e] = GElem<T>::load(rs_in, (pix[f] + d.x) | (bit_mask(nok[f], d.y) & GATHER_OOB));
                        xr[set][b][f][e + 1] = GElem<T>::load(rs_in, (pix[f] + d.z) | (bit_mask(nok[f], d.w) & GATHER_OOB));
                    }
                }
                if constexpr (WROW) {
                    const unsigned off = wrow + (unsigned)(k0 + b * NK) * SZ;
                    if constexpr (sizeof(T) == 4) wv[set][b] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_wt, (int)off, 0, 0));
                    else wv[set][b] = load_bf16x8(rs_wt, off);
                } else {
#pragma unroll
                    for (int e = 0; e < U; e += 4) {
                        const uint4 d = *reinterpret_cast<const uint4 *>(wtab + kk + e);
                        wr[set][b][e] = GElem<T>::load(rs_wt, wrow + d.x);
                        wr[set][b][e + 1] = GElem<T>::load(rs_wt, wrow + d.y);
                        wr[set][b][e + 2] = GElem<T>::load(rs_wt, wrow + d.z);
                        wr[set][b][e + 3] = GElem<T>::load(rs_wt, wrow + d.w);
                    }
                }
            }
        };
        auto multiply = [&](int set, int grp, gf32x16 (&chain)[NF]) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                uint4 a;
                if constexpr (WROW) {
                    a = wv[set][b];
                    // a row goes on past the last index: the next row's elements are no part of the sum
                    const int over = grp * (NK * B) + b * NK + half * U + U - kred;
                    if (__builtin_expect(grp >= ngroups - 1, 0)) {       // uniform
                        uint32_t w4[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if constexpr (sizeof(T) == 4) w4[e] = over >= 4 - e ? 0 : w4[e];
                            else w4[e] = over >= 8 - 2 * e ? 0 : over == 7 - 2 * e ? w4[e] & 0xFFFFu : w4[e];
                        }
                        a = make_uint4(w4[0], w4[1], w4[2], w4[3]);
                    }
                } else {
                    keep_raw(wr[set][b]);
                    a = GElem<T>::pack(wr[set][b]);
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    keep_raw(xr[set][b][f]);
                    chain[f] = mma_pair<T>(a, GElem<T>::pack(xr[set][b][f]), chain[f]);
                }
            }
        };
        request(0, slice);
        for (int grp = slice; grp < ngroups; grp += 2 * KS) {
            // One chain of additions over all indices is as exact as the gather GEMM's where four slices share them; a wave with
            // all of them adds up 32 at a time: relative 2-norm error against 64 bits of fp32 3x3 48 -> 8, 2 x 46 x 59 3.6e-7 in
            // one chain, 1.9e-7 in four (as the gather GEMM), 1.3e-7 this way.
            gf32x16 part[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) part[f] = SHORT ? gf32x16{} : acc[f];
            request(1, grp + KS);
            multiply(0, grp, part);
            request(0, grp + 2 * KS);
            multiply(1, grp + KS < ngroups ? grp + KS : ngroups, part);  // the dead group adds zeros
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f] = SHORT ? acc[f] + part[f] : part[f];
        }
        if constexpr (KS > 1) {
            // slice z adds up the register groups (4 rows) z, z + KS, ... of the tile over all slices
            wg_barrier_nofence();
            float *red = reinterpret_cast<float *>(smem);
#pragma unroll
            for (int v = 0; v < NF * 16; ++v) red[(wave * (NF * 16) + v) * 64 + lane] = acc[v / 16][v % 16];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wg_barrier_nofence();
#pragma unroll
            for (int g = 0; g < NF * 4; ++g) {
                if (g % KS != slice) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float t = 0.f;
#pragma unroll
                    for (int z = 0; z < KS; ++z) t += red[((wave - slice + z) * (NF * 16) + g * 4 + e) * 64 + lane];
                    acc[g / 4][g % 4 * 4 + e] = t;
                }
            }
        }
    }

    const int cw = co0 + 4 * half;
    bool redo = false;
#pragma unroll
    for (int f = 0; f < NF; ++f) redo |= any_nan(acc[f]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo) != 0, 0)) {   // uniform: the block lies out of the way
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            if (m0 + 32 * f + l32 >= M) continue;
            int n, i, j;
            position(m0 + 32 * f + l32, n, i, j);
            gather_redo<T>(p, ca, cb, n, i, j, cw, acc[f]);
        }
    }
    float bias[4][4];
    gather_bias(p, cw, bias);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        if (m0 + 32 * f + l32 >= M) continue;
        int n, i, j;
        position(m0 + 32 * f + l32, n, i, j);
        gather_store<T, KS>(p, ca, cb, n, i, j, cw, 4 * f, slice, bias, acc[f]);
    }
}

// ---------------------------------------------------------------------------------------------- host side

template <typename T, int NF, int KS, int WN, bool WROW>
static hipError_t launch_stream_l(const GatherConvParams &p, unsigned max_m, int classes, size_t lds, hipStream_t st)
{
    static LdsLimitOnce lds_limit;
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&stream_conv<T, NF, KS, WN, WROW>));
    if (e != hipSuccess) return e;
    const dim3 grid((max_m + 32 * NF * WN - 1) / (32 * NF * WN), (p.Cout + 31) / 32, classes);
    const size_t red = KS > 1 ? (size_t)KS * WN * NF * 4096 : 0;
    NGC_LAUNCH((stream_conv<T, NF, KS, WN, WROW>), grid, dim3(64 * KS * WN), lds > red ? lds : red, st, p);
    return launch_result();
}

template <typename T, bool WROW>
static hipError_t launch_stream_t(const GatherConvParams &p, unsigned max_m, int classes, bool sliced, size_t lds, hipStream_t st)
{
    return sliced ? launch_stream_l<T, 1, 4, 1, WROW>(p, max_m, classes, lds, st) : launch_stream_l<T, 1, 1, 4, WROW>(p, max_m, classes, lds, st);
}

StreamChoice stream_conv_choice(const GatherConvParams &p, int dtype, unsigned max_m, int classes)
{
    constexpr StreamChoice NO = {};
    const char *force = env_switch(SW_STREAM);                            // tests only: 0 = never, 1 / 2 = positions / slices
    const int fv = force ? atoi(force) : -1;
    if (fv == 0 || env_switch(SW_GATHER_TILE)) return NO;                // a switch that shapes the gather kernel asks for it
    int nr = 0, ns = 0;
    for (int a = 0; a < p.os_h; ++a) nr = p.nr[a] > nr ? p.nr[a] : nr;
    for (int b = 0; b < p.os_w; ++b) ns = p.ns[b] > ns ? p.ns[b] : ns;
    const int ntaps = nr * ns;
    if (ntaps < 1 || ntaps > STREAM_DEAD) return NO;
    // a filter row lies in the order of the indices: forward (and backprop-data of a single input channel)
    const bool wrow = p.w_chan == ntaps && p.rst_h == 1 && p.rst_w == 1 && p.os_h == 1 && p.os_w == 1;
    const size_t kred = (size_t)ntaps * p.Cin, kpad = (kred + 15) / 16 * 16 + 16, lds = kpad * (wrow ? 8 : 12);
    if (lds > 64 * 1024) return NO;
    // Slices of the reduction or positions: a workgroup's four waves take a tile's reduction in turns, or four tiles.  Times in
    // us of some thirty nodes each of 0.01 to 4 GFLOP: fixed part, steps of a wave, tile-steps and workgroups per compute unit;
    // the estimates are within 10 % (fp32) and 25 % (bf16), the choice between them loses 0.3 % on average, 11 % at most.
    static const double cost[2][2][2][4] = {                              // [bf16][forward][slices]
        {{{3.2, 0.2245, 0.0282, 2.09}, {3.6, 0.243, 0.0515, 0.69}}, {{4.0, 0.164, 0.0133, 1.39}, {3.8, 0.166, 0.0278, 0.83}}},
        {{{4.7, 0.396, 0.0065, 0.0}, {4.2, 0.396, 0.0539, 0.10}}, {{4.25, 0.357, 0.0038, 0.66}, {3.4, 0.484, 0.0446, 0.53}}}};
    const int nk = dtype == NGC_F32 ? 8 : 16;
    const double steps = (double)((kred + nk - 1) / nk), cot = (p.Cout + 31) / 32, tiles = (double)((max_m + 31) / 32) * cot;
    int all_h = 0, all_w = 0;
    for (int a = 0; a < p.os_h; ++a) all_h += p.nr[a];
    for (int b = 0; b < p.os_w; ++b) all_w += p.ns[b];
    const double work = tiles * all_h * all_w * p.Cin / nk / 256;
    const bool strided = p.is_h > 1 || p.is_w > 1 || classes > 1;
    // fp32 backprop-data with stride 1, whose filter operand costs an access per lane: the smaller of two expected times, by rounds
    // of workgroups and the 64-byte lines of a filter load (32 rows, a window each), fitted to the same 1057 launches as the gather
    // GEMM's time (four fifths of them within 20 %).  Over all of them that takes 1.2 % more than the better kernel of each; a
    // limit of 600 tile-steps took 4.6 %.  Gather / this kernel, us: 8 x 96 -> 64 at 45x37, 3x3 30.8 / 33.0; 15 x 128 -> 49 at 54x39, 3x3 58.3
    // / 72.5; 22 x 157 -> 12 at 16x42, 5x5 81.8 / 52.5.
    if (fv < 0 && dtype == NGC_F32 && !wrow && !strided) {
        const double lines = 2 * ntaps + 1 < 32 ? 2 * ntaps + 1 : 32, n = kred / 8.0;
        const double rp = ceil((double)((max_m + 127) / 128) * cot / 256), rs = ceil(tiles / 256);
        const double by_pos = 3.28 + rp * (0.70 + n * (0.1985 + 0.0024 * lines)), by_slice = 3.24 + rs * (0.655 + n / 4 * (0.173 + 0.0033 * lines));
        const bool sliced = by_slice <= by_pos;
        return {(sliced ? by_slice : by_pos) <= gather_f32_bwd_us(p, max_m), sliced, wrow, lds};
    }
    // Elsewhere: tile-steps per compute unit past which the gather GEMM's tiles in LDS, which read an operand once for several
    // fragments, are faster (gather / this kernel, us, some 440 launches of up to 8 GFLOP).  fp32: forward never in the range, except strided (64 -> 160 at
    // 56x56 / 2, 1033 steps 72.9 / 83.5); backprop-data, strided 5x5, 155 18.9 / 23.8.  bf16 NCHW: forward 405 50.0 / 34.6, 1008 65.4 / 122.5, 5x5, 250
    // 18.7 / 23.2; backprop-data 200 21.8 / 27.6, 102 40.7 / 28.1.  bf16 blocked, where the gather kernel reads 16 bytes at a time: 154 31.1 / 57.7,
    // 29 11.3 / 13.5.
    const double most = dtype == NGC_F32 ? (wrow ? (strided ? 600.0 : 1e30) : 130.0)
                        : p.in_blocked   ? 20.0
                        : wrow           ? (ntaps > 9 ? 230.0 : 450.0)
                                         : 100.0;
    if (fv <= 0 && work > most) return NO;
    const double *c0 = cost[dtype != NGC_F32][wrow][0], *c1 = cost[dtype != NGC_F32][wrow][1];
    const double by_pos = c0[0] + c0[1] * steps + c0[2] * work + c0[3] * (double)((max_m + 127) / 128) * cot * classes / 256;
    const double by_slice = c1[0] + c1[1] * (double)((int)(steps + 3) / 4) + c1[2] * work + c1[3] * tiles * classes / 256;
    const bool sliced = fv > 0 ? fv == 2 : by_slice <= by_pos;
    return {true, sliced, wrow, lds};
}

hipError_t launch_stream_conv(const GatherConvParams &p, int dtype, unsigned max_m, int classes, const StreamChoice &c, hipStream_t st)
{
    if (dtype == NGC_F32) return c.wrow ? launch_stream_t<float, true>(p, max_m, classes, c.sliced, c.lds, st) : launch_stream_t<float, false>(p, max_m, classes, c.sliced, c.lds, st);
    return c.wrow ? launch_stream_t<uint16_t, true>(p, max_m, classes, c.sliced, c.lds, st) : launch_stream_t<uint16_t, false>(p, max_m, classes, c.sliced, c.lds, st);
}

}  // namespace ngc
