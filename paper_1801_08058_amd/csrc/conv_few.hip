// Forward and backprop-data of blocked bf16 nodes with few output tiles (gfx950): one image, or a few small ones.
//
// The strip kernel and the 1x1 GEMM give such a node a handful of workgroups, each of which walks all channels and taps in a
// chain of stages through LDS at some 0.4 us a stage, while most compute units idle.  Here a workgroup takes a tile of 32
// output channels x 32 positions (or 64 x 64) and its waves split the reduction: the (tap, 16-channel block) units are dealt to
// NW waves, whose operands go straight from memory to the registers - both blocked layouts hold the 8 consecutive channels of an
// MFMA lane as 16 bytes, a wave reads 1 KB of each - several units of loads in flight at a time.  No LDS ring, no barrier but the
// one in front of the sum of the waves' tiles.
//
// Backprop-data is the same walk over dy with the taps reversed, one class of dx positions per residue modulo the strides
// (gridDim.z of them, one launch): FewAxis holds the taps that meet a class on each axis.  A class that no tap meets stores
// zeros, so nothing clears dx first.
//
// Staged kernels / this one, us.  Backprop-data, one image: 3x3 256 -> 256 at 14x14 18.0 / 6.3, 1x1 256 -> 1024 13.4 / 4.6; strided 3x3
// 512 -> 32, 5 x 46x10 27.6 / 11.0; 3x3x3 224 -> 32 at 6x50x8, stride 2 30.5 / 6.1.  Forward 3x3x3 160 -> 32 at 13x14x24, stride 2 37.1 / 8.8.
// Forward, one image: 1x1 1024 -> 256 at 14x14 13.4 / 3.6 (16 workgroups / 56), 2048 -> 512 at 7x7 21.9 / 4.1,
// 3x3 256 -> 256 at 14x14 18.0 / 6.2 (4 workgroups / 56), 512 -> 512 at 7x7 30.1 / 7.8.
//
// Bound: the latency of U / (B NW) batches of loads and of the sum; many tiles: the L2 reads, 2 KB per MFMA (1 KB with 64 x 64
// tiles), which is why the staged kernels keep the larger nodes (few_rule).  Elements in the padding and channels past the end
// read as zeros through out-of-range offsets.
#include "common.h"

#include <math.h>
#include <stdlib.h>
#include <string.h>

namespace ngc {

typedef __bf16 fbf16x8 __attribute__((ext_vector_type(8)));
typedef float ff32x16 __attribute__((ext_vector_type(16)));

constexpr unsigned FEW_OOB = 0x80000000u;              // past the end of every descriptor below 2 GiB

// NW waves, a tile of TL x TL fragments (channels x positions), B units of loads in flight; R3: depth axis; BWD: several classes,
// ReLU mask, channel sums
template <int NW, int TL, int B, bool R3, bool BWD>
__global__ __launch_bounds__(64 * NW) void conv_few_bf16(const ConvFewArgs<BWD ? FEW_MAX_STRIDE : 1> p)
{
    __shared__ float4 red[NW][TL * TL * 4][64];
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    preload_kernargs(p);
    int rd = 0, rh = 0, rw = 0;
    if (BWD) {
        int z = blockIdx.z;
        rw = z % p.os[2];
        z /= p.os[2];
        rh = R3 ? z % p.os[1] : z;
        rd = R3 ? z / p.os[1] : 0;
    }
    const FewAxis &ad = p.ax[BWD ? rd : 0][0], &ah = p.ax[BWD ? rh : 0][1], &aw = p.ax[BWD ? rw : 0][2];
    // outputs of the class on an axis: indices below ceil((size - residue) / stride), none if the residue lies past the end
    const uint32_t ed = !R3 ? 1u : p.OD > rd ? ad.ext.d : 0u, eh = p.OP > rh ? ah.ext.d : 0u, ew = p.OQ > rw ? aw.ext.d : 0u;
    const uint32_t M = (uint32_t)p.N * ed * eh * ew;
    const uint32_t pos0 = blockIdx.x * 32 * TL;
    if (BWD && pos0 >= M && !p.dbp) return;
    const int k0 = blockIdx.y * 32 * TL;
    const unsigned vol = (unsigned)(p.H * p.W) * (R3 ? (unsigned)p.D : 1u) * 32u;
    bool live[TL];
    int id0[TL], ih0[TL], iw0[TL];
    unsigned x_base[TL], out_at[TL];                   // out_at: the pixel within [N][OD][OP][OQ] planes of 16 channels, n apart
    unsigned img[TL];
#pragma unroll
    for (int m = 0; m < TL; ++m) {
        const uint32_t pos = pos0 + m * 32 + l32;
        live[m] = pos < M;
        uint32_t t = fd_div(pos, aw.ext);
        const int ow = (int)(pos - t * aw.ext.d);
        uint32_t n = fd_div(t, ah.ext);
        const int oh = (int)(t - n * ah.ext.d);
        int od = 0;
        if (R3) {
            t = n;
            n = fd_div(t, ad.ext);
            od = (int)(t - n * ad.ext.d);
        }
        id0[m] = R3 ? od * p.is[0] + ad.off0 : 0;
        ih0[m] = oh * p.is[1] + ah.off0;
        iw0[m] = ow * p.is[2] + aw.off0;
        x_base[m] = n * (unsigned)p.CB * vol + half * 16;
        img[m] = n;
        unsigned o = (unsigned)(BWD ? oh * p.os[1] + rh : oh) * (unsigned)p.OQ + (unsigned)(BWD ? ow * p.os[2] + rw : ow);
        if (R3) o += (unsigned)(BWD ? od * p.os[0] + rd : od) * (unsigned)(p.OP * p.OQ);
        out_at[m] = o;
    }
    unsigned w_base[TL];
#pragma unroll
    for (int c = 0; c < TL; ++c) {
        const int k = k0 + c * 32 + l32;
        w_base[c] = k < p.K ? (unsigned)k * 32 + half * 16 : FEW_OOB;   // past the end: stays so with any offset below 2 GiB added
    }
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.in), 0, (int)p.in_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw_ = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.wt), 0, (int)p.wt_bytes, 0x00020000);

    ff32x16 acc[TL][TL];
#pragma unroll
    for (int c = 0; c < TL; ++c)
#pragma unroll
        for (int m = 0; m < TL; ++m)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][m][i] = 0.f;
    // unit = tap * CB + cb over the taps of the class; this wave's units are wave, wave + NW, ..
    const int ns = aw.cnt, nr = ah.cnt, U = (R3 ? ad.cnt : 1) * nr * ns * p.CB;
    int cb = wave, t = 0, r = 0, s = 0;
    for (int u0 = wave; u0 < U; u0 += NW * B) {
        __uint128_t xv[B][TL], wv[B][TL];
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const bool in_u = u0 + j * NW < U;
            while (cb >= p.CB) {                       // next tap: at most NW times, CB >= 1
                cb -= p.CB;
                if (++s == ns) {
                    s = 0;
                    if (++r == nr && R3) {
                        r = 0;
                        ++t;
                    }
                }
            }
            const int dd = R3 ? t * ad.doff : 0, dh = r * ah.doff, dw = s * aw.doff;
            int row = u0 + j * NW;                     // of the filter: forward has all taps, in order
            if (BWD) {
                int slab = (ah.t0 + r * ah.tstep) * p.S + aw.t0 + s * aw.tstep;
                if (R3) slab += (ad.t0 + t * ad.tstep) * p.R * p.S;
                row = slab * p.CB + cb;
            }
            const unsigned wo = (unsigned)row * (unsigned)p.K * 32;
#pragma unroll
            for (int m = 0; m < TL; ++m) {
                const int id = id0[m] + dd, ih = ih0[m] + dh, iw = iw0[m] + dw;
                const bool ok = in_u && live[m] && (!R3 || (unsigned)id < (unsigned)p.D) && (unsigned)ih < (unsigned)p.H && (unsigned)iw < (unsigned)p.W;
                const unsigned line = R3 ? (unsigned)id * (unsigned)p.H + (unsigned)ih : (unsigned)ih;
                const unsigned xo = x_base[m] + (unsigned)cb * vol + (line * (unsigned)p.W + (unsigned)iw) * 32;
                xv[j][m] = __builtin_bit_cast(__uint128_t, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? xo : FEW_OOB), 0, 0));
            }
#pragma unroll
            for (int c = 0; c < TL; ++c)
                wv[j][c] = __builtin_bit_cast(__uint128_t, __builtin_amdgcn_raw_buffer_load_b128(rw_, (int)(in_u ? w_base[c] + wo : FEW_OOB), 0, 0));
            cb += NW;
        }
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
            for (int c = 0; c < TL; ++c)
#pragma unroll
                for (int m = 0; m < TL; ++m)
                    acc[c][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(fbf16x8, wv[j][c]), __builtin_bit_cast(fbf16x8, xv[j][m]), acc[c][m], 0, 0, 0);
    }
    // acc[c][m][4 q + v]: channel k0 + 32 c + 8 q + 4 half + v of position 32 m + lane % 32
#pragma unroll
    for (int c = 0; c < TL; ++c)
#pragma unroll
        for (int m = 0; m < TL; ++m)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                red[wave][(c * 4 + q) * TL + m][lane] = make_float4(acc[c][m][4 * q], acc[c][m][4 * q + 1], acc[c][m][4 * q + 2], acc[c][m][4 * q + 3]);
    __syncthreads();
    if (wave >= TL * 4) return;                        // wave w sums the channel quads w of all positions: TL * 4 <= NW
    const int k = k0 + 8 * wave + 4 * half;            // 32 (w / 4) + 8 (w % 4) + 4 half
    if (k >= p.K) return;
    float cs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < TL; ++m) {
        if (!live[m]) continue;
        float f[4] = {0.f, 0.f, 0.f, 0.f};
        if (!BWD && p.bias) {
#pragma unroll
            for (int v = 0; v < 4; ++v) f[v] = p.bias[k + v];
        }
#pragma unroll
        for (int w = 0; w < NW; ++w) {                 // fixed order
            const float4 t4 = red[w][wave * TL + m][lane];
            f[0] += t4.x; f[1] += t4.y; f[2] += t4.z; f[3] += t4.w;
        }
        uint2 o = make_uint2(pack_bf16x2_hw(f[0], f[1]), pack_bf16x2_hw(f[2], f[3]));
        const size_t at = (((size_t)img[m] * (p.K >> 4) + (k >> 4)) * (unsigned)(p.OP * p.OQ * (R3 ? p.OD : 1)) + out_at[m]) * 16 + (k & 15);
        if (BWD) {
            if (p.mask) {
                const uint2 mk = *reinterpret_cast<const uint2 *>(p.mask + at);
                o.x = relu_keep2(o.x, mk.x);
                o.y = relu_keep2(o.y, mk.y);
            }
            if (p.dbp) {                               // the rounded, masked values as stored
                cs[0] += __uint_as_float(o.x << 16);
                cs[1] += __uint_as_float(o.x & 0xFFFF0000u);
                cs[2] += __uint_as_float(o.y << 16);
                cs[3] += __uint_as_float(o.y & 0xFFFF0000u);
            }
        } else {
            o.x = relu_bf16x2(o.x, p.relu);
            o.y = relu_bf16x2(o.y, p.relu);
        }
        *reinterpret_cast<uint2 *>(p.out + at) = o;
    }
    if (BWD && p.dbp) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int x = 16; x > 0; x >>= 1) cs[v] += __shfl_xor(cs[v], x, 64);    // within the half: same channels
        if (l32 == 0) *reinterpret_cast<float4 *>(p.dbp + (size_t)(blockIdx.z * gridDim.x + blockIdx.x) * p.dbp_ld + k) = make_float4(cs[0], cs[1], cs[2], cs[3]);
    }
}

namespace {

// either rank as a rank-3 node
struct FewNode {
    int n, c, k;
    int in[3], taps[3], stride[3], dil[3], pad[3], out[3];
    bool r3;
};

// Expected times, us: a start and, per round of workgroups (256 compute units; two workgroups of 8 waves and one fragment start on
// each), a start of its own, the units of a wave and the taps it walks past (every wave counts through all of them, at more cost with
// a depth axis and for the classes of backprop-data), at least one round of the class with most taps; up to 64 units also the
// operands' bytes through the L2s, at the share of them that the workgroups reach.  Fitted to 3245 launches of up to 3000 tiles, back
// to back in a graph: four fifths of them within 20 % (32 x 32 tiles) and 12 % (64 x 64).  Small tiles over the classes of rank 3 take
// 0.025 a unit more (303 launches: the choice of the tile costs 0.9 % with it, 4 % without, 1.7 times the better tile at worst).
double few_us(int tl, size_t M, int Cout, int CB, int classes, int units, double mean_units, bool r3, bool bwd)
{
    const double tiles = (double)((M + 32 * tl - 1) / (32 * tl)) * ((Cout + 32 * tl - 1) / (32 * tl)) * classes, rounds = ceil(tiles / 256);
    const double walk = mean_units / CB, longest = (double)units / CB;
    const double classes3 = tl == 1 && r3 && classes > 1 ? 0.025 * (rounds * mean_units > units ? rounds * mean_units : units) : 0.0;
    if (tl == 1 && units <= 64) {
        const double tap = 0.021 + 0.035 * r3 + 0.038 * bwd, share = tiles < 256 ? (tiles < 5 ? 0.02 : tiles / 256) : 1.0;
        return 1.77 + ceil(tiles / 512) * 0.68 + tap * (rounds * walk > longest ? rounds * walk : longest) + 65e-6 * tiles * mean_units / share + classes3;
    }
    const double wg = tl == 2 ? 2.43 : 1.67, unit = tl == 2 ? 0.242 / 8 : 0.212 / 16;
    const double tap = tl == 2 ? 0.014 + 0.052 * r3 + 0.017 * bwd : 0.026 + 0.079 * r3 + 0.063 * bwd;
    const double all = rounds * (wg + unit * mean_units + tap * walk), one = wg + unit * units + tap * longest;
    return (tl == 2 ? 0.89 : 1.45) + (all > one ? all : one) + classes3;
}

// The tile (fragments per axis) of a node, 0: the staged kernels, which take staged_us (0: no estimate; below: already decided
// against them).  units: of the class with most taps; mean_units: of a class on average
int few_rule(size_t M, int Cout, int CB, int classes, int units, double mean_units, double staged_us, bool r3, bool bwd, bool strided)
{
    const char *force = env_switch(SW_FWD_FEW);        // tests / benchmarks only: 0 = never, 1 / 2 = wherever it can, that tile
    const int fv = force ? atoi(force) : -1;
    if (fv >= 0) return fv > 2 ? 0 : fv;
    const double one = few_us(1, M, Cout, CB, classes, units, mean_units, r3, bwd), two = few_us(2, M, Cout, CB, classes, units, mean_units, r3, bwd);
    // the larger tile only where it reaches a good third of the compute units: fewer have too few loads in flight for operands from
    // memory (1x1 backprop-data 1728 -> 64, 49 x 9x11, 304 tiles of 32, 76 of 64 10.4 / 13.5 us; in cache 8.1 / 6.7)
    const int tile = two < one && (M + 63) / 64 * ((Cout + 63) / 64) * classes >= 96 ? 2 : 1;
    if (staged_us < 0) return tile;
    // a switch that shapes the staged kernels asks for them
    for (Switch sw : {SW_STRIP_NF, SW_STRIP_ROWS, SW_STRIP_BW, SW_STRIP_XCD, SW_STRIP_TAIL, SW_STRIP_SPLIT, SW_STRIP_CPS, SW_STRIP_STRIDED, SW_G1_VARIANT, SW_ROWS})
        if (env_switch(sw)) return 0;
    // About one round of workgroups and a reduction worth dealing out: here, unless expected to take longer (one round: by a tenth, the
    // estimates' error).  Beyond that only where it is expected to take a fifth less (two fifths with a reduction of under 8 units),
    // and not for more than 3000 tiles (5220 of 124 units 36.5 / 96.7 / 65.0) nor forward with strided reads, which fetch whole lines
    // for half of them (13 x 1024 -> 384, 1x1 stride 2 12.8 / 21.7 with tiles of 64).  Staged / 32 / 64, us: backprop-data of 4 x 64 -> 48
    // at 40x40, 5x5 (400 tiles of 75 units) 10.0 / 12.1 / 6.8, of 224 -> 48 at 42x31 (287, 84 of 64: staged) the same; 3x3x3 48 -> 80 (390
    // of 81) 11.6 / 15.1 / 7.8; 3x3, 176 -> 384 (468 of 99) 13.6 / 7.0 / 6.5.  2733 launches that the estimates were not fitted to take
    // 16.0 ms so, 31.5 staged, 15.0 the best of the three; 1269 with operands from memory 8.1, 15.5 and 7.5.
    const double us = tile == 2 ? two : one;
    const size_t tiles = (M + 31) / 32 * ((Cout + 31) / 32) * classes;
    if ((tiles <= 256 && units >= 8) || (tiles <= 448 && units >= 32)) return staged_us == 0.0 || us < (tiles <= 256 ? 1.1 : 1.0) * staged_us ? tile : 0;
    return tiles <= 3000 && !strided && us < (units >= 8 ? 0.8 : 0.6) * staged_us ? tile : 0;
}

bool few_plan(const FewNode &d, bool bwd, double staged_us, ConvFewParams *out)
{
    const int Cin = bwd ? d.k : d.c, Cout = bwd ? d.c : d.k;
    if (Cin % 16 || Cout % 16) return false;
    const int *in = bwd ? d.out : d.in, *os = bwd ? d.in : d.out;      // sizes of what is read and of what is written
    const size_t ivol = (size_t)in[0] * in[1] * in[2], ovol = (size_t)os[0] * os[1] * os[2];
    const size_t in_bytes = (size_t)d.n * Cin * ivol * 2, wt_bytes = (size_t)d.taps[0] * d.taps[1] * d.taps[2] * Cin * Cout * 2;
    const size_t lim = (size_t)1 << 31;
    if (in_bytes >= lim || wt_bytes >= lim || (size_t)d.n * Cout * ovol * 2 >= lim || (size_t)d.n * ovol >= ((size_t)1 << 24) || Cout > 32 * 65535) return false;
    ConvFewParams q;
    memset(&q, 0, sizeof(q));
    q.classes = 1;
    size_t M = (size_t)d.n;
    size_t ntaps = 1;
    for (int a = 0; a < 3; ++a) {
        const int st = d.stride[a], dil = d.dil[a], taps = d.taps[a], pad = d.pad[a];
        q.is[a] = bwd ? 1 : st;
        q.os[a] = bwd ? st : 1;
        if (!bwd) {
            q.ax[0][a] = FewAxis{taps, -pad, dil, 0, 1, make_fastdiv((uint32_t)os[a])};
            M *= os[a];
            ntaps *= taps;
            continue;
        }
        if (st > FEW_MAX_STRIDE) return false;
        q.classes *= st;
        M *= (os[a] + st - 1) / st;
        int g = st, most = 0;                          // gcd(st, dil)
        for (int b = dil; b;) { const int m = g % b; g = b; b = m; }
        for (int res = 0; res < st; ++res) {
            FewAxis x = {0, 0, -(dil / g), 0, st / g, make_fastdiv(os[a] > res ? (uint32_t)((os[a] - res + st - 1) / st) : 1u)};
            for (int t = 0; t < taps; ++t) {
                const int v = res + pad - t * dil;
                if (((v % st) + st) % st != 0) continue;
                if (x.cnt == 0) {
                    x.t0 = t;
                    x.off0 = v / st;                   // exact
                }
                ++x.cnt;
            }
            if (x.cnt > most) most = x.cnt;
            q.ax[res][a] = x;
        }
        ntaps *= most;
    }
    const size_t units = ntaps * (Cin / 16);
    if (units > (size_t)1 << 24) return false;
    const double mean = bwd ? (double)(wt_bytes / 2 / 16 / Cout) / q.classes : (double)units;
    q.tile = few_rule(M, Cout, Cin / 16, q.classes, (int)units, mean, staged_us, d.r3, bwd, !bwd && d.stride[2] > 1);
    if (q.tile == 0) return false;
    if (!out) return true;
    q.in_bytes = (uint32_t)in_bytes;
    q.wt_bytes = (uint32_t)wt_bytes;
    q.N = d.n; q.CB = Cin / 16; q.K = Cout;
    q.D = in[0]; q.H = in[1]; q.W = in[2];
    q.R = d.taps[1]; q.S = d.taps[2];
    q.OD = os[0]; q.OP = os[1]; q.OQ = os[2];
    q.M = (uint32_t)M;
    q.units = (int)units;
    q.r3 = d.r3;
    q.bwd = bwd;
    *out = q;
    return true;
}

}  // namespace

// Expected times of the staged kernels on nodes of this range, back to back in a graph as few_us (2618 launches, nine tenths within
// 15 %): rounds of workgroups, each a chain of stages of 16 input channels (times depth taps).  Strided backprop-data takes up to
// twice as long, one class of pixels after the other; that is not in them.
double few_strip_us(double workgroups, int stages, int taps, int nf)
{
    const double rounds = workgroups <= 256 ? 1.0 : (double)(((long)workgroups + 255) / 256);
    return 1.9 + rounds * (1.24 + stages * (0.243 + taps * (0.0263 * nf + 0.0289)));
}

double few_gemm1x1_us(size_t M, int Cin, int Cout)
{
    const double tiles = (double)((M + 63) / 64) * ((Cout + 63) / 64);
    return 3.0 + 0.171 * (tiles > 512 ? tiles / 512 : 1.0) * (Cin / 16);
}

bool conv_few_plan(const ngc_conv_desc *d, int op, int P, int Q, double staged_us, ConvFewParams *q)
{
    const FewNode nd = {d->n, d->c, d->k, {1, d->h, d->w}, {1, d->r, d->s}, {1, d->stride_h, d->stride_w}, {1, d->dil_h, d->dil_w},
                        {0, d->pad_below_h, d->pad_below_w}, {1, P, Q}, false};
    return few_plan(nd, op != NGC_OP_FWD, staged_us, q);
}

bool conv_few_plan3(const ngc_conv3d_desc *d, int op, int O, int P, int Q, double staged_us, ConvFewParams *q)
{
    const FewNode nd = {d->n, d->c, d->k, {d->d, d->h, d->w}, {d->t, d->r, d->s}, {d->stride_d, d->stride_h, d->stride_w},
                        {d->dil_d, d->dil_h, d->dil_w}, {d->pad_below_d, d->pad_below_h, d->pad_below_w}, {O, P, Q}, true};
    return few_plan(nd, op != NGC_OP_FWD, staged_us, q);
}

static unsigned few_tiles_m(const ConvFewParams &p) { return (p.M + 32 * p.tile - 1) / (32 * p.tile); }

int conv_few_dbp_rows(const ConvFewParams &p) { return (int)few_tiles_m(p) * p.classes; }

template <bool R3, bool BWD>
static hipError_t launch_few(const ConvFewParams &p, hipStream_t st)
{
    const dim3 grid(few_tiles_m(p), (unsigned)((p.K + 32 * p.tile - 1) / (32 * p.tile)), (unsigned)p.classes);
    ConvFewArgs<BWD ? FEW_MAX_STRIDE : 1> a;
    static_cast<ConvFewHead &>(a) = p;
    memcpy(a.ax, p.ax, sizeof(a.ax));
    // a batch no larger than what a wave has to do: loads past the last unit cost their issue (53 x 32 -> 416, 3x3, 18 units:
    // 100 us with batches of 8); separate kernels, since one with all batch sizes fetches 0.4 us more code
    if (p.tile == 2) {
        if (p.units > 16) NGC_LAUNCH((conv_few_bf16<8, 2, 4, R3, BWD>), grid, dim3(512), 0, st, a);
        else NGC_LAUNCH((conv_few_bf16<8, 2, 2, R3, BWD>), grid, dim3(512), 0, st, a);
    } else if (p.units > 64) NGC_LAUNCH((conv_few_bf16<16, 1, 8, R3, BWD>), grid, dim3(1024), 0, st, a);
    else if (p.units > 32) NGC_LAUNCH((conv_few_bf16<8, 1, 8, R3, BWD>), grid, dim3(512), 0, st, a);
    else if (p.units > 16) NGC_LAUNCH((conv_few_bf16<8, 1, 4, R3, BWD>), grid, dim3(512), 0, st, a);
    else NGC_LAUNCH((conv_few_bf16<8, 1, 2, R3, BWD>), grid, dim3(512), 0, st, a);
    return launch_result();
}

hipError_t launch_conv_few(const ConvFewParams &p, hipStream_t st)
{
    if (p.r3) return p.bwd ? launch_few<true, true>(p, st) : launch_few<true, false>(p, st);
    return p.bwd ? launch_few<false, true>(p, st) : launch_few<false, false>(p, st);
}

}  // namespace ngc
