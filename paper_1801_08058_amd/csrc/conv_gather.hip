// The Convolution op family on the matrix cores for the nodes the blocked bf16 kernels do not take: fp32 tensors, channel
// counts that are no multiple of 16, NCHW tensors of such nodes, low-channel first layers (gfx950).  Any stride, padding,
// dilation and window of up to 31 x 31, both element types, both data layouts, KCRS filters.
//
// Forward and backprop-data are one gather GEMM:
//   out[co][pos] = sum_kk wt[co][kk] * in[kk][pos],   kk = (reduction channel, tap row, tap column), columns fastest
// backprop-data runs one residue class of the output pixels modulo the stride per grid slice, whose taps are an arithmetic
// progression in each axis, so both directions walk kk with the same three counters.  Backprop-filters is the GEMM over
// positions dw[k][crs] = sum_pos dy[k][pos] * x[crs][pos].
//
// Operands are gathered element by element through buffer descriptors (elements in the padding, of channels or positions
// past the end get an out-of-range offset and read as zeros), packed into 16-byte units of U = 4 (fp32) or 8 (bf16)
// consecutive reduction indices and kept in LDS as planes [unit][row], so an MFMA operand is one conflict-free
// ds_read_b128.  fp32 runs on v_mfma_f32_32x32x2_f32 (fp32 products and sums, 157 TFLOP/s), bf16 on
// v_mfma_f32_32x32x16_bf16.
//
// What bounds it: the gather, four vector instructions and a load per element.  A 64 x 64 step of two slices takes 0.95 us on
// a chip with work for every unit, of which the fp32 matrix pipes have 0.43 us (1024 cycles).  conv_stream.hip and wgrad_stream.hip
// take the nodes they are expected to run faster; here run the others: large ones, windows of more than 31 taps, reductions past
// the index table, backprop-filters of blocked tensors.
#include "conv_gather.h"

#include <math.h>
#include <stdlib.h>

namespace ngc {

// A walk over kk: (channel, tap row, tap column), advanced a step of the reduction at a time
struct KWalk {
    int c, r, s;
    __device__ void start(int kk, int nr, int ns)
    {
        // quotients of small numbers (kk < 2^12, at most 31 x 31 taps) by the hardware reciprocal: exact, kk + 1/2 keeps
        // them half a divisor's share away from the next integer
        c = (int)(((float)kk + 0.5f) * __builtin_amdgcn_rcpf((float)(nr * ns)));
        const int t = kk - c * nr * ns;
        r = (int)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)ns));
        s = t - r * ns;
    }
    __device__ void advance(const KWalk &d, int nr, int ns)
    {
        s += d.s;
        const bool ws = s >= ns;
        s -= ws ? ns : 0;
        r += d.r + ws;
        const bool wr = r >= nr;
        r -= wr ? nr : 0;
        c += d.c + wr;
    }
};

// One workgroup: BM output channels x BN positions, WM x WN waves side by side times KS slices of the reduction: a slice
// takes UPS units (plane pairs) of every step, the accumulators of the slices are added in slice order through LDS at the
// end.  PF: steps requested ahead of the one being multiplied.  WV: a unit of kk is contiguous and aligned in the filter.
//
// Where the elements of a step lie (channel and tap offsets, tap row and column for the padding test) is worked out once
// per workgroup, one kk per thread, a step ahead, and handed round through a small ring in LDS: decoding kk in every thread
// cost more than the rest of the gather.
template <typename T, int BM, int BN, int WM, int WN, int KS, int UPS>
struct GatherTile {
    static constexpr int NW = WM * WN * KS, NT = 64 * NW, MF = BM / WM / 32, NF = BN / WN / 32;
    static constexpr int NU = UPS * KS, NK = NU * GElem<T>::U;           // units and reduction indices per step
    static constexpr int XU = NU * BN / NT, WU = (NU * BM + NT - 1) / NT;    // units a thread brings per step
    static constexpr int XPL = BN * 16, WPL = BM * 16, BUF = NU * (XPL + WPL);
    static constexpr int RED = KS > 1 ? NW * MF * NF * 16 * 64 * 4 : 0;
    static constexpr int ENT = NK * 8, ENTW = NK * 4;                    // a ring slot: {x offset, tap} pairs, filter offsets
    static constexpr size_t RING = 2 * BUF > RED ? 2 * BUF : RED, LDS = RING + 4 * (ENT + ENTW);
    static_assert(NU * BN % NT == 0 && MF * NF > 0 && NK <= NT && UPS % 2 == 0, "tile shape");
};

template <typename T, int BM, int BN, int WM, int WN, int KS, int UPS, bool WV>
__global__ __launch_bounds__(64 * WM * WN * KS) void gather_conv(const GatherConvParams p)
{
    preload_kernargs(p);
    typedef GatherTile<T, BM, BN, WM, WN, KS, UPS> G;
    constexpr int U = GElem<T>::U, NT = G::NT, MF = G::MF, NF = G::NF, NU = G::NU, NK = G::NK, XU = G::XU, WU = G::WU, PF = 2;
    constexpr int XPL = G::XPL, WPL = G::WPL, BUF = G::BUF, ENT = G::ENT, ENTW = G::ENTW;
    constexpr unsigned SZ = sizeof(T);
    extern __shared__ __align__(16) unsigned char smem[];
    unsigned char *ring = smem + G::RING;                                // four slots

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int wn = wave % WN, wm = wave / WN % WM, slice = wave / (WN * WM);

    const int ca = (int)blockIdx.z / p.os_w, cb = (int)blockIdx.z - ca * p.os_w;           // residue class of this grid slice
    const int nr = p.nr[ca], ns = p.ns[cb], OP = p.oph[ca], OQ = p.opw[cb];
    const int kred = nr * ns * p.Cin;
    const unsigned M = (unsigned)p.N * OP * OQ;
    const unsigned m0 = blockIdx.x * BN;
    if (m0 >= M) return;                                                 // uniform per workgroup
    const int co0 = blockIdx.y * BM;
    const FastDiv div_pq = p.div_pq[2 * (OP != p.oph[0]) + (OQ != p.opw[0])], div_q = p.div_q[OQ != p.opw[0]];
    auto position = [&](unsigned m, int &n, int &i, int &j) {
        n = (int)fd_div(m, div_pq);
        const unsigned t = m - (unsigned)n * div_pq.d;
        i = (int)fd_div(t, div_q);
        j = (int)(t - (unsigned)i * div_q.d);
    };

    gf32x16 acc[MF][NF];
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
        for (int b = 0; b < NF; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    if (kred > 0) {
        // this thread's position: byte offset of tap (0, 0), and per tap row / column whether it lies inside the image
        const int xpos = tid % BN, xu0 = tid / BN;
        unsigned pix = 0, okr = 0, okc = 0;
        if (m0 + xpos < M) {
            int n, i, j;
            position(m0 + xpos, n, i, j);
            const int ih = i * p.is_h + p.base_h[ca], iw = j * p.is_w + p.base_w[cb];
            pix = (unsigned)(n * p.in_n + (ih * p.Win + iw) * p.in_px) * SZ;
            for (int r = 0; r < nr; ++r) okr |= (unsigned)((unsigned)(ih + r * p.step_h) < (unsigned)p.Hin) << r;
            for (int s = 0; s < ns; ++s) okc |= (unsigned)((unsigned)(iw + s * p.step_w) < (unsigned)p.Win) << s;
        }
        const int wrow = tid % BM, wu0 = tid / BM;
        const unsigned wbase = co0 + wrow < p.Cout && wu0 < NU ? (unsigned)((co0 + wrow) * p.w_row + p.r0[ca] * p.S + p.s0[cb]) * SZ : GATHER_OOB;
        const __amdgpu_buffer_rsrc_t rs_in = __builtin_amdgcn_make_buffer_rsrc((void *)p.in, 0, (int)p.in_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t rs_wt = __builtin_amdgcn_make_buffer_rsrc((void *)p.wt, 0, (int)p.wt_bytes, 0x00020000);
        const int nsteps = (kred + NK - 1) / NK;
        const int row_off = p.step_h * p.Win * p.in_px * (int)SZ, col_off = p.step_w * p.in_px * (int)SZ;

        KWalk ek, dk;
        ek.start(tid, nr, ns);
        dk.start(NK, nr, ns);
        auto entries = [&](int step) {                                   // kk = step * NK + tid of threads 0 .. NK - 1
            if (tid < NK) {
                const bool live = ek.c < p.Cin;
                const unsigned chan = p.in_blocked ? (unsigned)(ek.c >> 4) * p.in_c + (ek.c & 15) : (unsigned)ek.c * p.in_c;
                const unsigned xo = (unsigned)(ek.r * row_off + ek.s * col_off) + chan * SZ;
                const unsigned wo = ((unsigned)ek.c * p.w_chan + ek.r * p.rst_h * p.S + ek.s * p.rst_w) * SZ;
                unsigned char *slot = ring + (step & 3) * (ENT + ENTW);
                *reinterpret_cast<uint2 *>(slot + tid * 8) = make_uint2(xo, live ? (unsigned)(ek.r | ek.s << 8) : 0x1F1Fu);   // bit 31: never inside
                // past the last index: wt_bytes, out of range on its own and on top of a wbase that already is (twice
                // GATHER_OOB would wrap to filter element 0)
                *reinterpret_cast<unsigned *>(slot + ENT + tid * 4) = live ? wo : p.wt_bytes;
            }
            ek.advance(dk, nr, ns);
        };
        uint32_t xr[PF][XU][U], wr[PF][WV ? 1 : WU][U];
        uint4 wv[PF][WV ? WU : 1];
        auto request = [&](int set, int step) {
            const unsigned char *slot = ring + (step & 3) * (ENT + ENTW);
#pragma unroll
            for (int i = 0; i < XU; ++i)
#pragma unroll
                for (int e = 0; e < U; e += 2) {
                    const uint4 d = *reinterpret_cast<const uint4 *>(slot + ((xu0 + i * (NT / BN)) * U + e) * 8);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const unsigned off = pix + (h ? d.z : d.x), tap = h ? d.w : d.y;
                        const unsigned ok = bit_mask(okr, tap) & bit_mask(okc, tap >> 8);
                        xr[set][i][e + h] = GElem<T>::load(rs_in, off | (GATHER_OOB & ~ok));
                    }
                }
#pragma unroll
            for (int i = 0; i < WU; ++i) {
                const int wu = wu0 + i * (NT / BM);
                if constexpr (WV) {
                    const int kk = (step * NU + wu) * U;
                    const unsigned off = kk < kred ? wbase + (unsigned)kk * SZ : GATHER_OOB;
                    wv[set][i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_wt, (int)off, 0, 0));
                } else {
#pragma unroll
                    for (int e = 0; e < U; e += 4) {
                        const uint4 d = *reinterpret_cast<const uint4 *>(slot + ENT + ((wu < NU ? wu : 0) * U + e) * 4);
                        wr[set][i][e] = GElem<T>::load(rs_wt, wbase + d.x);
                        wr[set][i][e + 1] = GElem<T>::load(rs_wt, wbase + d.y);
                        wr[set][i][e + 2] = GElem<T>::load(rs_wt, wbase + d.z);
                        wr[set][i][e + 3] = GElem<T>::load(rs_wt, wbase + d.w);
                    }
                }
            }
        };
        auto stage = [&](int set, int step) {
            unsigned char *xs = smem + (step & 1) * BUF, *ws = xs + NU * XPL;
#pragma unroll
            for (int i = 0; i < XU; ++i) keep_raw(xr[set][i]);
#pragma unroll
            for (int i = 0; i < (WV ? 0 : WU); ++i) keep_raw(wr[set][i]);
#pragma unroll
            for (int i = 0; i < XU; ++i)
                *reinterpret_cast<uint4 *>(xs + (xu0 + i * (NT / BN)) * XPL + xpos * 16) = GElem<T>::pack(xr[set][i]);
#pragma unroll
            for (int i = 0; i < WU; ++i)
                if (NU * BM >= NT || wu0 < NU)
                    *reinterpret_cast<uint4 *>(ws + (wu0 + i * (NT / BM)) * WPL + wrow * 16) = WV ? wv[set][WV ? i : 0] : GElem<T>::pack(wr[set][WV ? 0 : i]);
        };
        auto multiply = [&](int step) {
            const unsigned char *xs = smem + (step & 1) * BUF, *ws = xs + NU * XPL;
#pragma unroll
            for (int q = 0; q < UPS / 2; ++q) {
                const int pl = slice * UPS + 2 * q + half;
                uint4 xb[NF];
#pragma unroll
                for (int b = 0; b < NF; ++b) xb[b] = *reinterpret_cast<const uint4 *>(xs + pl * XPL + ((wn * NF + b) * 32 + l32) * 16);
#pragma unroll
                for (int a = 0; a < MF; ++a) {
                    const uint4 wa = *reinterpret_cast<const uint4 *>(ws + pl * WPL + ((wm * MF + a) * 32 + l32) * 16);
#pragma unroll
                    for (int b = 0; b < NF; ++b) acc[a][b] = mma_pair<T>(wa, xb[b], acc[a][b]);
                }
            }
        };
#pragma unroll
        for (int f = 0; f <= PF; ++f) entries(f);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier_nofence();
        // The first PF rounds only request (they stage and multiply zeros under the latency of the first loads): a loop with
        // a prologue of its own keeps the steps in flight in other registers than the loop and waits for all of them to copy.
#pragma unroll
        for (int f = 0; f < PF; ++f) {
#pragma unroll
            for (int e = 0; e < U; ++e) {
#pragma unroll
                for (int i = 0; i < XU; ++i) xr[f][i][e] = 0;
#pragma unroll
                for (int i = 0; i < (WV ? 1 : WU); ++i) wr[f][i][e] = 0;
            }
#pragma unroll
            for (int i = 0; i < (WV ? WU : 1); ++i) wv[f][i] = make_uint4(0, 0, 0, 0);
        }
        for (int s = -PF; s < nsteps; s += PF) {
#pragma unroll
            for (int f = 0; f < PF; ++f) {
                stage(f, s + f);
                request(f, s + f + PF);                                  // past the end: every offset out of range
                if (s + f >= 0) entries(s + f + PF + 1);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wg_barrier_nofence();
                multiply(s + f);                                         // a step past the end adds zeros
            }
        }
        if constexpr (KS > 1) {
            // slice z adds up the register groups (4 rows) z, z + KS, ... of its wave position over all slices
            wg_barrier_nofence();
            float *red = reinterpret_cast<float *>(smem);
#pragma unroll
            for (int v = 0; v < MF * NF * 16; ++v) red[(wave * (MF * NF * 16) + v) * 64 + lane] = acc[v / 16 / NF][v / 16 % NF][v % 16];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            wg_barrier_nofence();
#pragma unroll
            for (int g = 0; g < MF * NF * 4; ++g) {
                if (g % KS != slice) continue;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float t = 0.f;
#pragma unroll
                    for (int z = 0; z < KS; ++z) t += red[((wave % (WN * WM) + z * WN * WM) * (MF * NF * 16) + g * 4 + e) * 64 + lane];
                    acc[g / 4 / NF][g / 4 % NF][g % 4 * 4 + e] = t;
                }
            }
        }
    }

    const int cw = co0 + wm * MF * 32 + 4 * half;                        // this lane's first channel
    const unsigned mw = m0 + wn * NF * 32 + l32;
    bool redo = false;
#pragma unroll
    for (int a = 0; a < MF; ++a)
#pragma unroll
        for (int b = 0; b < NF; ++b) redo |= any_nan(acc[a][b]);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(redo) != 0, 0)) {     // uniform: the block lies out of the way
#pragma unroll
        for (int a = 0; a < MF; ++a)
#pragma unroll
            for (int b = 0; b < NF; ++b) {
                if (mw + 32 * b >= M) continue;
                int n, i, j;
                position(mw + 32 * b, n, i, j);
                gather_redo<T>(p, ca, cb, n, i, j, cw + a * 32, acc[a][b]);
            }
    }
#pragma unroll
    for (int a = 0; a < MF; ++a) {
        float bias[4][4];
        gather_bias(p, cw + a * 32, bias);
#pragma unroll
        for (int b = 0; b < NF; ++b) {
            const unsigned m = mw + 32 * b;
            if (m >= M) continue;
            int n, i, j;
            position(m, n, i, j);
            gather_store<T, KS>(p, ca, cb, n, i, j, cw + a * 32, (a * NF + b) * 4, slice, bias, acc[a][b]);
        }
    }
}

struct GatherWgradParams {
    const void *x, *dy;
    float *out;                    // [parts][pitch] partial sums, or dw itself (one part)
    uint32_t x_bytes, dy_bytes;
    int32_t C, H, W, K, P, Q, R, S;
    int32_t sh, sw, dil_h, dil_w, pb_h, pb_w;
    int32_t x_n, x_c, x_px, x_blocked, dy_n, dy_c, dy_px, dy_blocked;    // element strides, as in GatherConvParams
    int32_t ctiles;
    uint32_t M, chunk;             // positions; positions per part (a multiple of the step)
    uint32_t pitch;                // floats between the parts
    FastDiv div_pq, div_q;
};

// One workgroup: BT output channels x BT (c, r, s) columns of dw over a chunk of positions; (BT / 32)^2 waves side by side
// times KS slices of every step's positions, UPS units each.  DYV / XV: the U positions of a unit are contiguous and
// aligned in dy / x.
//
// dw is a sum over very many positions.  A single chain of additions per element lost bits that the kernel with 256 chains
// per element and a tree keeps (relative 2-norm error of 8 x 64 x 45 x 37 -> 96, 3x3, fp32: 2.3e-7 against 1.5e-7; in one
// part 1.4e-6), so chains are short here: 8 positions (bf16: 32) of a step, then into a sum over the steps, and (LONG, for few
// parts) 8 of those into a total: 1.1e-7, in one part 1.4e-7, for 43.5 -> 46.7 us.
template <typename T, int BT, int KS, int UPS>
struct GatherWgradTile {
    static constexpr int WT = BT / 32, NW = WT * WT * KS, NT = 64 * NW, NU = UPS * KS;
    static constexpr int STEP = NU * GElem<T>::U;                        // positions per step
    static constexpr int RPT = BT * NU / NT;                             // rows of an operand a thread brings per step
    static constexpr int PL = BT * 16 + 32, BUF = 2 * NU * PL;           // + 32: a 16-lane write hits all banks
    static constexpr int RED = KS > 1 ? NW * 16 * 64 * 4 : 0;
    static constexpr size_t LDS = 2 * BUF > RED ? 2 * BUF : RED;
    static_assert(RPT * NT == BT * NU && NT % NU == 0 && UPS % 2 == 0, "tile shape");
};

template <typename T, int BT, int KS, int UPS, bool DYV, bool XV, bool LONG>
__global__ __launch_bounds__(64 * (BT / 32) * (BT / 32) * KS) void gather_wgrad(const GatherWgradParams p)
{
    preload_kernargs(p);
    typedef GatherWgradTile<T, BT, KS, UPS> G;
    constexpr int U = GElem<T>::U, NU = G::NU, STEP = G::STEP, RPT = G::RPT, PL = G::PL, BUF = G::BUF, WT = G::WT, ROWS = G::NT / NU;
    constexpr unsigned SZ = sizeof(T);
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int kt = (int)blockIdx.y / p.ctiles, ct = (int)blockIdx.y - kt * p.ctiles;
    const int RS = p.R * p.S, CRS = p.C * RS;
    const unsigned mb = blockIdx.x * p.chunk;
    const unsigned me = mb + p.chunk < p.M ? mb + p.chunk : p.M;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)p.x, 0, (int)p.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_dy = __builtin_amdgcn_make_buffer_rsrc((void *)p.dy, 0, (int)p.dy_bytes, 0x00020000);

    // this thread: unit tid % NU of every step, RPT rows of both operands
    const int unit = tid % NU, row = tid / NU;
    int koff[RPT], xoff[RPT], xdh[RPT], xdw[RPT];                        // per row: channel offset; x: offset and tap shift
    bool kok[RPT], xok[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int k = kt * BT + row + ROWS * i, col = ct * BT + row + ROWS * i;
        kok[i] = k < p.K;
        koff[i] = p.dy_blocked ? (k >> 4) * p.dy_c + (k & 15) : k * p.dy_c;
        xok[i] = col < CRS;
        const int c = col / RS, t = col - c * RS;
        const int r = (int)(((float)t + 0.5f) * __builtin_amdgcn_rcpf((float)p.S));        // t < 31 * 31: exact, as in KWalk
        xdh[i] = r * p.dil_h;
        xdw[i] = (t - r * p.S) * p.dil_w;
        xoff[i] = (p.x_blocked ? (c >> 4) * p.x_c + (c & 15) : c * p.x_c) + (xdh[i] * p.W + xdw[i]) * p.x_px;
    }
    constexpr gf32x16 ZERO = {};
    constexpr int NCH = sizeof(T) == 4 ? 2 : 1;                          // chains of a step: 8 positions each (fp32), 32 (bf16)
    gf32x16 acc = ZERO, total = ZERO;
    uint32_t xr[RPT][U], kr[RPT][U];
    uint4 xv[RPT], kv[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        xv[i] = kv[i] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < U; ++e) xr[i][e] = kr[i][e] = 0;
    }

    auto request = [&](unsigned m1) {
        const unsigned m = m1 + unit * U;
        int n = (int)fd_div(m, p.div_pq);
        const int t = (int)(m - (unsigned)n * p.div_pq.d);
        int pp = (int)fd_div((unsigned)t, p.div_q), q = t - pp * p.Q;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            if constexpr (DYV) {
                const unsigned off = m < me && kok[i] ? (unsigned)(n * p.dy_n + t * p.dy_px + koff[i]) * SZ : GATHER_OOB;
                kv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_dy, (int)off, 0, 0));
            }
            if constexpr (XV) {
                const unsigned off = m < me && xok[i] ? (unsigned)(n * p.x_n + t * p.x_px + xoff[i]) * SZ : GATHER_OOB;
                xv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)off, 0, 0));
            }
        }
        if constexpr (!(DYV && XV)) {
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const bool in = m + e < me;
                if constexpr (!DYV) {
                    const int o = n * p.dy_n + (pp * p.Q + q) * p.dy_px;
#pragma unroll
                    for (int i = 0; i < RPT; ++i) kr[i][e] = GElem<T>::load(rs_dy, in && kok[i] ? (unsigned)(o + koff[i]) * SZ : GATHER_OOB);
                }
                if constexpr (!XV) {
                    const int ih = pp * p.sh - p.pb_h, iw = q * p.sw - p.pb_w;
                    const int o = n * p.x_n + (ih * p.W + iw) * p.x_px;
#pragma unroll
                    for (int i = 0; i < RPT; ++i) {
                        const bool ok = in && xok[i] && (unsigned)(ih + xdh[i]) < (unsigned)p.H && (unsigned)(iw + xdw[i]) < (unsigned)p.W;
                        xr[i][e] = GElem<T>::load(rs_x, ok ? (unsigned)(o + xoff[i]) * SZ : GATHER_OOB);
                    }
                }
                const bool wq = ++q == p.Q;
                q = wq ? 0 : q;
                pp += wq;
                const bool wp = pp == p.P;
                pp = wp ? 0 : pp;
                n += wp;
            }
        }
    };
    auto stage = [&](int buf) {
        unsigned char *ks = smem + buf * BUF, *xs = ks + NU * PL;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            if constexpr (!DYV) keep_raw(kr[i]);
            if constexpr (!XV) keep_raw(xr[i]);
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            *reinterpret_cast<uint4 *>(ks + unit * PL + (row + ROWS * i) * 16) = DYV ? kv[i] : GElem<T>::pack(kr[i]);
            *reinterpret_cast<uint4 *>(xs + unit * PL + (row + ROWS * i) * 16) = XV ? xv[i] : GElem<T>::pack(xr[i]);
        }
    };
    const int qk = wave % WT * 32, qx = wave / WT % WT * 32, slice = wave / (WT * WT);
    const int nsteps = (int)((me - mb + STEP - 1) / STEP);
    for (int s = -1; s < nsteps; ++s) {                                  // the first round only requests (see gather_conv)
        stage(s & 1);
        request(mb + (unsigned)(s + 1) * STEP);                          // past the end: every offset out of range
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier_nofence();
        const unsigned char *ks = smem + (s & 1) * BUF, *xs = ks + NU * PL;
        gf32x16 chain[2] = {ZERO, ZERO};
#pragma unroll
        for (int q = 0; q < UPS / 2; ++q) {
            const int pl = slice * UPS + 2 * q + half;
            chain[q % NCH] = mma_pair<T>(*reinterpret_cast<const uint4 *>(ks + pl * PL + (qk + l32) * 16),
                                       *reinterpret_cast<const uint4 *>(xs + pl * PL + (qx + l32) * 16), chain[q % NCH]);
        }
        acc += NCH > 1 ? chain[0] + chain[1] : chain[0];                 // carried into the next step: 16 registers and a workgroup less
        if (LONG && (s & 7) == 7) {
            total += acc;
            acc = ZERO;
        }
    }
    if (LONG) acc += total;
    if constexpr (KS > 1) {                                              // slice z adds up the groups (4 rows) z, z + KS, ... over all slices
        wg_barrier_nofence();
        float *red = reinterpret_cast<float *>(smem);
#pragma unroll
        for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[v];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        wg_barrier_nofence();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (g % KS != slice) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float t = 0.f;
#pragma unroll
                for (int z = 0; z < KS; ++z) t += red[((wave % (WT * WT) + z * WT * WT) * 16 + g * 4 + e) * 64 + lane];
                acc[g * 4 + e] = t;
            }
        }
    }
    const int col = ct * BT + qx + l32;
    if (col >= CRS) return;
    if constexpr (!XV) {
        // Positions whose tap lies in the padding are no part of the sum: see gather_conv
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(any_nan(acc)) != 0, 0)) {
            const int c = col / RS, t = col - c * RS, r = t / p.S, s = t - r * p.S;
            const int dh = r * p.dil_h - p.pb_h, dw = s * p.dil_w - p.pb_w;
            if (dh < 0 || dw < 0 || (p.P - 1) * p.sh + dh >= p.H || (p.Q - 1) * p.sw + dw >= p.W) {
                const int chan = p.x_blocked ? (c >> 4) * p.x_c + (c & 15) : c * p.x_c;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int k = kt * BT + qk + 8 * g + 4 * half;
                    float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
                    for (unsigned m = mb; m < me; ++m) {
                        const int n = (int)fd_div(m, p.div_pq);
                        const int pq = (int)(m - (unsigned)n * p.div_pq.d), pp = (int)fd_div((unsigned)pq, p.div_q);
                        const int ih = pp * p.sh + dh, iw = (pq - pp * p.Q) * p.sw + dw;
                        if ((unsigned)ih >= (unsigned)p.H || (unsigned)iw >= (unsigned)p.W) continue;
                        const float x = load_value<T>(rs_x, (unsigned)(n * p.x_n + chan + (ih * p.W + iw) * p.x_px) * SZ);
                        const int o = n * p.dy_n + pq * p.dy_px + (p.dy_blocked ? (k >> 4) * p.dy_c + (k & 15) : k * p.dy_c);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sum[e] = fmaf(load_value<T>(rs_dy, k + e < p.K ? (unsigned)(o + e * (p.dy_blocked ? 1 : p.dy_c)) * SZ : GATHER_OOB), x, sum[e]);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[4 * g + e] = acc[4 * g + e] != acc[4 * g + e] ? sum[e] : acc[4 * g + e];
                }
            }
        }
    }
    float *out = p.out + (size_t)blockIdx.x * p.pitch;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int k = kt * BT + qk + 8 * (v >> 2) + 4 * half + (v & 3);
        if ((KS == 1 || (v >> 2) % KS == slice) && k < p.K) out[(size_t)k * CRS + col] = acc[v];
    }
}

// ---------------------------------------------------------------------------------------------- host side

static int gcd_(int a, int b) { return b ? gcd_(b, a % b) : a; }

// what the kernels address: 32-bit byte offsets into every operand, window rows / columns in 31-bit masks, the residue
// classes of backprop-data in a table; what a grid holds: 2^32 - 1 threads (8 a position in the tiles that take most) and
// 65535 tiles of channels
bool gather_takes(const ngc_conv_desc &d, int op, int P, int Q)
{
    const char *force = env_switch(SW_GATHER_TILE);                       // tests only: 0 = never
    if (force && atoi(force) == 0) return false;
    const size_t sz = d.dtype == NGC_F32 ? 4 : 2, lim = (size_t)1 << 31;
    auto bytes = [&](int layout, size_t n, size_t c, size_t hw) { return n * (layout == NGC_NCHW ? c : (c + 15) / 16 * 16) * hw * sz; };
    if (d.r > 31 || d.s > 31 || bytes(d.x_layout, d.n, d.c, (size_t)d.h * d.w) >= lim || bytes(d.y_layout, d.n, d.k, (size_t)P * Q) >= lim ||
        (size_t)d.k * d.c * d.r * d.s * sz >= lim)
        return false;
    const size_t positions = op == NGC_OP_FWD ? (size_t)d.n * P * Q : (size_t)d.n * d.h * d.w;
    if (op != NGC_OP_BWD_FILTERS && (positions + 64 > (size_t)1 << 29 || ((op == NGC_OP_FWD ? d.k : d.c) + 31) / 32 > 65535)) return false;
    if (op == NGC_OP_BWD_DATA) return d.stride_h <= GATHER_CLASSES && d.stride_w <= GATHER_CLASSES;
    return op == NGC_OP_FWD || (size_t)((d.k + 63) / 64) * (((size_t)d.c * d.r * d.s + 63) / 64) <= 65535;
}

template <typename T, int BM, int BN, int WM, int WN, int KS, int UPS, bool WV>
static hipError_t launch_gather_conv_l(const GatherConvParams &p, dim3 grid, hipStream_t st)
{
    static LdsLimitOnce lds_limit;
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&gather_conv<T, BM, BN, WM, WN, KS, UPS, WV>));
    if (e != hipSuccess) return e;
    typedef GatherTile<T, BM, BN, WM, WN, KS, UPS> G;
    NGC_LAUNCH((gather_conv<T, BM, BN, WM, WN, KS, UPS, WV>), grid, dim3(G::NT), G::LDS, st, p);
    return launch_result();
}

template <typename T, int BM, int BN, int WM, int WN, int KS, int UPS>
static hipError_t launch_gather_conv_w(const GatherConvParams &p, unsigned max_m, int classes, bool wvec, hipStream_t st)
{
    const dim3 grid((max_m + BN - 1) / BN, (p.Cout + BM - 1) / BM, classes);
    return wvec ? launch_gather_conv_l<T, BM, BN, WM, WN, KS, UPS, true>(p, grid, st) : launch_gather_conv_l<T, BM, BN, WM, WN, KS, UPS, false>(p, grid, st);
}

// Tile of a launch: 1 = 64 x 64, four waves; 2 = 64 x 64, two slices of the reduction; 3 = 32 x 32, four slices.  A step
// takes about 0.45 us of latency whatever the tile; on a chip with work for every unit a 64 x 64 step costs a compute unit
// 0.5 us (two slices: 0.95 us for twice the indices), a 32 x 32 step 0.35 us for half as many indices and a quarter of the
// tile.  The larger of the two times the steps is within 15 % of the measured times of some forty nodes of 0.2 to 40 us; the
// smallest estimate is taken.
struct GatherLoad {
    int s4, s8;                    // steps of 4 and of 8 units
    double t64, t32;               // tiles per compute unit
};

static GatherLoad gather_load(const GatherConvParams &p, int U, unsigned max_m, int classes)
{
    int taps = 0;
    for (int a = 0; a < p.os_h; ++a)
        for (int b = 0; b < p.os_w; ++b) taps = p.nr[a] * p.ns[b] > taps ? p.nr[a] * p.ns[b] : taps;
    const int kred = taps * p.Cin;
    return {(kred + 4 * U - 1) / (4 * U), (kred + 8 * U - 1) / (8 * U), (double)((max_m + 63) / 64) * ((p.Cout + 63) / 64) * classes / 256,
            (double)((max_m + 31) / 32) * ((p.Cout + 31) / 32) * classes / 256};
}

static int gather_tile(const GatherLoad &l)
{
    const char *force = env_switch(SW_GATHER_TILE);                       // tests / experiments only
    if (force && atoi(force) >= 1 && atoi(force) <= 3) return atoi(force);
    auto larger = [](double x, double y) { return x > y ? x : y; };
    const double e1 = l.s4 * larger(0.45, 0.5 * l.t64), e2 = l.s8 * larger(0.5, 0.95 * l.t64) + 0.8, e3 = l.s8 * larger(0.45, 0.35 * l.t32) + 0.8;
    return e1 <= e2 && e1 <= e3 ? 1 : e2 < e3 ? 2 : 3;
}

// Expected time, us, of fp32 backprop-data with stride 1, to choose between this kernel and conv_stream.hip: a start and, per
// step, latency and rounds of workgroups.  Fitted to 1057 launches of the tile chosen above, four fifths of them within 12 %.
double gather_f32_bwd_us(const GatherConvParams &p, unsigned max_m)
{
    const GatherLoad l = gather_load(p, 4, max_m, 1);
    const double r64 = ceil(l.t64), r32 = ceil(l.t32);
    switch (gather_tile(l)) {
    case 1: return 4.75 + l.s4 * (0.179 + 0.412 * r64);
    case 2: return 5.61 + l.s8 * (0.165 + 0.687 * r64);
    default: return 4.33 + l.s8 * (0.242 + 0.224 * r32);
    }
}

template <typename T>
static hipError_t launch_gather_conv_t(const GatherConvParams &p, unsigned max_m, int classes, bool wvec, hipStream_t st)
{
    switch (gather_tile(gather_load(p, GElem<T>::U, max_m, classes))) {
    case 1: return launch_gather_conv_w<T, 64, 64, 2, 2, 1, 4>(p, max_m, classes, wvec, st);
    case 2: return launch_gather_conv_w<T, 64, 64, 2, 2, 2, 4>(p, max_m, classes, wvec, st);
    default: return launch_gather_conv_w<T, 32, 32, 1, 1, 4, 2>(p, max_m, classes, wvec, st);
    }
}

static void lattice_divisions(GatherConvParams *p)
{
    const int last_h = p->os_h - 1, last_w = p->os_w - 1;                // the extents of the classes: that of class 0 or one less
    const int oph[2] = {p->oph[0], p->oph[last_h]}, opw[2] = {p->opw[0], p->opw[last_w]};
    for (int i = 0; i < 4; ++i) p->div_pq[i] = make_fastdiv((uint32_t)(oph[i >> 1] * opw[i & 1] > 0 ? oph[i >> 1] * opw[i & 1] : 1));
    for (int i = 0; i < 2; ++i) p->div_q[i] = make_fastdiv((uint32_t)(opw[i] > 0 ? opw[i] : 1));
}

static hipError_t launch_gather_conv(const GatherConvParams &p, int dtype, hipStream_t st)
{
    const unsigned max_m = (unsigned)p.N * p.oph[0] * p.opw[0];
    const int classes = p.os_h * p.os_w;
    const StreamChoice c = stream_conv_choice(p, dtype, max_m, classes);
    if (c.take) return launch_stream_conv(p, dtype, max_m, classes, c, st);
    return dtype == NGC_F32 ? launch_gather_conv_t<float>(p, max_m, classes, p.wvec, st) : launch_gather_conv_t<uint16_t>(p, max_m, classes, p.wvec, st);
}

// the classes of one axis of backprop-data: output pixels congruent to a modulo the stride meet the taps r with
// (a + pad - r * dil) divisible by the stride, every rst-th one from the first
static void gather_axis(int extent, int stride, int dil, int pad, int taps, int32_t *rst, int32_t *step, int32_t *r0, int32_t *n, int32_t *base, int32_t *op)
{
    *rst = stride / gcd_(stride, dil);
    *step = -(*rst * dil / stride);
    for (int a = 0; a < stride; ++a) {
        int r = 0;
        while (r < *rst && r < taps && (a + pad - r * dil) % stride != 0) ++r;
        const bool any = r < *rst && r < taps;
        r0[a] = any ? r : 0;
        n[a] = any ? (taps - 1 - r) / *rst + 1 : 0;
        base[a] = any ? (a + pad - r * dil) / stride : 0;                // exact
        op[a] = a < extent ? (extent - a + stride - 1) / stride : 0;
    }
}

// the arguments of a node but its tensors
static GatherConvParams fwd_params(const ngc_conv_desc &d, int P, int Q)
{
    const size_t sz = d.dtype == NGC_F32 ? 4 : 2;
    GatherConvParams p = {};
    p.N = d.n; p.Cin = d.c; p.Cout = d.k; p.Hin = d.h; p.Win = d.w; p.Hout = P; p.Wout = Q;
    gather_strides(d.x_layout, d.c, d.h * d.w, &p.in_n, &p.in_c, &p.in_px);
    p.in_bytes = (uint32_t)((size_t)d.n * p.in_n * sz);
    p.wt_bytes = (uint32_t)((size_t)d.k * d.c * d.r * d.s * sz);
    p.in_blocked = d.x_layout == NGC_NCHW16C; p.out_blocked = d.y_layout == NGC_NCHW16C;
    p.w_row = d.c * d.r * d.s; p.w_chan = d.r * d.s; p.S = d.s;
    p.is_h = d.stride_h; p.is_w = d.stride_w; p.os_h = p.os_w = 1;
    p.rst_h = p.rst_w = 1; p.step_h = d.dil_h; p.step_w = d.dil_w;
    p.nr[0] = d.r; p.ns[0] = d.s; p.base_h[0] = -d.pad_below_h; p.base_w[0] = -d.pad_below_w; p.oph[0] = P; p.opw[0] = Q;
    p.relu = (d.epilogue & NGC_EPI_RELU) ? 1 : 0;
    p.wvec = p.w_row % (int)(16 / sz) == 0;
    lattice_divisions(&p);
    return p;
}

static GatherConvParams bwd_data_params(const ngc_conv_desc &d, int P, int Q)
{
    const size_t sz = d.dtype == NGC_F32 ? 4 : 2;
    GatherConvParams p = {};
    p.N = d.n; p.Cin = d.k; p.Cout = d.c; p.Hin = P; p.Win = Q; p.Hout = d.h; p.Wout = d.w;
    gather_strides(d.y_layout, d.k, P * Q, &p.in_n, &p.in_c, &p.in_px);
    p.in_bytes = (uint32_t)((size_t)d.n * p.in_n * sz);
    p.wt_bytes = (uint32_t)((size_t)d.k * d.c * d.r * d.s * sz);
    p.in_blocked = d.y_layout == NGC_NCHW16C; p.out_blocked = d.x_layout == NGC_NCHW16C;
    p.w_row = d.r * d.s; p.w_chan = d.c * d.r * d.s; p.S = d.s;
    p.is_h = p.is_w = 1; p.os_h = d.stride_h; p.os_w = d.stride_w;
    gather_axis(d.h, d.stride_h, d.dil_h, d.pad_below_h, d.r, &p.rst_h, &p.step_h, p.r0, p.nr, p.base_h, p.oph);
    gather_axis(d.w, d.stride_w, d.dil_w, d.pad_below_w, d.s, &p.rst_w, &p.step_w, p.s0, p.ns, p.base_w, p.opw);
    lattice_divisions(&p);
    return p;
}

hipError_t launch_gather_fwd(const ngc_conv_desc &d, int P, int Q, const void *x, const void *w, const float *bias, void *y, hipStream_t st)
{
    GatherConvParams p = fwd_params(d, P, Q);
    p.in = x; p.wt = w; p.out = y; p.bias = bias;
    return launch_gather_conv(p, d.dtype, st);
}

hipError_t launch_gather_bwd_data(const ngc_conv_desc &d, int P, int Q, const void *dy, const void *w, const void *mask, void *dx, hipStream_t st)
{
    GatherConvParams p = bwd_data_params(d, P, Q);
    p.in = dy; p.wt = w; p.out = dx; p.mask = mask;
    return launch_gather_conv(p, d.dtype, st);
}

bool gather_streams(const ngc_conv_desc &d, int op, int P, int Q)
{
    if (op == NGC_OP_BWD_FILTERS) {
        bool takes;
        wgrad_stream_workspace(d, P, Q, &takes);
        return takes;
    }
    const GatherConvParams p = op == NGC_OP_FWD ? fwd_params(d, P, Q) : bwd_data_params(d, P, Q);
    return stream_conv_choice(p, d.dtype, (unsigned)p.N * p.oph[0] * p.opw[0], p.os_h * p.os_w).take;
}

// How backprop-filters runs: the tile (1 = 64 x 64, two slices; 2 = 32 x 32, eight slices; 3 = 32 x 32, four slices) and the
// parts the positions are cut into.  Up to two or three steps of the eight-slice kernel: one part, a second launch costs more
// than it saves.  Else enough parts to give the chip three workgroups per compute unit (eight of the small ones), of at
// least two steps each, at most 16 MB of partial sums.  The small tile is for fp32 results that would leave half of a large
// one empty: 31 x 119 x 10 x 50, K = 11, 3x3 35 us against 45 us (bf16, K = 17: 138 us against 69 us).
struct GatherWgradPlan {
    int tile, parts;
};

static GatherWgradPlan wgrad_plan(const ngc_conv_desc &d, int P, int Q)
{
    const size_t M = (size_t)d.n * P * Q, crs = (size_t)d.c * d.r * d.s, U = d.dtype == NGC_F32 ? 4 : 8;
    auto tiles = [&](size_t t) { return ((size_t)d.k + t - 1) / t * ((crs + t - 1) / t); };
    const char *force = env_switch(SW_GATHER_WGRAD);                     // tests / experiments only: tile * 1000 + parts
    if (force && atoi(force) >= 1000) return {atoi(force) / 1000, atoi(force) % 1000 > 0 ? atoi(force) % 1000 : 1};
    const bool small = d.dtype == NGC_F32 && (d.k <= 32 || crs <= 32) && tiles(32) <= 65535;
    if (M <= (d.dtype == NGC_F32 ? 384 : 512) && tiles(32) <= 65535) return {2, 1};
    size_t parts = small ? (2048 + tiles(32) - 1) / tiles(32) : (768 + tiles(64) - 1) / tiles(64);
    const size_t most = M / ((small ? 2 * 16 : 2 * 8) * U), cap = ((size_t)16 << 20) / ((d.k * crs + 15) / 16 * 64);
    if (parts > most) parts = most;
    if (parts > cap) parts = cap;
    if (parts > 256) parts = 256;
    return {small ? 3 : 1, parts < 1 ? 1 : (int)parts};
}

static uint32_t wgrad_pitch(const ngc_conv_desc &d) { return (uint32_t)(((size_t)d.k * d.c * d.r * d.s + 15) / 16 * 16); }

size_t gather_wgrad_workspace(const ngc_conv_desc &d, int P, int Q)
{
    bool takes;
    const size_t b = wgrad_stream_workspace(d, P, Q, &takes);
    if (takes) return b;
    const int parts = wgrad_plan(d, P, Q).parts;
    return parts > 1 ? (size_t)parts * wgrad_pitch(d) * sizeof(float) : 0;
}

template <typename T, int BT, int KS, int UPS, bool DYV, bool XV, bool LONG>
static hipError_t launch_gather_wgrad_l(const GatherWgradParams &p, dim3 grid, hipStream_t st)
{
    static LdsLimitOnce lds_limit;
    const hipError_t e = lds_limit.raise(reinterpret_cast<const void *>(&gather_wgrad<T, BT, KS, UPS, DYV, XV, LONG>));
    if (e != hipSuccess) return e;
    typedef GatherWgradTile<T, BT, KS, UPS> G;
    NGC_LAUNCH((gather_wgrad<T, BT, KS, UPS, DYV, XV, LONG>), grid, dim3(G::NT), G::LDS, st, p);
    return launch_result();
}

template <typename T, int BT, int KS, int UPS, bool LONG>
static hipError_t launch_gather_wgrad_t(GatherWgradParams &p, int parts, bool dyvec, bool xvec, hipStream_t st)
{
    constexpr uint32_t step = GatherWgradTile<T, BT, KS, UPS>::STEP;
    p.chunk = ((p.M + parts - 1) / parts + step - 1) / step * step;
    p.ctiles = (p.C * p.R * p.S + BT - 1) / BT;
    const dim3 grid((p.M + p.chunk - 1) / p.chunk, (unsigned)((p.K + BT - 1) / BT) * p.ctiles);
    if (dyvec) return xvec ? launch_gather_wgrad_l<T, BT, KS, UPS, true, true, LONG>(p, grid, st) : launch_gather_wgrad_l<T, BT, KS, UPS, true, false, LONG>(p, grid, st);
    return launch_gather_wgrad_l<T, BT, KS, UPS, false, false, LONG>(p, grid, st);  // x is only contiguous where dy is
}

template <typename T>
static hipError_t launch_gather_wgrad(GatherWgradParams &p, int v, int parts, bool dyvec, bool xvec, hipStream_t st)
{
    // The sum over the steps is as long as a chain of 256 per element from 8 parts on (32 positions a step in two slices),
    // from 4 on in the small tile (64 in four).
    switch (v) {
    case 1:
        return parts < 8 ? launch_gather_wgrad_t<T, 64, 2, 4, true>(p, parts, dyvec, xvec, st) : launch_gather_wgrad_t<T, 64, 2, 4, false>(p, parts, dyvec, xvec, st);
    case 2: return launch_gather_wgrad_t<T, 32, 8, 4, false>(p, parts, dyvec, xvec, st);      // at most 512 positions
    default:
        return parts < 4 ? launch_gather_wgrad_t<T, 32, 4, 4, true>(p, parts, dyvec, xvec, st) : launch_gather_wgrad_t<T, 32, 4, 4, false>(p, parts, dyvec, xvec, st);
    }
}

// A node whose reduction is split, called without the workspace for it: one part of the gather GEMM takes some 1.05 us per
// step and round of tiles, the kernel with a workgroup per element of dw about 1 us per 550 thousand products.  Measured,
// gather / direct, us: 8 x 64 x 45 x 37 -> 96 3x3 439 / 1091, 4 x 300 x 20 x 20 -> 300 3x3 60 / 2188; 32 x 3 x 64 x 64 -> 11 3x3
// 3039 / 247, 64 x 3 x 224 x 224 -> 32 3x3 94063 / 7660, 22 x 25 x 10 x 29 -> 68 3x3 215 / 153.
static bool one_part_is_slow(const ngc_conv_desc &d, size_t M)
{
    const size_t crs = (size_t)d.c * d.r * d.s, rounds = ((size_t)((d.k + 63) / 64) * ((crs + 63) / 64) + 255) / 256;
    const double gather = 1.05 * (double)((M + (d.dtype == NGC_F32 ? 31 : 63)) / (d.dtype == NGC_F32 ? 32 : 64)) * (double)rounds;
    return (double)d.k * (double)crs * (double)M / 550000.0 < gather;
}

hipError_t launch_gather_bwd_filters(const ngc_conv_desc &d, int P, int Q, const void *x, const void *dy, float *dw, void *ws, size_t ws_bytes,
                                     hipStream_t st)
{
    hipError_t se;
    if (launch_wgrad_stream(d, P, Q, x, dy, dw, ws, ws_bytes, st, &se)) return se;
    const size_t sz = d.dtype == NGC_F32 ? 4 : 2;
    const int U = (int)(16 / sz);
    GatherWgradParams p = {};
    p.M = (uint32_t)d.n * P * Q;
    p.pitch = wgrad_pitch(d);
    GatherWgradPlan plan = wgrad_plan(d, P, Q);
    if (plan.parts > 1 && (!ws || ws_bytes < (size_t)plan.parts * p.pitch * sizeof(float))) {
        if (one_part_is_slow(d, p.M)) return launch_direct_bwd_filters(d, P, Q, x, dy, dw, st);
        plan = {1, 1};
    }
    p.x = x; p.dy = dy;
    p.C = d.c; p.H = d.h; p.W = d.w; p.K = d.k; p.P = P; p.Q = Q; p.R = d.r; p.S = d.s;
    p.sh = d.stride_h; p.sw = d.stride_w; p.dil_h = d.dil_h; p.dil_w = d.dil_w; p.pb_h = d.pad_below_h; p.pb_w = d.pad_below_w;
    gather_strides(d.x_layout, d.c, d.h * d.w, &p.x_n, &p.x_c, &p.x_px);
    gather_strides(d.y_layout, d.k, P * Q, &p.dy_n, &p.dy_c, &p.dy_px);
    p.x_bytes = (uint32_t)((size_t)d.n * p.x_n * sz);
    p.dy_bytes = (uint32_t)((size_t)d.n * p.dy_n * sz);
    p.x_blocked = d.x_layout == NGC_NCHW16C; p.dy_blocked = d.y_layout == NGC_NCHW16C;
    p.div_pq = make_fastdiv((uint32_t)(P * Q));
    p.div_q = make_fastdiv((uint32_t)Q);
    const bool dyvec = !p.dy_blocked && (P * Q) % U == 0;
    const bool xvec = dyvec && !p.x_blocked && d.r == 1 && d.s == 1 && d.stride_h == 1 && d.stride_w == 1 && P == d.h && Q == d.w &&
                      d.pad_below_h == 0 && d.pad_below_w == 0;
    p.out = plan.parts > 1 ? static_cast<float *>(ws) : dw;
    const hipError_t e = d.dtype == NGC_F32 ? launch_gather_wgrad<float>(p, plan.tile, plan.parts, dyvec, xvec, st)
                                            : launch_gather_wgrad<uint16_t>(p, plan.tile, plan.parts, dyvec, xvec, st);
    if (e != hipSuccess || plan.parts == 1) return e;
    return launch_bias_grad_reduce(p.out, dw, (int)((p.M + p.chunk - 1) / p.chunk), d.k * d.c * d.r * d.s, (int)p.pitch, st);
}

}  // namespace ngc
