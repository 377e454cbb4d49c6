// Depthwise convolution (one R x S filter per channel) with the same fused epilogue as the
// GEMMs.  No matrix cores: per output there are only R*S multiply-accumulates against ~2
// bytes of traffic, so the layer is bound by memory, not arithmetic (the depthwise rows of
// the paper's Table 5).  Forward and input gradient are the same gather with the tap offsets
// mirrored; the weight gradient reduces over all pixels per (tap, channel).
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

struct DwArgs {
    const int8_t *A, *Wt;
    const int32_t *wsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, C;                      // output pixels, channels
    int R, S, Hs, Ws, Ho, Wo, stride, pad, dgrad;
    int sr_on;                     // 1: stochastic rounding with the seed below
    HqSr sr;
};

__device__ inline int sbyte(int v, int k) { return (v << (24 - 8 * k)) >> 24; }

// One thread: one output pixel, four consecutive channels (one 32-bit word of codes).
__global__ __launch_bounds__(HQ_THREADS) void hq_depthwise_kernel(const DwArgs a)
{
    __shared__ int red[4 * (HQ_THREADS / 64)];
    const int c4n = a.C >> 2;
    const size_t total = (size_t)a.M * c4n;
    const int za = a.aq->zero_point;
    const int fill = (int)((unsigned)(za & 0xff) * 0x01010101u);   // unsigned: the product may set bit 31
    const bool fused = a.out32 == nullptr;
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqRequant rq = {1.0f, 0.0f, 0.0f, 0};
    if (fused) rq = hq_make_requant(acc_scale, a.range->qp, a.range->qlo, a.range->qhi);
    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;

    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(idx % c4n) * 4;
        const int m = (int)(idx / c4n);
        const int x = m % a.Wo, y = (m / a.Wo) % a.Ho, b = m / (a.Wo * a.Ho);
        const int8_t *img = a.A + (size_t)b * a.Hs * a.Ws * a.C;
        const int y0 = a.dgrad ? y + a.pad : y * a.stride - a.pad;
        const int x0 = a.dgrad ? x + a.pad : x * a.stride - a.pad;
        int acc[4] = {0, 0, 0, 0};
        for (int r = 0; r < a.R; r++) {
            for (int s = 0; s < a.S; s++) {
                int iy, ix; bool ok = true;
                if (!a.dgrad) { iy = y0 + r; ix = x0 + s; }
                else {
                    iy = y0 - r; ix = x0 - s;
                    if (a.stride != 1) {
                        ok = iy >= 0 && ix >= 0 && (iy % a.stride == 0) && (ix % a.stride == 0);
                        iy /= a.stride; ix /= a.stride;
                    }
                }
                ok = ok && iy >= 0 && iy < a.Hs && ix >= 0 && ix < a.Ws;
                const int xv = ok ? *reinterpret_cast<const int *>(img + ((size_t)iy * a.Ws + ix) * a.C + c) : fill;
                const int wv = *reinterpret_cast<const int *>(a.Wt + (size_t)(r * a.S + s) * a.C + c);
#pragma unroll
                for (int e = 0; e < 4; e++) acc[e] += sbyte(xv, e) * sbyte(wv, e);
            }
        }
        const v4i ws = *reinterpret_cast<const v4i *>(a.wsum + c);
        int q[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int cv = acc[e] - za * ws[e];
            mn = min(mn, cv); mx = max(mx, cv);
            q[e] = cv;
        }
        if (fused) {
#pragma unroll
            for (int e = 0; e < 4; e++)
                q[e] = a.sr_on ? hq_requant_sr(q[e], rq, a.sr, (size_t)m * a.C + c + e, nlo, nhi) : hq_requant(q[e], rq, nlo, nhi);
            *reinterpret_cast<unsigned *>(a.out8 + (size_t)m * a.C + c) = hq_pack4(q[0], q[1], q[2], q[3]);
        } else {
            v4i v = {q[0], q[1], q[2], q[3]};
            *reinterpret_cast<v4i *>(a.out32 + (size_t)m * a.C + c) = v;
        }
    }
    hq_block_stats_commit(mn, mx, nlo, nhi, a.st, red, blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.C);
        if (fused) *a.outq = a.range->qp;
    }
}

// ---------------------------------------------------------------------------------------
// 3x3 with padding 1 and stride 1 or 2: the depthwise layers of MobileNetV2-style blocks (Table 5, DW rows).
//
// What bounds these kernels is the vector ALU: 19.5 instructions per output, whose issue takes 86 % of the 44 us of 128 x 56 x 56 x
// 192 (30 us of memory traffic; the earlier stride-1 kernel, one column per thread, had 26 and took 71 us), 65 % of the time with
// stride 2 (18 us instead of 67) and 91 % in its input gradient (25 instead of 239).  Hence few instructions per output.  A
// thread owns four channels (one word) of two neighbouring output columns and slides down a strip of rows.  Pixels come as packed words of four channels; the words of four adjacent columns are byte-transposed (8
// v_perm_b32) into one word per channel, and a filter row on it is one 4-way byte dot product per output: the second column's
// weights are the first's shifted by one byte.  Rows are addressed by a uniform pointer plus a fixed lane offset, so loads cost
// no address arithmetic, and the fill of columns outside the image is one select per word.  Lanes run along (column,
// channel) of a row, which is how NHWC lies in memory.
// ---------------------------------------------------------------------------------------
struct Dw3Args {
    const int8_t *A, *Wt;
    const int32_t *wsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int B, H, W, OH, OW, C;        // H x W: image A for the stencil, dX for the strided input gradient; OH x OW: the other one
    int rows_per_strip, flip;
    HqSr sr;                       // MODE 2
};

// four words = four pixels of four channels -> t[e] = (pixel0[e], pixel1[e], pixel2[e], pixel3[e])
__device__ inline void dw_transpose4(int a0, int a1, int a2, int a3, int *t)
{
    // v_perm_b32: selector bytes 0..3 pick bytes of the second source, 4..7 of the first, 0x0c is zero
    const unsigned p0 = __builtin_amdgcn_perm((unsigned)a1, (unsigned)a0, 0x05010400u);   // (a0.0, a1.0, a0.1, a1.1)
    const unsigned p1 = __builtin_amdgcn_perm((unsigned)a1, (unsigned)a0, 0x07030602u);   // (a0.2, a1.2, a0.3, a1.3)
    const unsigned q0 = __builtin_amdgcn_perm((unsigned)a3, (unsigned)a2, 0x05010400u);
    const unsigned q1 = __builtin_amdgcn_perm((unsigned)a3, (unsigned)a2, 0x07030602u);
    t[0] = (int)__builtin_amdgcn_perm(q0, p0, 0x05040100u);
    t[1] = (int)__builtin_amdgcn_perm(q0, p0, 0x07060302u);
    t[2] = (int)__builtin_amdgcn_perm(q1, p1, 0x05040100u);
    t[3] = (int)__builtin_amdgcn_perm(q1, p1, 0x07060302u);
}

// Word e of the transposed four pixels moved one pixel on: (t.1, t.2, t.3, next[e]); and one back: (prev[e], t.0, t.1, t.2).
template <int E> __device__ inline int dw_shift_in(int t, int next)
{
    return (int)__builtin_amdgcn_perm((unsigned)next, (unsigned)t, 0x00030201u | ((4u + E) << 24));
}
template <int E> __device__ inline int dw_shift_back(int t, int prev)
{
    return (int)__builtin_amdgcn_perm((unsigned)t, (unsigned)prev, 0x06050400u | (unsigned)E);
}

// A word at a uniform address plus a lane's offset.  The statement keeps the widening of the offset next to the access, where it
// is part of the instruction; hoisted out of the row loop it would cost a 64-bit addition per word and row.
__device__ inline int dw_load(const int8_t *p, unsigned off)
{
    asm volatile("" : "+v"(off));
    return *reinterpret_cast<const int *>(p + off);
}
__device__ inline void dw_store(int8_t *p, unsigned off, int v)
{
    asm volatile("" : "+v"(off));
    *reinterpret_cast<int *>(p + off) = v;
}

// Epilogue of two neighbouring pixels' four channels each (`both`: the second exists; `pair`: it exists in every lane).
// Stores through a uniform base and lane offsets.
template <int MODE, bool FULL>
__device__ inline void dw_emit(const Dw3Args &a, const HqEpilogue &ep, int (&cv)[8], size_t base, unsigned off0, unsigned off1,
                               bool pair, bool both, int &mn, int &mx, unsigned &nlo, unsigned &nhi)
{
    if constexpr (MODE == 0) {
        int32_t *o = a.out32 + base;
        hq_minmax_group<4>(cv, mn, mx);
        *reinterpret_cast<v4i *>(o + off0) = v4i{cv[0], cv[1], cv[2], cv[3]};
        if (both) {
            hq_minmax_group<4>(cv + 4, mn, mx);
            *reinterpret_cast<v4i *>(o + off1) = v4i{cv[4], cv[5], cv[6], cv[7]};
        }
    } else {
        int8_t *o = a.out8 + base;
        int w[2];
        if constexpr (MODE == 2) {
            hq_requant_group_sr<4, FULL>(cv, ep, a.sr, base + off0, mn, mx, nlo, nhi, w);
            dw_store(o, off0, w[0]);
            if (both) {
                hq_requant_group_sr<4, FULL>(cv + 4, ep, a.sr, base + off1, mn, mx, nlo, nhi, w + 1);
                dw_store(o, off1, w[1]);
            }
        } else if (pair) {
            hq_requant_group<8, FULL>(cv, ep, mn, mx, nlo, nhi, w);
            dw_store(o, off0, w[0]);
            dw_store(o, off1, w[1]);
        } else {
            hq_requant_group<4, FULL>(cv, ep, mn, mx, nlo, nhi, w);
            dw_store(o, off0, w[0]);
            if (both) {
                hq_requant_group<4, FULL>(cv + 4, ep, mn, mx, nlo, nhi, w + 1);
                dw_store(o, off1, w[1]);
            }
        }
    }
}

template <int N> using dw_int = std::integral_constant<int, N>;

// Forward, and with stride 1 the input gradient as the same stencil with mirrored taps.
template <int STRIDE, int MODE>
__global__ __launch_bounds__(HQ_THREADS) void hq_dw3x3_kernel(const Dw3Args a)
{
    constexpr int NW = STRIDE == 1 ? 4 : 5;                          // input columns of the two outputs
    constexpr int NT = STRIDE;                                       // transposed words per channel and row
    constexpr int NR = STRIDE;                                       // new input rows per output row
    constexpr int RING = STRIDE == 1 ? 3 : 2;                        // output rows whose input is under way
    __shared__ int red[4 * (HQ_THREADS / 64)];
    const int c4n = a.C >> 2, cols2 = (a.OW + 1) >> 1;
    const unsigned q = blockIdx.x * HQ_THREADS + threadIdx.x;        // (image, column pair, word)
    const bool live = q < (unsigned)a.B * cols2 * c4n;
    const unsigned qx = (live ? q : 0) / c4n, b = qx / cols2;
    const int x = 2 * (int)(qx - b * cols2), c = (int)((live ? q : 0) - qx * c4n) * 4;
    const int y0 = blockIdx.y * a.rows_per_strip, y1 = min(a.OH, y0 + a.rows_per_strip);
    const size_t rowbytes = (size_t)a.W * a.C, orow = (size_t)a.OW * a.C;
    // (tensors have fewer than 2^32 elements)
    const unsigned ibase = b * (unsigned)a.H * (unsigned)rowbytes + (unsigned)c, obase = b * (unsigned)a.OH * (unsigned)orow + (unsigned)c;

    const int za = a.aq->zero_point;
    const int fill = (int)((unsigned)(za & 0xff) * 0x01010101u);     // unsigned: the product may set bit 31
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);

    // weights: per filter row and channel one word (w[r][0], w[r][1], w[r][2], 0), mirrored for the input gradient
    int wt[3][4];
#pragma unroll
    for (int r = 0; r < 3; r++) {
        int pk[3];
#pragma unroll
        for (int sx = 0; sx < 3; sx++) {
            const int t = r * 3 + sx, ts = a.flip ? 8 - t : t;
            pk[sx] = *reinterpret_cast<const int *>(a.Wt + (size_t)ts * a.C + c);
        }
        dw_transpose4(pk[0], pk[1], pk[2], 0, wt[r]);
    }
    const v4i wsv = *reinterpret_cast<const v4i *>(a.wsum + c);
    int nz[4];
#pragma unroll
    for (int e = 0; e < 4; e++) nz[e] = -(za * wsv[e]);

    unsigned off[NW];
    bool ok[NW];
#pragma unroll
    for (int k = 0; k < NW; k++) {
        const int xi = STRIDE * x - 1 + k;
        ok[k] = xi >= 0 && xi < a.W;
        off[k] = ibase + (unsigned)(ok[k] ? xi : STRIDE * x) * (unsigned)a.C;
    }
    const bool both = x + 1 < a.OW, pair = (a.OW & 1) == 0;
    const unsigned off0 = obase + (unsigned)x * (unsigned)a.C, off1 = off0 + (unsigned)a.C;

    auto load_row = [&](int y, int (&raw)[NW]) {                     // y is the same for the whole workgroup
        if (y >= 0 && y < a.H) {
            const int8_t *p = a.A + (size_t)y * rowbytes;
#pragma unroll
            for (int k = 0; k < NW; k++) raw[k] = dw_load(p, off[k]);
        } else {
#pragma unroll
            for (int k = 0; k < NW; k++) raw[k] = fill;
        }
    };
    auto transpose = [&](int (&raw)[NW], int (&t)[NT][4]) {
#pragma unroll
        for (int k = 0; k < NW; k++)
            if (k != 1) raw[k] = ok[k] ? raw[k] : fill;
        dw_transpose4(raw[0], raw[1], raw[2], raw[3], t[0]);
        if constexpr (STRIDE == 2)                                   // columns 2x+1, 2x+2, 2x+3
            dw_transpose4(raw[2], raw[3], raw[4], 0, t[1]);
    };

    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    int win[3][NT][4], ring[RING][NR][NW];
    auto run = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        {
            int tmp[NW];
            load_row(STRIDE * y0 - 1, tmp);
            int tmp1[NW];
            if constexpr (STRIDE == 1) load_row(y0, tmp1);
#pragma unroll
            for (int k = 0; k < RING; k++)
#pragma unroll
                for (int r = 0; r < NR; r++) load_row(STRIDE == 1 ? y0 + 1 + k : 2 * (y0 + k) + r, ring[k][r]);
            transpose(tmp, win[0]);
            if constexpr (STRIDE == 1) transpose(tmp1, win[1]);
        }
        int oy = y0;
        // window slots of the filter's rows rotate with the output row: by one of three, or (stride 2) by swapping two
        auto step = [&](auto phase) {
            constexpr int P = decltype(phase)::value;
            constexpr int TOP = STRIDE == 1 ? P : 2 * P, MID = STRIDE == 1 ? (P + 1) % 3 : 1, BOT = STRIDE == 1 ? (P + 2) % 3 : 2 - 2 * P;
            if constexpr (STRIDE == 1) {
                transpose(ring[P][0], win[BOT]);
            } else {
                transpose(ring[P][0], win[MID]);
                transpose(ring[P][1], win[BOT]);
            }
            if (oy + RING < y1)
#pragma unroll
                for (int r = 0; r < NR; r++) load_row(STRIDE == 1 ? oy + RING + 1 : 2 * (oy + RING) + r, ring[P][r]);
            int cv[8];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                int p = __builtin_amdgcn_sdot4(win[TOP][0][e], wt[0][e], nz[e], false);
                p = __builtin_amdgcn_sdot4(win[MID][0][e], wt[1][e], p, false);
                cv[e] = __builtin_amdgcn_sdot4(win[BOT][0][e], wt[2][e], p, false);
                p = __builtin_amdgcn_sdot4(win[TOP][NT - 1][e], STRIDE == 1 ? wt[0][e] << 8 : wt[0][e], nz[e], false);
                p = __builtin_amdgcn_sdot4(win[MID][NT - 1][e], STRIDE == 1 ? wt[1][e] << 8 : wt[1][e], p, false);
                cv[4 + e] = __builtin_amdgcn_sdot4(win[BOT][NT - 1][e], STRIDE == 1 ? wt[2][e] << 8 : wt[2][e], p, false);
            }
            dw_emit<MODE, FULL>(a, ep, cv, (size_t)oy * orow, off0, off1, pair, both, mn, mx, nlo, nhi);
            oy++;
        };
        while (true) {
            step(dw_int<0>());
            if (oy >= y1) break;
            step(dw_int<1>());
            if (oy >= y1) break;
            if constexpr (STRIDE == 1) {
                step(dw_int<2>());
                if (oy >= y1) break;
            }
        }
    };
    if (live) {
        if (MODE == 0 || ep.full_grid) run(std::true_type()); else run(std::false_type());
    }
    hq_block_stats_commit(mn, mx, nlo, nhi, a.st, red, blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.B * a.OH * a.OW * (unsigned long long)a.C);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

// Input gradient of the stride-2 layer.  dX pixel (2p + i, 2q + j) sees the taps r with (i + 1 - r) even: the block of 2 x 2
// pixels (p, q) depends on the gradient pixels (p, q), (p, q+1), (p+1, q), (p+1, q+1) alone, which are one transposed word per
// channel, so each of the four outputs is one dot product with a word of that parity's weights.
template <int MODE>
__global__ __launch_bounds__(HQ_THREADS) void hq_dw3x3_s2_dgrad_kernel(const Dw3Args a)
{
    constexpr int RING = 3;
    __shared__ int red[4 * (HQ_THREADS / 64)];
    const int c4n = a.C >> 2;
    const unsigned q = blockIdx.x * HQ_THREADS + threadIdx.x;        // (image, gradient column, word)
    const bool live = q < (unsigned)a.B * a.OW * c4n;
    const unsigned qx = (live ? q : 0) / c4n, b = qx / a.OW;
    const int x = (int)(qx - b * a.OW), c = (int)((live ? q : 0) - qx * c4n) * 4;
    const int y0 = blockIdx.y * a.rows_per_strip, y1 = min(a.OH, y0 + a.rows_per_strip);       // gradient rows
    const size_t grow = (size_t)a.OW * a.C, orow = (size_t)a.W * a.C;
    const unsigned ibase = b * (unsigned)a.OH * (unsigned)grow + (unsigned)c, obase = b * (unsigned)a.H * (unsigned)orow + (unsigned)c;

    const int za = a.aq->zero_point;
    const int fill = (int)((unsigned)(za & 0xff) * 0x01010101u);
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);

    // weights by output parity (row, column), bytes in the order of the gradient pixels above
    int wt[4][4], nz[4][4];
    {
        int k[9];
#pragma unroll
        for (int t = 0; t < 9; t++) k[t] = *reinterpret_cast<const int *>(a.Wt + (size_t)t * a.C + c);
        dw_transpose4(k[4], 0, 0, 0, wt[0]);                         // even, even: w[1][1]
        dw_transpose4(k[5], k[3], 0, 0, wt[1]);                      // even, odd:  w[1][2], w[1][0]
        dw_transpose4(k[7], 0, k[1], 0, wt[2]);                      // odd, even:  w[2][1], w[0][1]
        dw_transpose4(k[8], k[6], k[2], k[0], wt[3]);                // odd, odd:   w[2][2], w[2][0], w[0][2], w[0][0]
    }
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int e = 0; e < 4; e++) nz[s][e] = -(za * __builtin_amdgcn_sdot4(wt[s][e], 0x01010101, 0, false));

    const bool okr = x + 1 < a.OW, both = 2 * x + 1 < a.W, pair = (a.W & 1) == 0;
    const unsigned goff = ibase + (unsigned)x * (unsigned)a.C, goff1 = okr ? goff + (unsigned)a.C : goff;
    const unsigned off0 = obase + 2u * (unsigned)x * (unsigned)a.C, off1 = off0 + (unsigned)a.C;
    auto load_row = [&](int y, int (&raw)[2]) {
        if (y < a.OH) {
            const int8_t *p = a.A + (size_t)y * grow;
            raw[0] = dw_load(p, goff);
            raw[1] = dw_load(p, goff1);
        } else {
            raw[0] = raw[1] = fill;
        }
    };

    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    int ring[RING][2];                                               // slot k: gradient row y0 + k, y0 + k + 3, ...
    auto run = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int k = 0; k < RING; k++) load_row(y0 + k, ring[k]);
        ring[0][1] = okr ? ring[0][1] : fill;
        int y = y0;
        auto step = [&](auto phase) {
            constexpr int P = decltype(phase)::value, Q = (P + 1) % 3;
            ring[Q][1] = okr ? ring[Q][1] : fill;                    // (the upper row's turn came one step earlier)
            int t[4];
            dw_transpose4(ring[P][0], ring[P][1], ring[Q][0], ring[Q][1], t);
            if (y + RING <= y1) load_row(y + RING, ring[P]);
#pragma unroll
            for (int i = 0; i < 2; i++) {
                if (2 * y + i >= a.H) continue;
                int cv[8];
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    cv[e] = __builtin_amdgcn_sdot4(t[e], wt[2 * i][e], nz[2 * i][e], false);
                    cv[4 + e] = __builtin_amdgcn_sdot4(t[e], wt[2 * i + 1][e], nz[2 * i + 1][e], false);
                }
                dw_emit<MODE, FULL>(a, ep, cv, (size_t)(2 * y + i) * orow, off0, off1, pair, both, mn, mx, nlo, nhi);
            }
            y++;
        };
        while (true) {
            step(dw_int<0>());
            if (y >= y1) break;
            step(dw_int<1>());
            if (y >= y1) break;
            step(dw_int<2>());
            if (y >= y1) break;
        }
    };
    if (live) {
        if (MODE == 0 || ep.full_grid) run(std::true_type()); else run(std::false_type());
    }
    hq_block_stats_commit(mn, mx, nlo, nhi, a.st, red, blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z));
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.B * a.H * a.W * (unsigned long long)a.C);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

// Weight gradient: acc[tap][c] = sum_m Xg[m][tap][c] * G[m][c], plus the column sums that
// remove the zero points.  Each workgroup takes a run of pixels; a thread owns four channels
// and strides over the run; partial sums meet in LDS and leave with one atomic per value.
constexpr int DW_MAX_TAPS = 9;

struct DwWgradArgs {
    const int8_t *X, *G;
    const hq_qparams *xq;
    int32_t *acc, *gsum, *xsum;
    int M, C, R, S, H, W, OH, OW, stride, pad;
    int m_per_block;
    int CT;                        // channels per workgroup (multiple of 4, <= 256)
};

__global__ __launch_bounds__(HQ_THREADS) void hq_depthwise_wgrad_kernel(const DwWgradArgs a)
{
    extern __shared__ int lds[];                 // [taps][CT] acc, [CT] gsum, [taps][CT] xsum
    const int taps = a.R * a.S, CT = a.CT;
    const int ct0 = blockIdx.y * CT, ct = min(CT, a.C - ct0);      // this workgroup's channel tile
    const int words = (2 * taps + 1) * CT;
    for (int i = threadIdx.x; i < words; i += blockDim.x) lds[i] = 0;
    __syncthreads();
    const int zx = a.xq->zero_point;
    const int fill = (int)((unsigned)(zx & 0xff) * 0x01010101u);   // unsigned: the product may set bit 31
    const int lanes_per_pixel = ct >> 2;                           // <= 64
    const int pixels_per_pass = HQ_THREADS / lanes_per_pixel;
    const int cg = threadIdx.x % lanes_per_pixel, prow = threadIdx.x / lanes_per_pixel;
    const int cl = cg * 4, c = ct0 + cl;
    const int m_begin = blockIdx.x * a.m_per_block, m_end = min(a.M, m_begin + a.m_per_block);
    if (prow < pixels_per_pass) {
        int acc[DW_MAX_TAPS][4], xs[DW_MAX_TAPS][4], gs[4] = {0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < DW_MAX_TAPS; t++)
#pragma unroll
            for (int e = 0; e < 4; e++) { acc[t][e] = 0; xs[t][e] = 0; }
        for (int m = m_begin + prow; m < m_end; m += pixels_per_pass) {
            const int ow = m % a.OW, oh = (m / a.OW) % a.OH, b = m / (a.OW * a.OH);
            const int gv = *reinterpret_cast<const int *>(a.G + (size_t)m * a.C + c);
            int g[4];
#pragma unroll
            for (int e = 0; e < 4; e++) { g[e] = sbyte(gv, e); gs[e] += g[e]; }
#pragma unroll
            for (int t = 0; t < DW_MAX_TAPS; t++) {
                if (t < taps) {
                    const int r = t / a.S, s = t % a.S;
                    const int iy = oh * a.stride - a.pad + r, ix = ow * a.stride - a.pad + s;
                    const bool ok = iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
                    const int xv = ok ? *reinterpret_cast<const int *>(a.X + (((size_t)b * a.H + iy) * a.W + ix) * a.C + c) : fill;
#pragma unroll
                    for (int e = 0; e < 4; e++) { const int x = sbyte(xv, e); acc[t][e] += x * g[e]; xs[t][e] += x; }
                }
            }
        }
#pragma unroll
        for (int t = 0; t < DW_MAX_TAPS; t++)
            if (t < taps)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    atomicAdd(&lds[t * CT + cl + e], acc[t][e]);
                    atomicAdd(&lds[(taps + 1 + t) * CT + cl + e], xs[t][e]);
                }
#pragma unroll
        for (int e = 0; e < 4; e++) atomicAdd(&lds[taps * CT + cl + e], gs[e]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < words; i += blockDim.x) {
        const int v = lds[i];
        const int row = i / CT, col = i % CT;
        if (v == 0 || col >= ct) continue;
        if (row < taps) atomicAdd(a.acc + row * a.C + ct0 + col, v);
        else if (row == taps) atomicAdd(a.gsum + ct0 + col, v);
        else atomicAdd(a.xsum + (row - taps - 1) * a.C + ct0 + col, v);
    }
}

// Weight gradient of the 3x3 layers with padding 1 and stride 1 or 2, in the manner of hq_dw3x3_kernel: a thread owns four
// channels of four neighbouring output columns and walks down a strip of rows and over several images.  The reduction
// runs over pixels, so the four columns' gradients and the inputs of one tap column are byte-transposed words, and a tap's
// share of the four pixels is one 4-way dot product; the words of the neighbouring tap columns are the same pixels moved
// by one (one v_perm each).  7.0 vector instructions per pixel and channel (22.5 in the earlier kernel, which packed rows and
// fetched every input three times): 38 us instead of 68 for 128 x 56 x 56 x 192, stride 2 21 instead of 86.  Their issue is a third of
// that now; one workgroup per compute unit waits for its loads.  Threads that share channels meet in LDS, and the workgroup
// leaves with one atomic per value.  Where the gradient's zero point is not 0 a second walk, with ones in place of the gradients, gathers the
// column sums of the input that remove it.
struct Dw3WgradArgs {
    const int8_t *X, *G;
    const hq_qparams *xq, *gq;
    int32_t *acc, *gsum, *xsum;
    int B, H, W, OH, OW, C;
    int images;                    // images side by side; a thread takes every images-th
    int rows_per_strip;
};

constexpr int DW_WG_THREADS = 512;

template <int STRIDE>
__global__ __launch_bounds__(DW_WG_THREADS) void hq_dw3x3_wgrad_kernel(const Dw3WgradArgs a)
{
    constexpr int NW = STRIDE == 1 ? 6 : 9;                          // input columns of the four outputs
    extern __shared__ int lds[];                                     // [9][C] acc or xsum, [C] gsum
    const int c4n = a.C >> 2, cols4 = (a.OW + 3) >> 2;
    const unsigned q = blockIdx.x * DW_WG_THREADS + threadIdx.x;                // (image of the first round, column group, word)
    const bool live = q < (unsigned)a.images * cols4 * c4n;
    const unsigned qx = (live ? q : 0) / c4n, b0 = qx / cols4;
    const int x = 4 * (int)(qx - b0 * cols4), c = (int)((live ? q : 0) - qx * c4n) * 4;
    const int y0 = blockIdx.y * a.rows_per_strip, y1 = min(a.OH, y0 + a.rows_per_strip);
    const size_t xrow = (size_t)a.W * a.C, grow = (size_t)a.OW * a.C;
    const int zx = a.xq->zero_point;
    const int fill = (int)((unsigned)(zx & 0xff) * 0x01010101u);     // unsigned: the product may set bit 31
    const int passes = a.gq->zero_point != 0 ? 2 : 1;

    unsigned xoff[NW], goff[4];
    bool xok[NW], gok[4];
#pragma unroll
    for (int k = 0; k < NW; k++) {
        const int xi = STRIDE * x - 1 + k;
        xok[k] = xi >= 0 && xi < a.W;
        xoff[k] = (unsigned)(xok[k] ? xi : STRIDE * x) * (unsigned)a.C + (unsigned)c;
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        gok[k] = x + k < a.OW;
        goff[k] = (unsigned)(gok[k] ? x + k : x) * (unsigned)a.C + (unsigned)c;
    }

    for (int pass = 0; pass < passes; pass++) {
        for (int i = threadIdx.x; i < 10 * a.C; i += DW_WG_THREADS) lds[i] = 0;
        __syncthreads();
        int acc[9][4], gs[4] = {0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < 9; t++)
#pragma unroll
            for (int e = 0; e < 4; e++) acc[t][e] = 0;
        if (live) {
            for (int b = (int)b0; b < a.B; b += a.images) {
                // (tensors have fewer than 2^32 elements)
                const unsigned ximg = (unsigned)b * (unsigned)a.H * (unsigned)xrow, gimg = (unsigned)b * (unsigned)a.OH * (unsigned)grow;
                auto load_x = [&](int y, int (&raw)[NW]) {           // y is the same for the whole workgroup
                    if (y >= 0 && y < a.H) {
                        const int8_t *p = a.X + (size_t)y * xrow;
#pragma unroll
                        for (int k = 0; k < NW; k++) raw[k] = dw_load(p, ximg + xoff[k]);
                    } else {
#pragma unroll
                        for (int k = 0; k < NW; k++) raw[k] = fill;
                    }
                };
                auto load_g = [&](int y, int (&raw)[4]) {            // rows outside the strip count as zero
                    if (y >= y0 && y < y1) {
                        const int8_t *p = a.G + (size_t)y * grow;
#pragma unroll
                        for (int k = 0; k < 4; k++) raw[k] = dw_load(p, gimg + goff[k]);
                    } else {
#pragma unroll
                        for (int k = 0; k < 4; k++) raw[k] = 0;
                    }
                };
                // words of the three tap columns: t[s][e] = input pixels STRIDE * (x .. x+3) - 1 + s of channel e
                auto transpose_x = [&](int (&raw)[NW], int (&t)[3][4]) {
#pragma unroll
                    for (int k = 0; k < NW; k++)
                        if (k != 1) raw[k] = xok[k] ? raw[k] : fill;
                    if constexpr (STRIDE == 1) {
                        dw_transpose4(raw[1], raw[2], raw[3], raw[4], t[1]);
                        t[0][0] = dw_shift_back<0>(t[1][0], raw[0]); t[0][1] = dw_shift_back<1>(t[1][1], raw[0]);
                        t[0][2] = dw_shift_back<2>(t[1][2], raw[0]); t[0][3] = dw_shift_back<3>(t[1][3], raw[0]);
                        t[2][0] = dw_shift_in<0>(t[1][0], raw[5]); t[2][1] = dw_shift_in<1>(t[1][1], raw[5]);
                        t[2][2] = dw_shift_in<2>(t[1][2], raw[5]); t[2][3] = dw_shift_in<3>(t[1][3], raw[5]);
                    } else {
                        dw_transpose4(raw[0], raw[2], raw[4], raw[6], t[0]);
                        dw_transpose4(raw[1], raw[3], raw[5], raw[7], t[1]);
                        t[2][0] = dw_shift_in<0>(t[0][0], raw[8]); t[2][1] = dw_shift_in<1>(t[0][1], raw[8]);
                        t[2][2] = dw_shift_in<2>(t[0][2], raw[8]); t[2][3] = dw_shift_in<3>(t[0][3], raw[8]);
                    }
                };
                auto transpose_g = [&](int (&raw)[4], int y, int (&t)[4]) {
                    if (pass == 1) {                                 // ones where an output exists
                        const bool row = y >= y0 && y < y1;
#pragma unroll
                        for (int k = 0; k < 4; k++) raw[k] = row ? 0x01010101 : 0;
                    }
#pragma unroll
                    for (int k = 1; k < 4; k++) raw[k] = gok[k] ? raw[k] : 0;
                    dw_transpose4(raw[0], raw[1], raw[2], raw[3], t);
#pragma unroll
                    for (int e = 0; e < 4; e++) gs[e] = __builtin_amdgcn_sdot4(t[e], 0x01010101, gs[e], false);
                };
                auto tap_row = [&](int r, const int (&t)[3][4], const int (&g)[4]) {
#pragma unroll
                    for (int s = 0; s < 3; s++)
#pragma unroll
                        for (int e = 0; e < 4; e++) acc[3 * r + s][e] = __builtin_amdgcn_sdot4(t[s][e], g[e], acc[3 * r + s][e], false);
                };
                if constexpr (STRIDE == 1) {
                    // input row y meets gradient rows y + 1, y, y - 1 with the filter's rows 0, 1, 2
                    int xr[2][NW], gr[2][4], g[3][4] = {};
                    load_x(y0 - 1, xr[0]); load_g(y0, gr[0]);
                    load_x(y0, xr[1]); load_g(y0 + 1, gr[1]);
                    int y = y0 - 1;
                    auto step = [&](auto phase) {                    // 6 phases: two raw sets, three gradient slots
                        constexpr int P = decltype(phase)::value, R = P % 2, N = P % 3, C0 = (P + 2) % 3, L = (P + 1) % 3;
                        int t[3][4];
                        transpose_x(xr[R], t);
                        transpose_g(gr[R], y + 1, g[N]);
                        if (y + 2 <= y1) { load_x(y + 2, xr[R]); load_g(y + 3, gr[R]); }
                        tap_row(0, t, g[N]);
                        tap_row(1, t, g[C0]);
                        tap_row(2, t, g[L]);
                        y++;
                    };
                    while (true) {
                        step(dw_int<0>()); if (y > y1) break;
                        step(dw_int<1>()); if (y > y1) break;
                        step(dw_int<2>()); if (y > y1) break;
                        step(dw_int<3>()); if (y > y1) break;
                        step(dw_int<4>()); if (y > y1) break;
                        step(dw_int<5>()); if (y > y1) break;
                    }
                } else {
                    // output row y meets input rows 2y - 1, 2y, 2y + 1; the last is the next row's first
                    int xr[2][NW], gr[4], t[2][3][4];
                    load_x(2 * y0 - 1, xr[0]);
                    transpose_x(xr[0], t[0]);
                    load_x(2 * y0, xr[0]); load_x(2 * y0 + 1, xr[1]); load_g(y0, gr);
                    int y = y0;
                    auto step = [&](auto phase) {
                        constexpr int P = decltype(phase)::value;
                        int g[4], te[3][4];
                        transpose_x(xr[0], te);
                        transpose_x(xr[1], t[1 - P]);
                        transpose_g(gr, y, g);
                        if (y + 1 < y1) { load_x(2 * y + 2, xr[0]); load_x(2 * y + 3, xr[1]); load_g(y + 1, gr); }
                        tap_row(0, t[P], g);
                        tap_row(1, te, g);
                        tap_row(2, t[1 - P], g);
                        y++;
                    };
                    while (true) {
                        step(dw_int<0>()); if (y >= y1) break;
                        step(dw_int<1>()); if (y >= y1) break;
                    }
                }
            }
#pragma unroll
            for (int t = 0; t < 9; t++)
#pragma unroll
                for (int e = 0; e < 4; e++) atomicAdd(&lds[t * a.C + c + e], acc[t][e]);
            if (pass == 0)
#pragma unroll
                for (int e = 0; e < 4; e++) atomicAdd(&lds[9 * a.C + c + e], gs[e]);
        }
        __syncthreads();
        int32_t *sums = pass == 0 ? a.acc : a.xsum;
        for (int i = threadIdx.x; i < 10 * a.C; i += DW_WG_THREADS) {
            const int v = lds[i];
            if (v != 0) atomicAdd(i < 9 * a.C ? sums + i : a.gsum + (i - 9 * a.C), v);
        }
        __syncthreads();
    }
}

__global__ void dw_zero_kernel(int32_t *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

__global__ void dw_wgrad_finalize_kernel(const int32_t *acc, const int32_t *gsum, const int32_t *xsum,
                                         const hq_qparams *xq, const hq_qparams *gq, unsigned M, int K, int C,
                                         float *dW, int32_t *dW_acc, const HqRideAlong ride)
{
    if (hq_ride_along(ride)) return;
    const unsigned zx = (unsigned)xq->zero_point, zg = (unsigned)gq->zero_point;
    const float s = __fmul_rn(xq->scale, gq->scale);
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const unsigned c = (unsigned)acc[k] - zx * (unsigned)gsum[k % C] - zg * (unsigned)xsum[k] + M * zx * zg;
    if (dW_acc) dW_acc[k] = (int)c;
    dW[k] = __fmul_rn(s, (float)(int)c);
}

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

} // namespace

int hq_launch_depthwise(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Wt,
                        const hq_qparams *bq, const int32_t *wsum, const hq_range *range, int8_t *out8,
                        int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    if (sr_seed && out32) return HQ_E_BADARG;
    DwArgs a;
    a.sr_on = sr_seed ? 1 : 0;
    a.sr.k0 = sr_seed ? (unsigned)*sr_seed : 0u; a.sr.k1 = sr_seed ? (unsigned)(*sr_seed >> 32) : 0u;
    a.A = A; a.Wt = Wt; a.wsum = wsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    a.C = p->C; a.R = p->R; a.S = p->S; a.stride = p->stride; a.pad = p->pad; a.dgrad = dgrad;
    if (!dgrad) { a.M = p->B * OH * OW; a.Hs = p->H; a.Ws = p->W; a.Ho = OH; a.Wo = OW; }
    else        { a.M = p->B * p->H * p->W; a.Hs = OH; a.Ws = OW; a.Ho = p->H; a.Wo = p->W; }
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    if (p->R == 3 && p->S == 3 && p->stride <= 2 && p->pad == 1) {
        Dw3Args d;
        d.A = A; d.Wt = Wt; d.wsum = wsum; d.aq = aq; d.bq = bq; d.range = range;
        d.out8 = out8; d.out32 = out32; d.outq = outq; d.st = st;
        d.B = p->B; d.H = p->H; d.W = p->W; d.OH = OH; d.OW = OW; d.C = p->C; d.flip = dgrad; d.sr = a.sr;
        const bool s2_dgrad = dgrad && p->stride == 2;
        const int cols = s2_dgrad ? OW : (OW + 1) / 2;
        const long xb = ((long)p->B * cols * (p->C / 4) + HQ_THREADS - 1) / HQ_THREADS;
        // strips of output rows: about 16 workgroups per compute unit, at least four rows each (a strip reads two input
        // rows beyond its own); shorter ones as long as that makes no more than two workgroups per compute unit, since a
        // strip is a serial chain (1 x 14 x 14 x 960, stride 2, stochastic input gradient: four rows 8.6 us, one 4.7)
        int strips = (int)std::max(std::min((4096 + xb - 1) / xb, (long)(OH + 3) / 4), std::min((long)OH, 512 / xb));
        d.rows_per_strip = (OH + strips - 1) / strips;
        strips = (OH + d.rows_per_strip - 1) / d.rows_per_strip;
        const dim3 grid((unsigned)xb, (unsigned)strips);
        if (s2_dgrad) {
            auto k = mode == 0 ? hq_dw3x3_s2_dgrad_kernel<0> : mode == 1 ? hq_dw3x3_s2_dgrad_kernel<1> : hq_dw3x3_s2_dgrad_kernel<2>;
            hipLaunchKernelGGL(k, grid, dim3(HQ_THREADS), 0, stream, d);
        } else if (p->stride == 2) {
            auto k = mode == 0 ? hq_dw3x3_kernel<2, 0> : hq_dw3x3_kernel<2, 1>;       // (forward only: never stochastic)
            hipLaunchKernelGGL(k, grid, dim3(HQ_THREADS), 0, stream, d);
        } else {
            auto k = mode == 0 ? hq_dw3x3_kernel<1, 0> : mode == 1 ? hq_dw3x3_kernel<1, 1> : hq_dw3x3_kernel<1, 2>;
            hipLaunchKernelGGL(k, grid, dim3(HQ_THREADS), 0, stream, d);
        }
        return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
    }
    const size_t total = (size_t)a.M * (a.C / 4);
    size_t blocks = (total + HQ_THREADS - 1) / HQ_THREADS;
    if (blocks > 256u * 64u) blocks = 256u * 64u;
    hipLaunchKernelGGL(hq_depthwise_kernel, dim3((unsigned)blocks), dim3(HQ_THREADS), 0, stream, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

int hq_launch_depthwise_wgrad(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                              const hq_qparams *gq, float *dW, int32_t *dW_acc, void *ws, hipStream_t stream,
                              const HqRideAlong *ride)
{
    if (p->R * p->S > DW_MAX_TAPS) return HQ_E_BADSHAPE;
    HqRideAlong ra = {nullptr, nullptr, 0, 0};
    if (ride) ra = *ride;
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    const int taps = p->R * p->S;
    const size_t K = (size_t)taps * p->C;
    DwWgradArgs a;
    a.X = X; a.G = dY; a.xq = xq;
    char *w = static_cast<char *>(ws);
    a.acc = reinterpret_cast<int32_t *>(w);
    a.gsum = reinterpret_cast<int32_t *>(w + align16(4 * K));
    a.xsum = reinterpret_cast<int32_t *>(w + align16(4 * K) + align16(4 * (size_t)p->C));
    a.M = p->B * OH * OW; a.C = p->C; a.R = p->R; a.S = p->S; a.H = p->H; a.W = p->W; a.OH = OH; a.OW = OW;
    a.stride = p->stride; a.pad = p->pad;
    const size_t ws_words = hq_wgrad_workspace_bytes(p) / 4;
    hipLaunchKernelGGL(dw_zero_kernel, dim3(16), dim3(256), 0, stream, a.acc, ws_words);
    const size_t dw3_lds = 10 * (size_t)p->C * 4;
    if (p->R == 3 && p->S == 3 && p->stride <= 2 && p->pad == 1 && dw3_lds <= 64 * 1024) {
        Dw3WgradArgs d;
        d.X = X; d.G = dY; d.xq = xq; d.gq = gq; d.acc = a.acc; d.gsum = a.gsum; d.xsum = a.xsum;
        d.B = p->B; d.H = p->H; d.W = p->W; d.OH = OH; d.OW = OW; d.C = p->C;
        // One workgroup of DW_WG_THREADS per compute unit: every workgroup ends with up to 10 * C atomics on the same
        // addresses, so more of them cost more than the latency they hide.  Strips of at least four rows where the
        // images alone are too few, then images in turn; shorter ones up to 64 workgroups and 28 strips (32 x 7 x 7 x 32: four rows
        // 10.3 us, one 9.4).
        const long per = (long)((OW + 3) / 4) * (p->C / 4);          // threads of one image
        const long most = 256L * DW_WG_THREADS;
        int strips = (int)std::max({1L, std::min(most / (per * p->B), (long)(OH + 3) / 4), std::min({(long)OH, 28L, 64L * DW_WG_THREADS / (per * p->B)})});
        d.rows_per_strip = (OH + strips - 1) / strips;
        strips = (OH + d.rows_per_strip - 1) / d.rows_per_strip;
        d.images = (int)std::max(1L, std::min((long)p->B, most / (per * strips)));
        const unsigned blocks = (unsigned)((d.images * per + DW_WG_THREADS - 1) / DW_WG_THREADS);
        auto k = p->stride == 1 ? hq_dw3x3_wgrad_kernel<1> : hq_dw3x3_wgrad_kernel<2>;
        hipLaunchKernelGGL(k, dim3(blocks, (unsigned)strips), dim3(DW_WG_THREADS), dw3_lds, stream, d);
        ra.first = (int)((K + 255) / 256);
        hipLaunchKernelGGL(dw_wgrad_finalize_kernel, dim3((unsigned)((K + 255) / 256) + (unsigned)ra.n), dim3(256), 0, stream,
                           a.acc, a.gsum, a.xsum, xq, gq, (unsigned)a.M, (int)K, p->C, dW, dW_acc, ra);
        return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
    }
    a.CT = p->C < 256 ? p->C : 256;
    const int ctiles = (p->C + a.CT - 1) / a.CT;
    int blocks = (2048 + ctiles - 1) / ctiles;
    a.m_per_block = (a.M + blocks - 1) / blocks;
    if (a.m_per_block < 1) a.m_per_block = 1;
    blocks = (a.M + a.m_per_block - 1) / a.m_per_block;
    const size_t lds_bytes = (size_t)(2 * taps + 1) * a.CT * 4;       // at most 19 KiB
    hipLaunchKernelGGL(hq_depthwise_wgrad_kernel, dim3((unsigned)blocks, (unsigned)ctiles), dim3(HQ_THREADS),
                       lds_bytes, stream, a);
    ra.first = (int)((K + 255) / 256);
    hipLaunchKernelGGL(dw_wgrad_finalize_kernel, dim3((unsigned)((K + 255) / 256) + (unsigned)ra.n), dim3(256), 0, stream,
                       a.acc, a.gsum, a.xsum, xq, gq, (unsigned)a.M, (int)K, p->C, dW, dW_acc, ra);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}
