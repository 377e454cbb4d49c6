// Weight gradient G_W = X~^T . G~_Y on int8 MFMA (paper Sec. 3.1; kept in FP32, no quantizer).
//
//   acc[n][tap][c] = sum_m  G[m][n] * Xg[m][tap][c]          m = (b, oh, ow) over all output pixels
//
// The reduction runs over pixels, which is the slow dimension of both NHWC operands, while
// an MFMA lane wants 16 reduction-contiguous bytes.  Both tiles are therefore staged in LDS
// as they lie in memory ([pixel][channel], 16-byte coalesced loads) and read back through the
// transposing LDS load of gfx950 (ds_read_b64_tr_b8): 16 lanes hand in 16 row addresses and
// receive, per lane, one channel of 8 consecutive pixels.
//
// Zero points: taps outside the image are filled with X's zero-point code, rows past the end
// of the tensor with code 0 in both operands, and the raw sum is corrected afterwards by
//   c = acc - z_x * sum_m G[m][n] - z_g * sum_m Xg[m][tap][c] + M * z_x * z_g .
// The two column sums come from the same fragments (dot4 against ones) in the workgroups of
// the first tile column / row.  The pixel range is split over workgroups (split-K); partial
// tiles are merged with 32-bit integer atomics, which is exact in any order.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>

namespace {

constexpr int WP_THREADS = 512;
constexpr int MB = 64;             // pixels staged per step (two MFMA k-steps of 32)

struct WgradArgs {
    const int8_t *X, *G;
    const hq_qparams *xq, *gq;
    int32_t *acc;                  // [N][taps][C], zeroed
    int32_t *gsum;                 // [N], zeroed
    int32_t *xsum;                 // [taps][C], zeroed
    int M, N, C;
    int R, S, H, W, OH, OW, stride, pad;
    int m_per_split;               // multiple of MB
    int ctiles;                    // tiles along C inside one tap
    int xt, yt, splits;            // tile columns (taps * ctiles), tile rows, pixel splits
    int g16, x16;                  // rows of G / X are 16-byte aligned (N % 16 == 0 / C % 16 == 0)
    int direct;                    // splits == 1: every sum has one writer, plain stores into acc (not zeroed)
    unsigned magic_OW, magic_OH;   // ceil(2^32 / d) for the pixel decode, or 0, 0 with magic_ok == 0: plain division
    int magic_ok;
};

__device__ inline v4i load16(const int8_t *p, int nbytes, bool aligned16)
{
    if (aligned16) return *reinterpret_cast<const v4i *>(p);
    v4i v;
    const int *q = reinterpret_cast<const int *>(p);
    v[0] = nbytes > 0 ? q[0] : 0;
    v[1] = nbytes > 4 ? q[1] : 0;
    v[2] = nbytes > 8 ? q[2] : 0;
    v[3] = nbytes > 12 ? q[3] : 0;
    return v;
}

// PACKED: layers with fewer than 16 input channels (a network's first layer).  The tile's columns
// then run over (tap, channel) pairs as they lie in a row of G_W, so a 16-byte chunk of the staged
// tile holds 16 / C taps (one 4-byte load each) instead of one tap padded with zeros.
// PACKED3: 3-channel inputs (RGB images).  The S * 3 <= 32 bytes of a filter row are contiguous in the
// input; every filter row gets 32 tile columns of its own (column = 32 * r + 3 * s + channel, the columns
// past S * 3 stay zero), so a thread's 16-byte chunk is 16 consecutive bytes of memory at any byte
// address: aligned loads plus a byte-wise funnel shift, then byte masks that replace the taps outside the
// image with the zero-point code.
// ALIGNED: rows of both operands are whole 16-byte chunks (and the pixel decode fits hq_magic_div): loads without a branch, lanes without
// a source read the tensor's first bytes, and what they hold is replaced when it is stored to LDS.  With a branch per load
// and per alignment a stage of 8 MFMAs was some 400 instructions: 3x3 stride 2, 256 x 28 x 28 x 128 -> 256 58.0 us, now 53.5;
// linear 8192 x 1024 -> 1024 47.4, now 43.6.
template <int TN, int TK, bool PACKED, bool PACKED3 = false, bool ALIGNED = false>
__global__ __launch_bounds__(HQ_THREADS) void hq_wgrad_kernel(const WgradArgs a)
{
    static_assert(!PACKED3 || PACKED, "the 3-channel form is a packed form");
    constexpr int PG = TN + 32, PX = TK + 32;           // LDS pitches (32 mod 64: best for the transposing reads)
    constexpr int WTN = TN / 2, WTK = TK / 2;           // 2 x 2 wavefronts
    constexpr int NT = WTN / 32, KT = WTK / 32;
    constexpr int GCH = TN / 16, XCH = TK / 16;         // 16-byte chunks per tile row
    constexpr int GLD = MB * GCH / HQ_THREADS, XLD = MB * XCH / HQ_THREADS;
    static_assert(GLD >= 1 && XLD >= 1, "tile too small for 256 loader threads");

    __shared__ __attribute__((aligned(16))) int8_t Gs[2][MB * PG];
    __shared__ __attribute__((aligned(16))) int8_t Xs[2][MB * PX];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: branches on it are uniform
    const int wn = wave >> 1, wk = wave & 1;
    // Workgroup -> (tile column bx, tile row by, pixel split bz).  All tile columns and rows of
    // one pixel split read the same X / dY rows; consecutive workgroup ids go round-robin over
    // the 8 XCDs, so the ids are re-mapped to keep one split's tiles on one XCD, back to back,
    // where its L2 serves the re-reads.
    int bx, by, bz;
    {
        const int per_split = a.xt * a.yt, total = per_split * a.splits;
        const int full = (total / (8 * per_split)) * (8 * per_split);   // ids covered by complete groups of 8 splits
        int split, tile;
        if ((int)blockIdx.x < full) {
            const int grp = blockIdx.x / (8 * per_split), r = blockIdx.x % (8 * per_split);
            split = grp * 8 + (r & 7); tile = r >> 3;
        } else {
            const int r = blockIdx.x - full;
            split = full / per_split + r / per_split; tile = r % per_split;
        }
        bx = tile % a.xt; by = tile / a.xt; bz = split;
    }
    const int tap = PACKED ? 0 : bx / a.ctiles, c0 = PACKED ? bx * TK : (bx % a.ctiles) * TK;
    const int tr = tap / a.S, ts = tap % a.S;
    const int kcols = a.R * a.S * a.C;            // PACKED: columns of the whole weight row
    const int n0 = by * TN;
    const int m_begin = bz * a.m_per_split;
    const int m_end = min(a.M, m_begin + a.m_per_split);
    const int zx = a.xq->zero_point;
    const int fill = (int)((unsigned)(zx & 0xff) * 0x01010101u);   // unsigned: the product may set bit 31
    // (a column sum is only ever multiplied by the other operand's zero point: not formed when that is 0)
    const bool do_gsum = bx == 0 && wk == 0 && zx != 0;                      // column sums of G: first tile column
    const bool do_xsum = by == 0 && wn == 0 && a.gq->zero_point != 0;        // column sums of Xg: first tile row

    int pk_r[4], pk_s[4], pk_off[4], pk_ow[XLD], pk_oh[XLD], pk_b[XLD];
    if (PACKED) {
#pragma unroll
        for (int d = 0; d < 4; d++) {
            const int kc = c0 + (tid % XCH) * 16 + 4 * d;
            if (PACKED3) {
                // word d = bytes 4 * d .. 4 * d + 3 of this thread's 16 bytes of filter row pk_r[0]
                const int q = (c0 >> 4) + (tid % XCH);                 // 16-byte chunk: filter row q / 2, half q % 2
                pk_r[d] = (q >> 1) < a.R ? (q >> 1) : -1;
                pk_s[d] = 16 * (q & 1) + 4 * d;                        // first byte of the word inside the filter row
                pk_off[d] = pk_r[d] * a.W * 3 + 16 * (q & 1);
                continue;
            }
            const int t = kc / a.C, cc = kc - t * a.C;
            pk_r[d] = kc < kcols ? t / a.S : -1;
            pk_s[d] = t % a.S;
            pk_off[d] = (pk_r[d] * a.W + pk_s[d]) * a.C + cc;
        }
#pragma unroll
        for (int i = 0; i < XLD; i++) {
            const int m = m_begin + (tid + i * HQ_THREADS) / XCH;
            pk_ow[i] = m % a.OW; pk_oh[i] = (m / a.OW) % a.OH; pk_b[i] = m / (a.OW * a.OH);
        }
    }
    v4i greg[GLD], xreg[XLD];
    unsigned gok = 0, xin = 0, xrow = 0;                        // ALIGNED, a bit per load: gradient, input pixel, pixel at all
    auto load_stage = [&](int mb) {
        if constexpr (ALIGNED) {
            const int n = n0 + (tid % GCH) * 16, c = c0 + (tid % XCH) * 16;          // (HQ_THREADS is a multiple of both)
            gok = xin = xrow = 0;
#pragma unroll
            for (int i = 0; i < GLD; i++) {
                const int m = mb + (tid + i * HQ_THREADS) / GCH;
                const bool ok = m < m_end && n < a.N;
                greg[i] = *reinterpret_cast<const v4i *>(ok ? a.G + (size_t)m * a.N + n : a.G);
                gok |= ok ? 1u << i : 0u;
            }
#pragma unroll
            for (int i = 0; i < XLD; i++) {
                const int m = mb + (tid + i * HQ_THREADS) / XCH;
                const unsigned t = hq_magic_div((unsigned)m, a.magic_OW), b = hq_magic_div(t, a.magic_OH);
                const int iy = (int)(t - b * (unsigned)a.OH) * a.stride - a.pad + tr;
                const int ix = (int)((unsigned)m - t * (unsigned)a.OW) * a.stride - a.pad + ts;
                const bool row = m < m_end && c < a.C, in = row && (unsigned)iy < (unsigned)a.H && (unsigned)ix < (unsigned)a.W;
                xreg[i] = *reinterpret_cast<const v4i *>(in ? a.X + (((size_t)b * a.H + iy) * a.W + ix) * a.C + c : a.X);
                xin |= in ? 1u << i : 0u;
                xrow |= row ? 1u << i : 0u;
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < GLD; i++) {
            const int idx = tid + i * HQ_THREADS, row = idx / GCH, col = (idx % GCH) * 16;
            const int m = mb + row, n = n0 + col;
            v4i v = {0, 0, 0, 0};
            if (m < m_end && n < a.N) v = load16(a.G + (size_t)m * a.N + n, a.N - n, a.g16);
            greg[i] = v;
        }
#pragma unroll
        for (int i = 0; i < XLD; i++) {
            const int idx = tid + i * HQ_THREADS, row = idx / XCH, col = (idx % XCH) * 16;
            const int m = mb + row, c = c0 + col;
            v4i v = {0, 0, 0, 0};
            if (PACKED) {
                // the thread's four (tap, channel) columns never change; its pixels advance by MB per stage
                if (PACKED3 && m < m_end) {
                    const int iy0 = pk_oh[i] * a.stride - a.pad, ix0 = pk_ow[i] * a.stride - a.pad;
                    const int iy = iy0 + pk_r[0];
                    const bool rok = pk_r[0] >= 0 && iy >= 0 && iy < a.H;
                    const int8_t *base = a.X + (((ptrdiff_t)pk_b[i] * a.H + iy0) * a.W + ix0) * 3;
                    const int8_t *xend = a.X + (size_t)(a.M / (a.OH * a.OW)) * a.H * a.W * 3;
                    const int j0 = 3 * max(0, -ix0), j1 = 3 * min(a.S, a.W - ix0);   // bytes of a filter row inside the image
                    const v4i x = hq_load16_any(rok ? base + pk_off[0] : a.X, a.X, xend);
#pragma unroll
                    for (int d = 0; d < 4; d++) {
                        const unsigned mk = rok ? hq_bytemask(j0 - pk_s[d], j1 - pk_s[d]) : 0u;
                        const unsigned all = pk_r[0] >= 0 ? hq_bytemask(0, a.S * 3 - pk_s[d]) : 0u;   // columns that exist
                        v[d] = (int)(((unsigned)x[d] & mk) | ((unsigned)fill & all & ~mk));             // outside the image: real zero
                    }
                } else if (m < m_end) {
                    const int iy0 = pk_oh[i] * a.stride - a.pad, ix0 = pk_ow[i] * a.stride - a.pad;
                    const int8_t *base = a.X + (((size_t)pk_b[i] * a.H + iy0) * a.W + ix0) * a.C;
#pragma unroll
                    for (int d = 0; d < 4; d++) {
                        // branch-free: lanes without a source read the tensor's first word and drop it
                        const int iy = iy0 + pk_r[d], ix = ix0 + pk_s[d];
                        const bool in = pk_r[d] >= 0 && iy >= 0 && iy < a.H && ix >= 0 && ix < a.W;
                        const int x = *reinterpret_cast<const int *>(in ? base + pk_off[d] : a.X);
                        v[d] = in ? x : pk_r[d] >= 0 ? fill : 0;
                    }
                }
                pk_ow[i] += MB;
                while (pk_ow[i] >= a.OW) { pk_ow[i] -= a.OW; pk_oh[i]++; }
                while (pk_oh[i] >= a.OH) { pk_oh[i] -= a.OH; pk_b[i]++; }
            } else if (m < m_end && c < a.C) {
                int ow, oh, b;                                    // (a division costs some 40 instructions, three a stage's worth of MFMAs)
                if (a.magic_ok) {
                    const unsigned t = hq_magic_div((unsigned)m, a.magic_OW), bb = hq_magic_div(t, a.magic_OH);
                    ow = (int)((unsigned)m - t * (unsigned)a.OW); oh = (int)(t - bb * (unsigned)a.OH); b = (int)bb;
                } else {
                    ow = m % a.OW; oh = (m / a.OW) % a.OH; b = m / (a.OW * a.OH);
                }
                const int iy = oh * a.stride - a.pad + tr, ix = ow * a.stride - a.pad + ts;
                if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W) {
                    v = load16(a.X + (((size_t)b * a.H + iy) * a.W + ix) * a.C + c, a.C - c, a.x16);
                } else {
                    // real zero; bytes past the last channel stay 0 so they add nothing to xsum
                    const int nb = a.C - c;
                    v[0] = nb > 0 ? fill : 0; v[1] = nb > 4 ? fill : 0; v[2] = nb > 8 ? fill : 0; v[3] = nb > 12 ? fill : 0;
                }
            }
            xreg[i] = v;
        }
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < GLD; i++) {
            const int idx = tid + i * HQ_THREADS, row = idx / GCH, col = (idx % GCH) * 16;
            *reinterpret_cast<v4i *>(&Gs[buf][row * PG + col]) = !ALIGNED || (gok >> i & 1) ? greg[i] : v4i{0, 0, 0, 0};
        }
#pragma unroll
        for (int i = 0; i < XLD; i++) {
            const int idx = tid + i * HQ_THREADS, row = idx / XCH, col = (idx % XCH) * 16;
            const int z = xrow >> i & 1 ? fill : 0;             // a tap outside the image: real zero; past the end: nothing
            *reinterpret_cast<v4i *>(&Xs[buf][row * PX + col]) = !ALIGNED || (xin >> i & 1) ? xreg[i] : v4i{z, z, z, z};
        }
    };

    v16i acc[NT][KT];
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
        for (int j = 0; j < KT; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0;
    int gs[NT], xs[KT];
#pragma unroll
    for (int i = 0; i < NT; i++) gs[i] = 0;
#pragma unroll
    for (int j = 0; j < KT; j++) xs[j] = 0;

    if (m_begin < m_end) {
        const int stages = (m_end - m_begin + MB - 1) / MB;
        load_stage(m_begin);
        store_stage(0);
        __syncthreads();
        for (int st = 0; st < stages; st++) {
            const int buf = st & 1;
            const bool more = st + 1 < stages;
            if (more) load_stage(m_begin + (st + 1) * MB);
#pragma unroll
            for (int ks = 0; ks < MB / 32; ks++) {
                v4i gf[NT], xf[KT];
#pragma unroll
                for (int i = 0; i < NT; i++)
                    gf[i] = hq_read_frag_tr<PG>(&Gs[buf][ks * 32 * PG + wn * WTN + i * 32], lane);
#pragma unroll
                for (int j = 0; j < KT; j++)
                    xf[j] = hq_read_frag_tr<PX>(&Xs[buf][ks * 32 * PX + wk * WTK + j * 32], lane);
#pragma unroll
                for (int i = 0; i < NT; i++)
#pragma unroll
                    for (int j = 0; j < KT; j++)
                        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gf[i], xf[j], acc[i][j], 0, 0, 0);
                if (do_gsum) {
#pragma unroll
                    for (int i = 0; i < NT; i++)
#pragma unroll
                        for (int d = 0; d < 4; d++) gs[i] = __builtin_amdgcn_sdot4(gf[i][d], 0x01010101, gs[i], false);
                }
                if (do_xsum) {
#pragma unroll
                    for (int j = 0; j < KT; j++)
#pragma unroll
                        for (int d = 0; d < 4; d++) xs[j] = __builtin_amdgcn_sdot4(xf[j][d], 0x01010101, xs[j], false);
                }
            }
            if (more) store_stage(buf ^ 1);
            __syncthreads();
        }
    }

    // ---- merge the partial tile.  G fragments were the first MFMA operand: lane l holds
    // column c = l % 32 of the block and rows n = 8*(r/4) + 4*(l/32) + r%4.
    const size_t krow = (size_t)a.R * a.S * a.C;
#pragma unroll
    for (int i = 0; i < NT; i++)
#pragma unroll
        for (int j = 0; j < KT; j++) {
            int c = c0 + wk * WTK + j * 32 + (lane & 31);
            if (PACKED3) c = (c >> 5) < a.R && (c & 31) < a.S * 3 ? (c >> 5) * a.S * 3 + (c & 31) : kcols;   // tile column -> weight column
            if (c >= (PACKED ? kcols : a.C)) continue;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const int n = n0 + wn * WTN + i * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
                if (n >= a.N) continue;
                int32_t *dst = a.acc + (size_t)n * krow + (size_t)tap * a.C + c;
                if (a.direct) *dst = acc[i][j][r];
                else if (acc[i][j][r] != 0) atomicAdd(dst, acc[i][j][r]);
            }
        }
    if (do_gsum) {
#pragma unroll
        for (int i = 0; i < NT; i++) {
            int s = gs[i] + __shfl_xor(gs[i], 32);
            const int n = n0 + wn * WTN + i * 32 + (lane & 31);
            if (lane < 32 && n < a.N && s != 0) atomicAdd(a.gsum + n, s);
        }
    }
    if (do_xsum) {
#pragma unroll
        for (int j = 0; j < KT; j++) {
            int s = xs[j] + __shfl_xor(xs[j], 32);
            int c = c0 + wk * WTK + j * 32 + (lane & 31);
            if (PACKED3) c = (c >> 5) < a.R && (c & 31) < a.S * 3 ? (c >> 5) * a.S * 3 + (c & 31) : kcols;
            if (lane < 32 && c < (PACKED ? kcols : a.C) && s != 0) atomicAdd(a.xsum + (size_t)tap * a.C + c, s);
        }
    }
}

// ---------------------------------------------------------------------------------------
// Weight gradient of a network's first layer (3 or 4 input channels, W a multiple of 4, at most 8 filter rows and
// 8 taps per filter row, at most 64 output channels in multiples of 16) with the input rows staged in LDS.
// A workgroup walks bands of whole output rows.  The input rows of a band are copied into LDS once, every
// pixel widened to 4 bytes, inside a frame of zero-point pixels; filter row r of output pixel (oy, ox) is then
// the 32 bytes at (oy * stride + r) * pitch + 4 * stride * ox: rows of an implicit [pixel][32 columns] matrix
// with a pitch of 4 * stride bytes, which the transposing LDS read takes as they lie (column 4 s + c of
// filter row r; the columns of the fourth byte and of taps past S are dropped at the end).  The gradient rows
// of the band are copied beside them.  Wavefront (wn, wk) owns output channels 32 wn .. 32 wn + 31 and filter
// rows 4 wk .. 4 wk + 3 (at most 4 filter rows: all of them, for every second k-step); sums stay in registers over all bands
// of the workgroup.
// The transposing read wants 8-byte addresses.  Under an odd stride the odd pixels of a row lie 4 bytes off, and read a second
// copy of the rows that is shifted by as much.
// Measured, whole call with its clearing and finalizing launches (9 us), before -> now: 3x3 stride 1, 128 x 64 x 64 x 3 -> 64 (then one
// tile column per 32 packed columns, loads of unaligned runs) 73.5 -> 36.4 us, 64 x 32 x 32 x 3 -> 32 40.5 -> 14.3, 5x5 on
// 64 x 96 x 96 x 4 -> 48 63 -> 36; 3x3 stride 2, 128 x 112 x 112 x 3 -> 32 38.7 -> 27.1; 7x7 stride 2, 256 x 224 x 224 x 3 -> 64 135 -> 125.
// Wide images, a band of one or two output rows whose input rows are staged again for the next: 3x3 stride 1, 224 x 224 x 3 -> 64 35.7 -> 18.1,
// 5 x 224 x 224 x 3 -> 16 57.3 -> 21.4, 320 x 320 x 3 -> 32 46.2 -> 19.2; where no row fits (320 x 320 x 3 -> 64) the other kernel stays.
// What bounds it now: small ones the 512 workgroups' atomics on the same lines (256 workgroups: 34 us for the first, but 199 for the
// last), the 7x7 one its 76 vector instructions per k-step and wavefront (44 % of the time) and the wait for a band's loads.
struct WstemArgs {
    WgradArgs w;
    int rows_out, in_rows, LP;     // output rows per band, input rows it needs, LDS pitch of an input row
    int xrows;                     // input rows a buffer has room for: (rows_out - 1) * stride + 8 (4 with at most 4 filter rows)
    int second;                    // odd strides: offset of the second copy of the input rows, 4 bytes further right; else 0
    int bands_per_image, nbands;
    int groups;                    // 16-byte groups of four pixels per input row: W / 4
    unsigned magic_groups, magic_OW;
    int gpitch, gchunks;           // LDS pitch of a gradient row, 16-byte chunks of a gradient row that are staged
    int kpad;                      // pixels of a full band rounded up to 32
};
constexpr int WS_XT = 3;           // staged groups of four pixels per thread and band
constexpr int WS_GT = 4;           // staged 16-byte gradient chunks per thread and band

template <int CH>
__global__ __launch_bounds__(HQ_THREADS, 2) void hq_wgrad_stem_kernel(const WstemArgs sa)
{
    const WgradArgs &a = sa.w;
    extern __shared__ __attribute__((aligned(16))) int8_t ws_lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wn = wave >> 1, wk = wave & 1;
    const int zx = a.xq->zero_point;
    const int fill = (int)((unsigned)(zx & 0xff) * 0x01010101u);   // unsigned: the product may set bit 31
    const bool halves = a.R <= 4;                                   // the filter rows fit one wavefront: two share the k-steps
    const int row0 = halves ? 0 : wk * 4;
    const int xbytes = sa.xrows * sa.LP * (sa.second ? 2 : 1), gbytes = sa.kpad * sa.gpitch, buf_bytes = xbytes + gbytes;
    int8_t *zero_row = ws_lds + 2 * (size_t)buf_bytes;              // 64 bytes of 0: the source of pixels past a band
    const bool do_gsum = (wk == 0 || halves) && zx != 0;            // column sums of G (times z_x later)
    const bool do_xsum = wn == 0 && a.gq->zero_point != 0;          // column sums of the gathered input

    // the frame: the input part of both buffers starts as zero-point pixels; staging only writes the W image
    // columns of a row
    for (int b = 0; b < 2; b++)
        for (int q = tid; q < xbytes / 16; q += HQ_THREADS)
            *reinterpret_cast<v4i *>(ws_lds + (size_t)b * buf_bytes + (size_t)q * 16) = v4i{fill, fill, fill, fill};
    if (tid < 4) *reinterpret_cast<v4i *>(zero_row + tid * 16) = v4i{0, 0, 0, 0};

    int stx[WS_XT][CH];
    v4i stg[WS_GT];
    auto band_rows = [&](int band, int &b, int &oy0, int &nrows) {
        b = band / sa.bands_per_image;
        oy0 = (band - b * sa.bands_per_image) * sa.rows_out;
        nrows = min(sa.rows_out, a.OH - oy0);
    };
    // staging plan of this thread, the same for every band: its groups of four input pixels (input row of the
    // band, source offset from the band's first input row, LDS offset) and its 16-byte chunks of the gradient
    int x_row[WS_XT], x_src[WS_XT], x_dst[WS_XT];
#pragma unroll
    for (int k = 0; k < WS_XT; k++) {
        const int t = tid + k * HQ_THREADS;
        const int row = (int)hq_magic_div((unsigned)t, sa.magic_groups), g = t - row * sa.groups;
        x_row[k] = row < sa.in_rows ? row : -1;
        x_src[k] = (row * a.W + 4 * g) * CH;
        x_dst[k] = row * sa.LP + (a.pad + 4 * g) * 4;
    }
    int g_px[WS_GT], g_src[WS_GT], g_dst[WS_GT];
#pragma unroll
    for (int k = 0; k < WS_GT; k++) {
        const int t = tid + k * HQ_THREADS;
        const int px = t / sa.gchunks, cc = t - px * sa.gchunks;
        g_px[k] = px < sa.kpad && 16 * cc < a.N ? px : 0x7fffffff;        // never below a band's pixel count
        g_src[k] = px * a.N + 16 * cc;
        g_dst[k] = px < sa.kpad ? px * sa.gpitch + 16 * cc : -1;
    }
    auto stage_load = [&](int band) {
        int b, oy0, nrows;
        band_rows(band, b, oy0, nrows);
        const int iy0 = oy0 * a.stride - a.pad;
        const int8_t *xrow0 = a.X + ((ptrdiff_t)b * a.H + iy0) * a.W * CH;   // (may lie before the tensor: only rows inside are read)
#pragma unroll
        for (int k = 0; k < WS_XT; k++) {
            const int iy = iy0 + x_row[k];
            const bool ok = x_row[k] >= 0 && iy >= 0 && iy < a.H;
            const int8_t *src = ok ? xrow0 + x_src[k] : a.X;
#pragma unroll
            for (int c = 0; c < CH; c++) stx[k][c] = reinterpret_cast<const int *>(src)[c];
        }
        const int npix = nrows * a.OW;
        const int8_t *g0 = a.G + ((size_t)b * a.OH + oy0) * a.OW * a.N;
#pragma unroll
        for (int k = 0; k < WS_GT; k++) {
            const bool ok = g_px[k] < npix;
            stg[k] = *reinterpret_cast<const v4i *>(ok ? g0 + g_src[k] : a.G);
        }
    };
    // (what lies outside the image or past the band is replaced here: next to the loads it would wait for them)
    auto stage_store = [&](int buf, int band) {
        int8_t *xb = ws_lds + (size_t)buf * buf_bytes, *gb = xb + xbytes;
        int b, oy0, nrows;
        band_rows(band, b, oy0, nrows);
        const int iy0 = oy0 * a.stride - a.pad, npix = nrows * a.OW;
#pragma unroll
        for (int k = 0; k < WS_XT; k++) {
            if (x_row[k] < 0) continue;
            v4i v;
            if (CH == 4) {
                v = v4i{stx[k][0], stx[k][1], stx[k][2], stx[k][3]};
            } else {
                const unsigned w0 = (unsigned)stx[k][0], w1 = (unsigned)stx[k][1], w2 = (unsigned)stx[k][2];
                v[0] = (int)w0;
                v[1] = (int)__builtin_amdgcn_alignbyte(w1, w0, 3);
                v[2] = (int)__builtin_amdgcn_alignbyte(w2, w1, 2);
                v[3] = (int)(w2 >> 8);
            }
            const int iy = iy0 + x_row[k];
            if (iy < 0 || iy >= a.H) v = v4i{fill, fill, fill, fill};
            *reinterpret_cast<v4i *>(xb + x_dst[k]) = v;
            if (sa.second) *reinterpret_cast<v4i *>(xb + x_dst[k] + sa.second) = v;
        }
#pragma unroll
        for (int k = 0; k < WS_GT; k++)
            if (g_dst[k] >= 0) *reinterpret_cast<v4i *>(gb + g_dst[k]) = g_px[k] < npix ? stg[k] : v4i{0, 0, 0, 0};
    };

    v16i acc[4];
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[j][e] = 0;
    int gs = 0, xs[4] = {0, 0, 0, 0};

    const int per = (sa.nbands + gridDim.x - 1) / gridDim.x;
    const int band_begin = blockIdx.x * per, band_end = min(sa.nbands, band_begin + per);
    __syncthreads();
    if (band_begin < band_end) {
        stage_load(band_begin);
        stage_store(0, band_begin);
    }
    __syncthreads();
    // transposing read: lane l hands in the address of 8 bytes (columns 16 * grp + 8 * (j & 1) ..) of pixel row
    // half * 16 + j / 2 (and of the row 8 further down) and receives column l % 32 of the 16 pixels of its half
    const int tj = lane & 15, tgrp = (lane >> 4) & 1, thalf = lane >> 5;
    const int tcol = 16 * tgrp + 8 * (tj & 1);
    typedef LDS_PTR(int8_t) lds_bytes;
    const lds_bytes lds0 = (lds_bytes)ws_lds;
    const unsigned zero_off = 2u * (unsigned)buf_bytes + (unsigned)tcol;
    for (int band = band_begin; band < band_end; band++) {
        const int buf = (band - band_begin) & 1;
        int b, oy0, nrows;
        band_rows(band, b, oy0, nrows);
        const int npix = nrows * a.OW, nks = (npix + 31) / 32;
        if (band + 1 < band_end) stage_load(band + 1);
        const unsigned xoff = (unsigned)buf * (unsigned)buf_bytes, goff = xoff + (unsigned)xbytes;
        // fragments of k-step ks: the gradient block and the wavefront's four filter rows (rows past R read rows
        // of the buffer that exist but hold anything: their sums are dropped at the end)
        auto load_frags = [&](int ks, v4i &gf, v4i (&xf)[4]) {
            const unsigned g0 = goff + (unsigned)((ks * 32 + thalf * 16 + (tj >> 1)) * sa.gpitch + wn * 32 + tcol);
            const tr_v2i glo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(lds0 + g0));
            const tr_v2i ghi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(lds0 + g0 + 8 * sa.gpitch));
            gf = v4i{glo[0], glo[1], ghi[0], ghi[1]};
            unsigned pa[2], pstep[2];
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int px = ks * 32 + thalf * 16 + (tj >> 1) + 8 * h;
                const bool ok = px < npix;
                const unsigned q = ok ? (unsigned)px : 0u;
                const unsigned orow = hq_magic_div(q, sa.magic_OW), ox = q - orow * (unsigned)a.OW;
                // (a transposing read wants 8-byte addresses: under an odd stride the odd pixels have theirs in the second copy)
                pa[h] = ok ? xoff + (orow * (unsigned)a.stride + (unsigned)row0) * (unsigned)sa.LP + 4u * (unsigned)a.stride * ox +
                                 (ox & 1u) * (unsigned)sa.second + (unsigned)tcol
                           : zero_off;
                pstep[h] = ok ? (unsigned)sa.LP : 0u;
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const tr_v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(lds0 + pa[0] + j * pstep[0]));
                const tr_v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(lds0 + pa[1] + j * pstep[1]));
                xf[j] = v4i{lo[0], lo[1], hi[0], hi[1]};
            }
        };
        auto multiply = [&](const v4i &gf, const v4i (&xf)[4]) {
#pragma unroll
            for (int j = 0; j < 4; j++) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gf, xf[j], acc[j], 0, 0, 0);
            if (do_gsum) {
#pragma unroll
                for (int d = 0; d < 4; d++) gs = __builtin_amdgcn_sdot4(gf[d], 0x01010101, gs, false);
            }
            if (do_xsum) {
#pragma unroll
                for (int j = 0; j < 4; j++)
#pragma unroll
                    for (int d = 0; d < 4; d++) xs[j] = __builtin_amdgcn_sdot4(xf[j][d], 0x01010101, xs[j], false);
            }
        };
        // two fragment sets: the next k-step's reads are on their way while this one is multiplied
        v4i gfA, gfB, xfA[4], xfB[4];
        const int first = halves ? wk : 0, step = halves ? 2 : 1;
        if (first < nks) load_frags(first, gfA, xfA);
        for (int ks = first; ks < nks; ks += 2 * step) {
            if (ks + step < nks) load_frags(ks + step, gfB, xfB);
            multiply(gfA, xfA);
            if (ks + step >= nks) break;
            if (ks + 2 * step < nks) load_frags(ks + 2 * step, gfA, xfA);
            multiply(gfB, xfB);
        }
        if (band + 1 < band_end) stage_store(buf ^ 1, band + 1);
        __syncthreads();
    }

    // ---- flush.  G fragments were the first MFMA operand: lane l holds column l % 32 of the filter row and
    // output channels 8 * (e / 4) + 4 * (l / 32) + e % 4 of the wavefront's block.  All workgroups add to the same few lines, where
    // every request of a line queues (about 13 clocks), however few of its words it adds to: straight from the fragments, 9 or 21
    // words of a line at a time, that queue took most of a small launch.  The wavefronts' sums are put together in LDS (free
    // after the last band's barrier) and go out as whole lines, each workgroup starting elsewhere.
    const int krow = a.R * a.S * CH, words = a.N * krow;
    int *sum = reinterpret_cast<int *>(ws_lds);
    const int col = lane & 31, tap = col >> 2, ch = col & 3;
    const bool col_ok = tap < a.S && ch < CH;
    // every word belongs to one lane and is stored, not added to a cleared one; two wavefronts that share the k-steps each have a copy
    int *own = sum + (halves ? wk * words : 0);
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int r = row0 + j;
        if (r >= a.R || !col_ok) continue;
        const int wc = (r * a.S + tap) * CH + ch;
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int n = wn * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
            if (n < a.N) own[n * krow + wc] = acc[j][e];
        }
        if (do_xsum) {
            const int s = xs[j] + __shfl_xor(xs[j], 32);
            if (lane < 32 && s != 0) atomicAdd(a.xsum + wc, s);
        }
    }
    if (do_gsum) {
        const int s = gs + __shfl_xor(gs, 32);
        const int n = wn * 32 + (lane & 31);
        if (lane < 32 && n < a.N && s != 0) atomicAdd(a.gsum + n, s);
    }
    __syncthreads();
    const int chunks = (words + HQ_THREADS - 1) / HQ_THREADS;
    int q = (int)(blockIdx.x % (unsigned)chunks) * HQ_THREADS + tid;
    for (int k = 0; k < chunks; k++) {
        const int v = q < words ? sum[q] + (halves ? sum[words + q] : 0) : 0;
        if (v != 0) atomicAdd(a.acc + q, v);
        q += HQ_THREADS;
        if (q >= chunks * HQ_THREADS) q -= chunks * HQ_THREADS;
    }
}

// ---------------------------------------------------------------------------------------
// 1x1 and linear layers of a few blocks of 32 x 32 weights (channel counts multiples of 32, unit stride): a stream of pixels.  All of G_W fits
// one wavefront's accumulators, so every wavefront works alone: 32 pixels of both operands, two pieces of memory, go straight into its own LDS (two
// buffers, the next pixels on their way while these are multiplied) and are read transposed; a pixel is fetched once, and there is no
// barrier before the end, where a workgroup puts its sums together in LDS and adds them to the accumulator as whole lines.
// Whole call, 64 x 64 tiles behind a barrier per 64 pixels / this (us): 401,408 pixels 32 -> 192 (90 MB: 16 at the rate of a copy; about 5 are the
// clearing and the scaling) 29.0 / 22.5, 192 -> 32 29.5 / 21.8, 64 -> 64 27.4 / 16.3; 1,254,400 32 -> 32 50.6 / 19.1; 25,088 64 -> 64 19.0 / 9.1.
template <int CT, int NT>
__global__ __launch_bounds__(WP_THREADS, 2) void hq_wgrad_point_kernel(const WgradArgs a)
{
    constexpr int C = 32 * CT, N = 32 * NT, BUF = 32 * (C + N), WAVES = WP_THREADS / 64, WORDS = C * N + C + N;
    extern __shared__ __attribute__((aligned(16))) int8_t wp_lds[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int all = (a.M + 31) / 32;
    const int begin = (int)((long)all * blockIdx.x / gridDim.x), end = (int)((long)all * (blockIdx.x + 1) / gridDim.x);
    int8_t *mine = wp_lds + 2 * BUF * wave;
    const unsigned lds0 = hq_lds_address(mine);
    // pixels past the last are zeros in both operands
    auto load = [&](int buf, int block) __attribute__((always_inline)) {
        const int left = a.M - 32 * block;
#pragma unroll
        for (int j = 0; j < CT + NT; j++) {
            const bool x = j < CT;
            const int at = 1024 * (x ? j : j - CT) + 16 * lane;
            const int8_t *src = (x ? a.X + (size_t)block * (32 * C) : a.G + (size_t)block * (32 * N)) + at;
            if (left < 32 && at / (x ? C : N) >= left) src = reinterpret_cast<const int8_t *>(hq_fill_rows.w[0]);
            hq_lds_load16(src, lds0 + BUF * buf + 1024 * j);
        }
    };
    v16i acc[NT][CT];
    int gs[NT], xs[CT];
#pragma unroll
    for (int n = 0; n < NT; n++)
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[n][c][e] = 0;
#pragma unroll
    for (int n = 0; n < NT; n++) gs[n] = 0;
#pragma unroll
    for (int c = 0; c < CT; c++) xs[c] = 0;
    const bool do_gsum = a.xq->zero_point != 0, do_xsum = a.gq->zero_point != 0;      // (a sum is only multiplied by the other's zero point)
    int block = begin + wave, buf = 0;
    if (block < end) load(0, block);
    for (; block < end; block += WAVES, buf ^= 1) {
        if (block + WAVES < end) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // the buffer's last reads are done
            load(buf ^ 1, block + WAVES);
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(CT + NT) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        const int8_t *xb = mine + BUF * buf, *gb = xb + 32 * C;
        v4i xf[CT], gf[NT];
#pragma unroll
        for (int c = 0; c < CT; c++) xf[c] = hq_read_frag_tr<C>(xb + 32 * c, lane);
#pragma unroll
        for (int n = 0; n < NT; n++) gf[n] = hq_read_frag_tr<N>(gb + 32 * n, lane);
#pragma unroll
        for (int n = 0; n < NT; n++)
#pragma unroll
            for (int c = 0; c < CT; c++) acc[n][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gf[n], xf[c], acc[n][c], 0, 0, 0);
        if (do_gsum)
#pragma unroll
            for (int n = 0; n < NT; n++)
#pragma unroll
                for (int d = 0; d < 4; d++) gs[n] = __builtin_amdgcn_sdot4(gf[n][d], 0x01010101, gs[n], false);
        if (do_xsum)
#pragma unroll
            for (int c = 0; c < CT; c++)
#pragma unroll
                for (int d = 0; d < 4; d++) xs[c] = __builtin_amdgcn_sdot4(xf[c][d], 0x01010101, xs[c], false);
    }

    // ---- the wavefronts' sums: [N][C], [N], [C] in LDS, over the buffers.  Lane l holds column l % 32 of the input block and output
    // channels 8 * (e / 4) + 4 * (l / 32) + e % 4.
    __syncthreads();
    int *sum = reinterpret_cast<int *>(wp_lds);
    for (int i = tid; i < WORDS; i += WP_THREADS) sum[i] = 0;
    __syncthreads();
    const int half = lane >> 5, r32 = lane & 31;
#pragma unroll
    for (int n = 0; n < NT; n++) {
#pragma unroll
        for (int c = 0; c < CT; c++)
#pragma unroll
            for (int e = 0; e < 16; e++) atomicAdd(sum + (32 * n + 8 * (e >> 2) + 4 * half + (e & 3)) * C + 32 * c + r32, acc[n][c][e]);
        if (do_gsum) atomicAdd(sum + N * C + 32 * n + r32, gs[n]);
    }
    if (do_xsum)
#pragma unroll
        for (int c = 0; c < CT; c++) atomicAdd(sum + N * C + N + 32 * c + r32, xs[c]);
    __syncthreads();
    // (every workgroup starts elsewhere: all add to the same lines)
    constexpr int chunks = (C * N + WP_THREADS - 1) / WP_THREADS;
    int q = (int)(blockIdx.x % (unsigned)chunks) * WP_THREADS + tid;
    for (int k = 0; k < chunks; k++) {
        const int v = q < C * N ? sum[q] : 0;
        if (v != 0) atomicAdd(a.acc + q, v);
        q += WP_THREADS;
        if (q >= chunks * WP_THREADS) q -= chunks * WP_THREADS;
    }
    if (do_gsum && tid < N && sum[C * N + tid] != 0) atomicAdd(a.gsum + tid, sum[C * N + tid]);
    if (do_xsum && tid < C && sum[C * N + N + tid] != 0) atomicAdd(a.xsum + tid, sum[C * N + N + tid]);
}

template <int CT, int NT> bool wp_launch(const WgradArgs &a, int blocks, hipStream_t stream)
{
    constexpr int C = 32 * CT, N = 32 * NT;
    constexpr size_t lds = std::max((size_t)(WP_THREADS / 64) * 2 * 32 * (C + N), 4 * (size_t)(C * N + C + N));
    static_assert(lds <= 156 * 1024 && C <= WP_THREADS && N <= WP_THREADS, "the buffers fit, a thread to a column sum");
    static std::atomic<unsigned long long> allowed{0};
    auto kern = hq_wgrad_point_kernel<CT, NT>;
    if (!hq_allow_lds(kern, lds, allowed)) return false;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(WP_THREADS), lds, stream, a);
    return true;
}

// ---------------------------------------------------------------------------------------
__global__ void zero_kernel(int32_t *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0;
}

// Removes the zero points (32-bit wrap-around arithmetic is exact as long as the true
// result fits 32 bits) and applies the one FP32 scale.
__global__ void wgrad_finalize_kernel(const int32_t *acc, const int32_t *gsum, const int32_t *xsum,
                                      const hq_qparams *xq, const hq_qparams *gq, unsigned M, int N, int K,
                                      int gsum_per_k, float *dW, int32_t *dW_acc, const HqRideAlong ride)
{
    if (hq_ride_along(ride)) return;
    const unsigned zx = (unsigned)xq->zero_point, zg = (unsigned)gq->zero_point;
    const float s = __fmul_rn(xq->scale, gq->scale);
    const size_t total = (size_t)N * K;
    const unsigned nblocks = ride.n ? (unsigned)ride.first : gridDim.x;       // workgroups doing this kernel's own work
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)nblocks * blockDim.x) {
        const int n = (int)(i / K), k = (int)(i % K);
        const unsigned g = (unsigned)gsum[gsum_per_k ? k % gsum_per_k : n];
        unsigned c = (unsigned)acc[i] - zx * g - zg * (unsigned)xsum[k] + M * zx * zg;
        if (dW_acc) dW_acc[i] = (int)c;
        dW[i] = __fmul_rn(s, (float)(int)c);
    }
}


size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

} // namespace

// Workspace: [Cout][K] integer sums, [Cout] and [K] column sums; or the band kernel's partial sums in their place.
size_t hq_wgrad_workspace_bytes(const hq_problem *p)
{
    const size_t K = (size_t)p->R * p->S * p->C;
    if (p->kind == HQ_DEPTHWISE) return align16(4 * K) + align16(4 * (size_t)p->C) + align16(4 * K);
    if (const size_t band = hq_wgrad_band_bytes(p)) return band;
    return align16(4 * (size_t)p->Cout * K) + align16(4 * (size_t)p->Cout) + align16(4 * K);
}

int hq_launch_wgrad(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                    const hq_qparams *gq, float *dW, int32_t *dW_acc, void *ws, hipStream_t stream,
                    const HqRideAlong *ride)
{
    HqRideAlong ra = {nullptr, nullptr, 0, 0};
    if (ride) ra = *ride;
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    const size_t K = (size_t)p->R * p->S * p->C;
    WgradArgs a;
    a.X = X; a.G = dY; a.xq = xq; a.gq = gq;
    char *w = static_cast<char *>(ws);
    a.acc = reinterpret_cast<int32_t *>(w);
    const size_t acc_bytes = align16(4 * (size_t)p->Cout * K);
    a.gsum = reinterpret_cast<int32_t *>(w + acc_bytes);
    a.xsum = reinterpret_cast<int32_t *>(w + acc_bytes + align16(4 * (size_t)p->Cout));
    const size_t sums_bytes = acc_bytes + align16(4 * (size_t)p->Cout) + align16(4 * K);
    a.M = p->B * OH * OW; a.N = p->Cout; a.C = p->C;
    a.R = p->R; a.S = p->S; a.H = p->H; a.W = p->W; a.OH = OH; a.OW = OW; a.stride = p->stride; a.pad = p->pad;
    a.g16 = (a.N % 16) == 0; a.x16 = (a.C % 16) == 0;
    a.magic_ok = (unsigned long long)a.M * (unsigned long long)(OW > OH ? OW : OH) < (1ull << 32);   // hq_magic_div's range
    a.magic_OW = a.magic_ok ? hq_magic32((unsigned)OW) : 0u;
    a.magic_OH = a.magic_ok ? hq_magic32((unsigned)OH) : 0u;

    const int rc = hq_try_launch_wgrad_small(p, X, xq, dY, gq, dW, dW_acc, stream, ride);
    if (rc != HQ_E_BADSHAPE) return rc;
    const int rc_band = hq_try_launch_wgrad_band(p, X, xq, dY, gq, dW, dW_acc, ws, stream, ride);
    if (rc_band != HQ_E_BADSHAPE) return rc_band;

    // first layers: input rows staged in LDS (hq_wgrad_stem_kernel)
    if ((a.C == 3 || a.C == 4) && p->W % 4 == 0 && p->S <= 8 && p->R <= 8 && a.N <= 64 &&
        a.N % 16 == 0 && (reinterpret_cast<uintptr_t>(X) & 3) == 0 && (reinterpret_cast<uintptr_t>(dY) & 15) == 0) {
        WstemArgs sa;
        sa.w = a;
        sa.w.direct = 0;
        const int copies = p->stride % 2 ? 2 : 1, frows = p->R <= 4 ? 4 : 8;
        const int lp_reads = 4 * (OW - 1) * p->stride + 32 + 4 * (copies - 1), lp_image = 4 * (p->W + p->pad) + 4 * (copies - 1);
        sa.LP = ((lp_reads > lp_image ? lp_reads : lp_image) + 15) & ~15;
        sa.groups = p->W / 4;
        sa.magic_groups = hq_magic32((unsigned)sa.groups);
        sa.magic_OW = hq_magic32((unsigned)OW);
        const int nb32 = (a.N + 31) / 32;
        sa.gpitch = nb32 * 32 + 32;
        sa.gchunks = nb32 * 2;
        int rows = 0;
        for (int r = 1; r <= OH; r++) {
            const int in_rows = (r - 1) * p->stride + p->R, kpad = (r * OW + 31) / 32 * 32;
            if ((size_t)copies * ((r - 1) * p->stride + frows) * sa.LP + (size_t)kpad * sa.gpitch > 39 * 1024 || in_rows * sa.groups > WS_XT * HQ_THREADS ||
                kpad * sa.gchunks > WS_GT * HQ_THREADS)
                break;
            rows = r;
        }
        // Small launches: bands short enough for 64 workgroups, since one's bands are a serial chain; more of them only add their sums to the
        // same lines (7x7 stride 2 x 3, whole call, bands of as many rows as fit / for 64 workgroups: one image of 32 x 32 -> 32 12.9 /
        // 11.2 us, six -> 64 14.9 / 12.9, 16 of 64 x 64 15.2 / 15.2; for 24 / 64 / 96 workgroups, two of 64 x 64 -> 32 11.7 / 11.2 / 11.2).
        rows = std::min(rows, (int)(((long)p->B * OH + 63) / 64));
        // Sums of 56 KB and more over few pixels: the kernel with packed columns has less to add up (this / that, 8x8 x 4 -> 64: one image
        // of 32 x 32 15.8 / 14.2 us, four 16.5 / 15.1, eight 16.9 / 18.5; stride 2, four of 64 x 64 16.5 / 15.1, 16 17.5 / 28.8; 7x7 x 4,
        // 49 KB, one image 14.1 / 14.3; 8x8 x 3, 48 KB, 14.3 / 14.7).
        if ((size_t)a.N * K >= 14336 && a.M < 6000) rows = 0;
        if (rows >= 1 && (unsigned long long)p->B * OH * OW < (1ull << 31)) {
            sa.rows_out = rows;
            sa.in_rows = (rows - 1) * p->stride + p->R;
            sa.xrows = (rows - 1) * p->stride + frows;
            sa.second = copies == 2 ? sa.xrows * sa.LP + 4 : 0;
            sa.kpad = (rows * OW + 31) / 32 * 32;
            sa.bands_per_image = (OH + rows - 1) / rows;
            sa.nbands = p->B * sa.bands_per_image;
            const size_t lds = std::max(2 * ((size_t)copies * sa.xrows * sa.LP + (size_t)sa.kpad * sa.gpitch) + 64,
                                        (p->R <= 4 ? 8 : 4) * (size_t)a.N * K);
            static std::atomic<unsigned long long> allowed[2];
            if (!hq_allow_lds(hq_wgrad_stem_kernel<3>, 80 * 1024, allowed[0]) || !hq_allow_lds(hq_wgrad_stem_kernel<4>, 80 * 1024, allowed[1]))
                return HQ_E_HIP;
            const size_t zwords = sums_bytes / 4;
            hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((zwords + 255) / 256 > 1024 ? 1024 : (zwords + 255) / 256)),
                               dim3(256), 0, stream, a.acc, zwords);
            const int sblocks = sa.nbands < 512 ? sa.nbands : 512;
            if (a.C == 3) hipLaunchKernelGGL(hq_wgrad_stem_kernel<3>, dim3(sblocks), dim3(HQ_THREADS), lds, stream, sa);
            else          hipLaunchKernelGGL(hq_wgrad_stem_kernel<4>, dim3(sblocks), dim3(HQ_THREADS), lds, stream, sa);
            const size_t total = (size_t)a.N * K;
            unsigned fb = (unsigned)((total + 255) / 256 > 2048 ? 2048 : (total + 255) / 256);
            ra.first = (int)fb;
            hipLaunchKernelGGL(wgrad_finalize_kernel, dim3(fb + (unsigned)ra.n), dim3(256), 0, stream, a.acc, a.gsum, a.xsum,
                               xq, gq, (unsigned)a.M, a.N, (int)K, 0, dW, dW_acc, ra);
            return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
        }
    }

    // 1x1 and linear layers whose G_W is at most eight blocks of 32 x 32 (hq_wgrad_point_kernel), of six and more from the number of pixels on at which the
    // longer end is paid for.  In tiles / here, us: 2 x 3 and 2 x 4 blocks or six in a row 16,384 pixels (192 -> 32 10.5 / 10.1, 32 -> 192 10.3 / 10.5, 64 -> 128 16.1 /
    // 11.4), seven 65,536 (32 -> 224 13.6 / 13.5, 401,408 30.9 / 24.4; 32,768 11.1 / 11.8, 10,989 9.2 / 11.0), eight 100,000 (100,352 x 256 -> 32 16.7 / 15.7,
    // 401,408 32.7 / 26.6; 65,536 13.7 / 14.7).
    const int cb = a.C / 32, nb = a.N / 32;
    const int least = cb * nb < 6 ? 0 : cb + nb <= 7 ? 16384 : cb + nb == 8 ? 65536 : 100000;
    if (p->R == 1 && p->S == 1 && p->stride == 1 && p->pad == 0 && a.C % 32 == 0 && a.N % 32 == 0 && cb * nb <= 8 && a.M >= least &&
        ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(dY)) & 15) == 0 && a.M < (1 << 30)) {
        const size_t zwords = sums_bytes / 4;
        hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((zwords + 255) / 256 > 1024 ? 1024 : (zwords + 255) / 256)), dim3(256), 0, stream, a.acc, zwords);
        // Half the compute units bring what memory gives, and every workgroup's sums queue at the same lines: 401,408 x 64 -> 64 16.3 us
        // in 128 workgroups, 17.8 in 192, 19.1 in 256; a wavefront gets four blocks of pixels, two where there are few (100,352 x 32 -> 192 13.0,
        // with one 16.3).
        const int all = (a.M + 31) / 32, blocks = std::max(1, std::min(128, std::max(all / 32, std::min(all / 16, 64))));
        bool ok = false;
        switch (16 * cb + nb) {
#define WP(c, n) case 16 * c + n: ok = wp_launch<c, n>(a, blocks, stream); break
        WP(1, 1); WP(1, 2); WP(1, 3); WP(1, 4); WP(1, 5); WP(1, 6); WP(2, 1); WP(2, 2);
        WP(1, 7); WP(1, 8); WP(2, 3); WP(2, 4); WP(3, 1); WP(3, 2); WP(4, 1); WP(4, 2);
        WP(5, 1); WP(6, 1); WP(7, 1); WP(8, 1);
#undef WP
        }
        if (!ok) return HQ_E_HIP;
        const size_t total = (size_t)a.N * K;
        const unsigned fb = (unsigned)((total + 255) / 256);
        ra.first = (int)fb;
        hipLaunchKernelGGL(wgrad_finalize_kernel, dim3(fb + (unsigned)ra.n), dim3(256), 0, stream, a.acc, a.gsum, a.xsum,
                           xq, gq, (unsigned)a.M, a.N, (int)K, 0, dW, dW_acc, ra);
        return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
    }

    const bool big = a.N > 64 && a.C > 64, packed = a.C < 16;
    const int TN = big ? 128 : 64, TK = packed ? 256 : big ? 128 : 64;
    a.ctiles = (a.C + TK - 1) / TK;
    // (3-channel inputs: 32 tile columns per filter row)
    const int xt = a.C == 3 ? (p->R * 32 + TK - 1) / TK : packed ? (int)((K + TK - 1) / TK) : p->R * p->S * a.ctiles;
    const int yt = (a.N + TN - 1) / TN;
    const int stages_total = (a.M + MB - 1) / MB;
    // Workgroups to aim at.  Small tiles need many resident workgroups to hide their stage latency;
    // 128x128 tiles carry 64 KB of atomics each, and those queue on the same lines when every split
    // finishes at once, so they get longer runs of pixels and fewer splits.
    // (first layers: three resident workgroups per compute unit; more splits only add atomics: 256 against 283 us
    // on the 7x7 stride-2 stem at batch 256)
    const int target = packed ? 768 : !big ? 2048 : p->R * p->S == 1 ? 256 : 512;
    int splits = (target + xt * yt - 1) / (xt * yt);
    if (splits > stages_total) splits = stages_total;
    // (a run shorter than about ten stages is mostly start-up and atomics: a 1x1 stride-2 layer 64 -> 128 at
    // 28x28 outputs, batch 256, takes 26 us with runs of 12 stages against 42 us with runs of 3)
    if (!big && !packed && splits > stages_total / 10) {
        const int fill = (512 + xt * yt - 1) / (xt * yt);          // but keep two workgroups per compute unit
        splits = stages_total / 10 > fill ? stages_total / 10 : splits < fill ? splits : fill;
    }
    if (splits < 1) splits = 1;
    const int stages_per = (stages_total + splits - 1) / splits;
    a.m_per_split = stages_per * MB;
    splits = (stages_total + stages_per - 1) / stages_per;
    a.xt = xt; a.yt = yt; a.splits = splits;
    // one split: the tiles partition [N][K], so the sums are stored, not added, and only the column sums start at zero
    a.direct = splits == 1 && !packed;
    int32_t *zero_from = a.direct ? a.gsum : a.acc;
    const size_t ws_words = (a.direct ? sums_bytes - acc_bytes : sums_bytes) / 4;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((ws_words + 255) / 256 > 1024 ? 1024 : (ws_words + 255) / 256)),
                       dim3(256), 0, stream, zero_from, ws_words);
    dim3 grid((unsigned)(xt * yt * splits));
    if (a.C == 3) hipLaunchKernelGGL((hq_wgrad_kernel<64, 256, true, true>), grid, dim3(HQ_THREADS), 0, stream, a);
    else if (packed) hipLaunchKernelGGL((hq_wgrad_kernel<64, 256, true>), grid, dim3(HQ_THREADS), 0, stream, a);
    else if (a.g16 && a.x16 && a.magic_ok) {
        if (big) hipLaunchKernelGGL((hq_wgrad_kernel<128, 128, false, false, true>), grid, dim3(HQ_THREADS), 0, stream, a);
        else     hipLaunchKernelGGL((hq_wgrad_kernel<64, 64, false, false, true>), grid, dim3(HQ_THREADS), 0, stream, a);
    }
    else if (big) hipLaunchKernelGGL((hq_wgrad_kernel<128, 128, false>), grid, dim3(HQ_THREADS), 0, stream, a);
    else          hipLaunchKernelGGL((hq_wgrad_kernel<64, 64, false>), grid, dim3(HQ_THREADS), 0, stream, a);

    const size_t total = (size_t)a.N * K;
    unsigned fb = (unsigned)((total + 255) / 256 > 2048 ? 2048 : (total + 255) / 256);
    ra.first = (int)fb;
    hipLaunchKernelGGL(wgrad_finalize_kernel, dim3(fb + (unsigned)ra.n), dim3(256), 0, stream, a.acc, a.gsum, a.xsum, xq, gq,
                       (unsigned)a.M, a.N, (int)K, 0, dW, dW_acc, ra);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}
