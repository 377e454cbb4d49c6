// Gather GEMM of whole 128-channel lines: hq_gemm_fwd (any stride), hq_gemm_dgrad of stride 1 and pass 1 of the dynamic baseline
// where the reduced channels are a multiple of 128.
//
//   out[m][n] = sum_{tap,c} A[pix(m,tap)][c] * Bw[n][tap][c]    (weight taps mirrored for the input gradient)
//
// A workgroup of eight wavefronts owns 128 pixels x 128 channels and reduces 128 bytes per stage: one tap and one line of every pixel
// and every filter, so the tap is the same for the whole workgroup and its bookkeeping is scalar.  Two stages of 32 KB, filled by
// direct-to-LDS loads; two workgroups to a compute unit.  What bounded the kernel with 256 threads on these layers was a wavefront's
// own chain of instructions between two barriers (18 vector instructions per MFMA and a wait for all loads at the end of every
// stage: 3.2 K cycles for 1 K of matrix work).  Here a wavefront takes half of a stage's k-steps for a 64 x 64 block (the two halves
// are added through LDS once), a stage is 8 MFMAs and about 40 other instructions, dealt out between the MFMAs: fragments of the
// next k-step are read, the loads of the stage after next are worked out and requested while one is carried out.
//
// Measured (with the kernels before / with this one): 3x3 stride 2 on 256 x 28 x 28 x 128 -> 256 30.2 / 26.1 us, 5x5 on
// 64 x 28 x 28 x 128 -> 128 49.6 / 28.7, linear 8192 x 4096 -> 4096 189 / 149 (1.84 POP/s); 3x3 of stride 1 and padding 1 has a kernel of its
// own (256 x 7 x 7 x 512 -> 512 37.2 us here, 32.4 there).  What bounds it now (counters of
// 4096 x 4096 x 4096, 79 us under collection): of 160 K cycles the matrix pipes are busy for 41 %, the LDS for 23 % without a conflict, and
// the path from L2 brings 28 bytes a clock of the 50 that loads alone reach; what is left is a wavefront's 14 other instructions
// per MFMA, in order, and its wait at the stage's barrier.  On random bytes the clock is 2.0 GHz: with all operands 0 the same cycles
// take 62 us.  Three or four stages with one workgroup per compute unit were slower wherever there is more than one tile for it
// (3x3 on 256 x 14 x 14 x 256: 55 us against 44), and four wavefronts with all k-steps each where there is one (8 x 8 x 512: 29 us
// against 25).
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int RG_THREADS = 512, RG_BM = 128, RG_BN = 128, RG_BK = 128;   // tile, bytes of the reduction per stage
constexpr int RG_STAGE = (RG_BM + RG_BN) * RG_BK;

struct RingArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, N;                      // output pixels, channels
    int Cs, nst;                   // reduced channels per tap; stages: taps * Cs / 128
    int ns;                        // taps per filter row
    int Hs, Ws, Ho, Wo;            // source image, output image
    int istep, pad;                // source pixel = istep * y - pad + tap row
    int w0, wr, wc;                // weight tap = w0 + wr * tap row + wc * tap column (mirrored: from the last one down)
    unsigned wrow;                 // bytes per weight row
    unsigned magic_Wo, magic_Ho;
    int m_tiles, n_tiles;
    HqSr sr;
};

template <int MODE>
__global__ __launch_bounds__(RG_THREADS, 4) void hq_ring_kernel(const RingArgs a)
{
    constexpr int NT = RG_THREADS, NW = NT / 64, L = 16 / NW;            // loads per operand and stage
    static_assert(L == 2, "a stage has four places for its loads");
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    __shared__ int red[4 * NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, r32 = lane & 31;
    const int group = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;    // share of every stage; 64 x 64 block of the tile

    // consecutive workgroups go to the 8 XCDs in turn: each XCD gets a run of tiles, channel blocks of the same pixels together
    int tile = blockIdx.x;
    const int per = a.m_tiles * a.n_tiles / 8;
    if (tile < per * 8) tile = (tile & 7) * per + (tile >> 3);
    // (in bands of 8 pixel tiles, so that the 64 workgroups of an XCD share 16 operand panels, not 2 + 32)
    int tile_m, tile_n;
    if (a.n_tiles > 8) {
        const int band = tile / (8 * a.n_tiles), rows = min(8, a.m_tiles - 8 * band), r = tile - band * 8 * a.n_tiles;
        tile_n = r / rows; tile_m = 8 * band + r - tile_n * rows;
    } else { tile_m = tile / a.n_tiles; tile_n = tile - tile_m * a.n_tiles; }
    const int m0 = tile_m * RG_BM, n0 = tile_n * RG_BN;

    const int za = a.aq->zero_point;
    const int8_t *fill = reinterpret_cast<const int8_t *>(hq_fill_rows.w[za & 0xff]);

    // ---- loads: blocks of 8 rows, whole 128-byte lines; lane l lands at 16 * l, the chunks of a row are XOR-swizzled by the row
    const int8_t *arow[L], *aptr[L];
    int ay[L], ax[L];
    unsigned boff[L];
#pragma unroll
    for (int k = 0; k < L; k++) {
        const int row = 8 * (NW * k + wave) + (lane >> 3), chunk = (lane & 7) ^ ((row >> 1) & 7);
        const unsigned m = (unsigned)min(m0 + row, a.M - 1);             // (rows past the end repeat the last; never stored)
        const unsigned t = hq_magic_div(m, a.magic_Wo), b = hq_magic_div(t, a.magic_Ho);
        ay[k] = (int)(t - b * (unsigned)a.Ho) * a.istep - a.pad;
        ax[k] = (int)(m - t * (unsigned)a.Wo) * a.istep - a.pad;
        arow[k] = a.A + ((ptrdiff_t)((ptrdiff_t)b * a.Hs + ay[k]) * a.Ws + ax[k]) * a.Cs + 16 * chunk;
        const int n = n0 + (row & ~31) + hq_sigma32(row & 31);
        boff[k] = (unsigned)(n < a.N ? n : 0) * a.wrow + 16u * (unsigned)chunk;
    }
    int lc = 0, ltr = 0, lts = 0;                                        // channel and tap of the next stage to load
    const unsigned lds0 = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(size_t)(__attribute__((address_space(3))) void *)smem) + wave * 1024;
    auto locate = [&](int k) __attribute__((always_inline)) {
        const bool in = (unsigned)(ay[k] + ltr) < (unsigned)a.Hs && (unsigned)(ax[k] + lts) < (unsigned)a.Ws;
        aptr[k] = in ? arow[k] + ((ltr * a.Ws + lts) * a.Cs + lc) : fill;
    };
    const int8_t *wb;
    auto advance = [&]() __attribute__((always_inline)) {
        wb = a.Bw + (ptrdiff_t)((a.w0 + ltr * a.wr + lts * a.wc) * a.Cs + lc);
        lc += RG_BK;
        const bool tap_done = lc == a.Cs, row_done = tap_done && lts + 1 == a.ns;
        lc = tap_done ? 0 : lc;
        lts = row_done ? 0 : tap_done ? lts + 1 : lts;
        ltr += row_done ? 1 : 0;
    };
    // (two stages ahead, and never fewer than two: the launcher takes 8 stages or more)
    for (int d = 0; d < 2; d++) {
#pragma unroll
        for (int k = 0; k < L; k++) locate(k);
        advance();
#pragma unroll
        for (int k = 0; k < L; k++) {
            hq_lds_load16(aptr[k], lds0 + d * RG_STAGE + 8192 * k);
            hq_lds_load16(wb, boff[k], lds0 + d * RG_STAGE + RG_BM * RG_BK + 8192 * k);
        }
    }

    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {1.0f, 0.0f, 0.0f, 0.0f, true};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);
    // the wavefront's own outputs: after the two halves of the reduction are added, 32 pixels x 64 channels
    v16i acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) acc[i][j][e] = 0;

    int foff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ks++) foff[ks] = r32 * RG_BK + 16 * ((2 * (2 * group + ks) + half) ^ ((r32 >> 1) & 7));
    v4i wf[2][2], af[2][2];
    auto fragments = [&](int buf, int ks) __attribute__((always_inline)) {
        const int8_t *Ab = smem + buf * RG_STAGE + wm * 64 * RG_BK + foff[ks], *Bb = smem + buf * RG_STAGE + (RG_BM + wn * 64) * RG_BK + foff[ks];
        wf[ks][0] = *reinterpret_cast<const v4i *>(Bb);
        af[ks][0] = *reinterpret_cast<const v4i *>(Ab);
        wf[ks][1] = *reinterpret_cast<const v4i *>(Bb + 32 * RG_BK);
        af[ks][1] = *reinterpret_cast<const v4i *>(Ab + 32 * RG_BK);
    };
    // one MFMA, and a line across which nothing moves: what stands between two of them runs while the first is carried out
    auto multiply = [&](int ks, int i, int j) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * L) : "memory");
    __syncthreads();
    fragments(0, 0);
    int cur = 0;
    // `more`: stage s + 2 exists; `next`: stage s + 1 does
    auto stage = [&](auto more, auto next) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more)::value, NEXT = decltype(next)::value;
        fragments(cur, 1);
        multiply(0, 0, 0);
        if (MORE) locate(0);
        multiply(0, 0, 1);
        if (MORE) locate(1);
        multiply(0, 1, 0);
        if (MORE) advance();
        multiply(0, 1, 1);
        const unsigned dst = lds0 + cur * RG_STAGE;
        if (NEXT) {
            // All fragments of this stage are in registers at the barrier: its buffer takes stage s + 2.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            cur ^= 1;
            fragments(cur, 0);
        }
        multiply(1, 0, 0);
        if (MORE) hq_lds_load16(aptr[0], dst);
        multiply(1, 0, 1);
        if (MORE) hq_lds_load16(aptr[1], dst + 8192);
        multiply(1, 1, 0);
        if (MORE) hq_lds_load16(wb, boff[0], dst + 16384);
        multiply(1, 1, 1);
        if (MORE) hq_lds_load16(wb, boff[1], dst + 24576);
    };
    for (int s = 2; s < a.nst; s++) stage(std::true_type(), std::true_type());
    stage(std::false_type(), std::true_type());
    stage(std::false_type(), std::false_type());

    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    // 32 pixels x 64 channels: 16 consecutive channels of a pixel per lane and j
    auto finish = [&](auto full, int i) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        const int m = m0 + 64 * wm + 32 * i + r32;
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const int nb = n0 + 64 * wn + 32 * j + 16 * half;
            if (m >= a.M || nb >= a.N) continue;                         // N % 16 == 0
            int c[16];
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const v4i bz = *reinterpret_cast<const v4i *>(a.bsum + nb + 4 * g);
                const v4i v = reinterpret_cast<const v4i *>(smem)[(wave * 8 + 4 * j + g) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; e++) c[4 * g + e] = (i ? acc[1][j][4 * g + e] : acc[0][j][4 * g + e]) + v[e] - za * bz[e];
            }
            const size_t o = (size_t)m * a.N + nb;
            if constexpr (MODE == 0) {
                hq_minmax_group<16>(c, mn, mx);
#pragma unroll
                for (int g = 0; g < 4; g++) *reinterpret_cast<v4i *>(a.out32 + o + 4 * g) = v4i{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
            } else {
                int w[4];
                if constexpr (MODE == 2) hq_requant_group_sr<16, FULL, 16>(c, ep, a.sr, o, mn, mx, nlo, nhi, w);
                else                     hq_requant_group<16, FULL>(c, ep, mn, mx, nlo, nhi, w);
                *reinterpret_cast<v4i *>(a.out8 + o) = v4i{w[0], w[1], w[2], w[3]};
            }
        }
    };
    {
        // the two shares are added through LDS: group 0 finishes the first 32 pixels of a block, group 1 the others
        __syncthreads();
        v4i *x = reinterpret_cast<v4i *>(smem);                          // [8 wavefronts][8][64]
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int g = 0; g < 4; g++) {
                v4i v;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = group ? acc[0][j][4 * g + e] : acc[1][j][4 * g + e];
                x[((wave ^ 4) * 8 + 4 * j + g) * 64 + lane] = v;
            }
        __syncthreads();
    }
    auto epilogue = [&](auto full) __attribute__((always_inline)) {
        finish(full, group);
    };
    if (MODE == 0 || ep.full_grid) epilogue(std::true_type()); else epilogue(std::false_type());
    hq_block_stats_commit_n<NT>(mn, mx, nlo, nhi, a.st, red);
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.N);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

template <int MODE> int launch(const RingArgs &a, hipStream_t s)
{
    const size_t lds = 2 * RG_STAGE;                                     // (also the 64 KB of the partial sums)
    static std::atomic<unsigned long long> allowed{0};
    if (!hq_allow_lds(hq_ring_kernel<MODE>, lds, allowed)) return HQ_E_HIP;
    hipLaunchKernelGGL(hq_ring_kernel<MODE>, dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(RG_THREADS), lds, s, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

} // namespace

int hq_try_launch_ring(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8, int32_t *out32,
                       hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    if (p->kind == HQ_DEPTHWISE || (dgrad && !(p->stride == 1 && p->R == p->S))) return HQ_E_BADSHAPE;
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    RingArgs a = {};
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    const int taps = p->R * p->S;
    if (!dgrad) { a.N = p->Cout; a.Cs = p->C; a.Hs = p->H; a.Ws = p->W; a.Ho = OH; a.Wo = OW; a.istep = p->stride; a.pad = p->pad; }
    else        { a.N = p->C; a.Cs = p->Cout; a.Hs = OH; a.Ws = OW; a.Ho = p->H; a.Wo = p->W; a.istep = 1; a.pad = p->R - 1 - p->pad; }
    if (a.Cs % RG_BK != 0 || a.N % 16 != 0 || a.N < 128) return HQ_E_BADSHAPE;
    const unsigned long long M = (unsigned long long)p->B * a.Ho * a.Wo, lim = 1ull << 32;
    // operands of hq_magic_div; 32-bit offsets into the weights and from a pixel's tap (0, 0)
    if (M * (unsigned)std::max(a.Ho, a.Wo) >= lim || M >= lim / 2 || (unsigned long long)a.N * taps * a.Cs >= lim ||
        (unsigned long long)(p->R + 1) * a.Ws * a.Cs >= lim / 2) return HQ_E_BADSHAPE;
    a.M = (int)M;
    a.ns = p->S; a.nst = taps * (a.Cs / RG_BK);
    a.wrow = (unsigned)taps * (unsigned)a.Cs;
    a.w0 = dgrad ? taps - 1 : 0; a.wr = dgrad ? -p->S : p->S; a.wc = dgrad ? -1 : 1;
    a.magic_Wo = hq_magic32((unsigned)a.Wo); a.magic_Ho = hq_magic32((unsigned)a.Ho);
    a.m_tiles = (a.M + RG_BM - 1) / RG_BM;
    a.n_tiles = (a.N + RG_BN - 1) / RG_BN;
    if (sr_seed && out32) return HQ_E_BADARG;
    // Short reductions do not pay for the start and for adding the two halves (1x1, this / tile kernel: 128 x 14 x 14 x 512 -> 1024, 4
    // stages 31.5 / 28.3 us; linear 8192 x 1024 -> 1024, 8 stages 14.9 / 17.9).
    if (a.nst < 8) return HQ_E_BADSHAPE;
    // At most 64 tiles: the smaller tiles of the other kernels fill more compute units (3x3 on 128 x 4 x 4 x 512 -> 512: 20.2 us, split
    // reduction 12.9).  From 65 on filters of several taps are faster here although most compute units have no tile (3x3 stride 2,
    // 58 x 16 x 16 x 128 -> 320, 87 tiles 9.0 / 10.8 us; input gradient 3 x 28 x 28 x 1024 -> 512, 76 tiles 46.3 / 51.0, with stochastic
    // rounding 26 x 14 x 14 x 640 -> 256, 80 tiles 26.0 / 31.3), also where most of the last column of tiles is empty (stride 2,
    // 11 x 56 x 56 x 128 -> 160, 136 tiles 9.2 / 11.1).
    const long tiles = (long)a.m_tiles * a.n_tiles;
    if (tiles <= 64) return HQ_E_BADSHAPE;
    // One tap: while the tile kernel holds all its 64 x 64 tiles at once, two to a compute unit, it is ahead of this kernel's longer
    // start and end, unless those weigh little: round-to-nearest-even from 10 lines on.  This / tile kernel, linear: input gradients
    // 5120 x 1024 -> 192 8.6 / 7.9 us, 4319 x 1280 -> 272 9.8 / 9.8, 640 x 3072 -> 2048 16.1 / 20.6, 12281 x 1024 -> 192 9.2 / 10.1,
    // 22528 x 1536 -> 320 26.8 / 36.6; with stochastic rounding 5120 x 1024 -> 192 10.5 / 8.4, 6016 x 1152 -> 320 11.3 / 10.3,
    // 8794 x 1280 -> 384 12.0 / 14.3; dynamic, forward, 4678 x 1024 -> 160 15.8 / 14.2, 10987 x 2560 -> 320 35.0 / 39.3.
    const long small_tiles = (long)((M + 63) / 64) * ((a.N + 63) / 64);
    if (taps == 1 && small_tiles <= 512 && (out32 || sr_seed || a.nst < 10)) return HQ_E_BADSHAPE;
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    return mode == 0 ? launch<0>(a, stream) : mode == 1 ? launch<1>(a, stream) : launch<2>(a, stream);
}
