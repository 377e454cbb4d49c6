// Weight gradients over few pixels, in one launch.  The split-K kernels need two or three (clear, sum, finalize) and the
// time of a small layer is theirs: 14 .. 16 us for layers whose operands are read in one.  Here a workgroup owns a tile
// of G_W for ALL pixels: its wavefronts share the pixels (wavefront w takes the 32-pixel steps w, w + NW, ...), each
// staging both operands' rows through LDS of its own (no barrier inside the reduction) into the transposing
// reads, and meet once, when the partial sums are added through LDS, freed of the zero points, scaled and stored.  Nothing has
// to be cleared and no atomics are needed.  The price is that every tile reads its columns of all pixels, M x (TN + TK)
// bytes at the 64 bytes a clock a compute unit loads, so the form is taken while that is short.
#include "hq_device.h"
#include "hq_internal.h"

namespace {

struct WsmallArgs {
    const int8_t *X, *G;
    const hq_qparams *xq, *gq;
    float *dW;
    int32_t *dW_acc;
    int M, N, C, taps, S, H, W, OW, OH, stride, pad;
    int ctiles, xt;                // tiles along C inside one tap; tile columns (taps * ctiles)
    int g16, x16;                  // rows of G / X are 16-byte aligned
    unsigned magic_OW, magic_OH, magic_S, magic_ctiles;
    HqRideAlong ride;
};

// 16 channels at p, of which `left` exist (a multiple of 4; nothing is read at or past them)
__device__ inline v4i load_channels(const int8_t *p, int left, bool aligned16)
{
    if (aligned16) return *reinterpret_cast<const v4i *>(p);
    v4i v;
#pragma unroll
    for (int d = 0; d < 4; d++) v[d] = 4 * d < left ? *reinterpret_cast<const int *>(p + 4 * d) : 0;
    return v;
}

// NB x KB: 32-channel blocks of dY and of the input.
template <int NB, int KB, int NW, int D>
__global__ __launch_bounds__(NW * 64) void hq_wgrad_small_kernel(const WsmallArgs a)
{
    constexpr int TN = 32 * NB, TK = 32 * KB;
    constexpr int PG = NB == 1 ? 32 : TN + 32, PX = KB == 1 ? 32 : TK + 32;     // LDS pitches (32 mod 64: transposing reads)
    constexpr int STAGE = 32 * (PG + PX);                                       // bytes of a wavefront's stage
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    if (hq_ride_along(a.ride)) return;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    v4i *sums = reinterpret_cast<v4i *>(smem);                                  // [NW][NB * KB][4][64]
    constexpr int BUF = NW * (NB * KB * 4096 > STAGE ? NB * KB * 4096 : STAGE);
    int *gsum = reinterpret_cast<int *>(smem + BUF), *xsum = gsum + TN;         // [TN], [TK]
    int8_t *gs = smem + wave * STAGE, *xs = gs + 32 * PG;

    const int by = blockIdx.x / a.xt, bx = blockIdx.x - by * a.xt;
    const int tap = (int)hq_magic_div((unsigned)bx, a.magic_ctiles), c0 = (bx - tap * a.ctiles) * TK, n0 = by * TN;
    const int tr = (int)hq_magic_div((unsigned)tap, a.magic_S), ts = tap - tr * a.S;
    const int zx = a.xq->zero_point, zg = a.gq->zero_point;
    const int fill = (int)((unsigned)(zx & 0xff) * 0x01010101u);
    for (int i = tid; i < TN + TK; i += NW * 64) gsum[i] = 0;

    // a lane's chunks: chunk i is 16 channels of row (lane + 64 i) / (TN / 16) of the step
    auto load = [&](int step, v4i (&g)[NB], v4i (&x)[KB]) {
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const int idx = lane + 64 * i, m = 32 * step + idx / (TN / 16), n = n0 + idx % (TN / 16) * 16;
            v4i v = {0, 0, 0, 0};
            if (m < a.M && n < a.N) v = load_channels(a.G + (size_t)m * a.N + n, a.N - n, a.g16);
            g[i] = v;
        }
#pragma unroll
        for (int i = 0; i < KB; i++) {
            const int idx = lane + 64 * i, m = 32 * step + idx / (TK / 16), c = c0 + idx % (TK / 16) * 16;
            v4i v = {0, 0, 0, 0};
            if (m < a.M && c < a.C) {
                const unsigned t = hq_magic_div((unsigned)m, a.magic_OW), b = hq_magic_div(t, a.magic_OH);
                const int iy = (int)(t - b * (unsigned)a.OH) * a.stride - a.pad + tr;
                const int ix = (int)((unsigned)m - t * (unsigned)a.OW) * a.stride - a.pad + ts;
                v = v4i{fill, fill, fill, fill};
                if (iy >= 0 && iy < a.H && ix >= 0 && ix < a.W)
                    v = load_channels(a.X + (((size_t)b * a.H + iy) * a.W + ix) * a.C + c, a.C - c, a.x16);
            }
            x[i] = v;
        }
    };

    v16i acc[NB][KB];
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < KB; j++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[i][j][r] = 0;
    int gacc[NB] = {}, xacc[KB] = {};

    const int nsteps = (a.M + 31) / 32;
    v4i greg[D][NB], xreg[D][KB];
#pragma unroll
    for (int d = 0; d < D; d++) load(wave + NW * d, greg[d], xreg[d]);
    for (int s = wave; s < nsteps; s += NW * D) {
#pragma unroll
        for (int d = 0; d < D; d++) {                     // (steps past the end hold zeros)
#pragma unroll
            for (int i = 0; i < NB; i++) {
                const int idx = lane + 64 * i;
                *reinterpret_cast<v4i *>(gs + idx / (TN / 16) * PG + idx % (TN / 16) * 16) = greg[d][i];
            }
#pragma unroll
            for (int i = 0; i < KB; i++) {
                const int idx = lane + 64 * i;
                *reinterpret_cast<v4i *>(xs + idx / (TK / 16) * PX + idx % (TK / 16) * 16) = xreg[d][i];
            }
            load(s + NW * (d + D), greg[d], xreg[d]);
            __builtin_amdgcn_wave_barrier();              // (LDS serves a wavefront's accesses in order)
            v4i gf[NB], xf[KB];
#pragma unroll
            for (int i = 0; i < NB; i++) gf[i] = hq_read_frag_tr<PG>(gs + 32 * i, lane);
#pragma unroll
            for (int j = 0; j < KB; j++) xf[j] = hq_read_frag_tr<PX>(xs + 32 * j, lane);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int i = 0; i < NB; i++)
#pragma unroll
                for (int j = 0; j < KB; j++) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(gf[i], xf[j], acc[i][j], 0, 0, 0);
            if (zx != 0)
#pragma unroll
                for (int i = 0; i < NB; i++)
#pragma unroll
                    for (int e = 0; e < 4; e++) gacc[i] = __builtin_amdgcn_sdot4(gf[i][e], 0x01010101, gacc[i], false);
            if (zg != 0)
#pragma unroll
                for (int j = 0; j < KB; j++)
#pragma unroll
                    for (int e = 0; e < 4; e++) xacc[j] = __builtin_amdgcn_sdot4(xf[j][e], 0x01010101, xacc[j], false);
        }
    }
    __syncthreads();                                      // the stages make room for the partial sums
#pragma unroll
    for (int i = 0; i < NB; i++)
#pragma unroll
        for (int j = 0; j < KB; j++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                sums[((wave * NB * KB + i * KB + j) * 4 + q) * 64 + lane] =
                    v4i{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    if (zx != 0)
#pragma unroll
        for (int i = 0; i < NB; i++) atomicAdd(gsum + 32 * i + (lane & 31), gacc[i]);
    if (zg != 0)
#pragma unroll
        for (int j = 0; j < KB; j++) atomicAdd(xsum + 32 * j + (lane & 31), xacc[j]);
    __syncthreads();

    // a thread = 4 consecutive channels of dY at one input channel; G fragments were the first operand: lane l holds column
    // c = l % 32 of the block and rows n = 8 q + 4 (l / 32) + e
    const float sc = __fmul_rn(a.xq->scale, a.gq->scale);
    const unsigned both = (unsigned)a.M * (unsigned)zx * (unsigned)zg;
    const size_t krow = (size_t)a.taps * a.C;
    for (int u = tid; u < NB * KB * 256; u += NW * 64) {
        const int l = u & 63, q = (u >> 6) & 3, j = (u >> 8) % KB, i = (u >> 8) / KB;
        const int cl = 32 * j + (l & 31), nl = 32 * i + 8 * q + 4 * (l >> 5);
        if (c0 + cl >= a.C || n0 + nl >= a.N) continue;   // N % 4 == 0
        v4i v = sums[u];
#pragma unroll
        for (int w = 1; w < NW; w++) v += sums[w * (NB * KB * 256) + u];
        const v4i gv = *reinterpret_cast<const v4i *>(gsum + nl);
        const unsigned xterm = (unsigned)zg * (unsigned)xsum[cl];
        const size_t o = (size_t)(n0 + nl) * krow + (size_t)tap * a.C + c0 + cl;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const unsigned r = (unsigned)v[e] - (unsigned)zx * (unsigned)gv[e] - xterm + both;
            if (a.dW_acc) a.dW_acc[o + e * krow] = (int)r;
            a.dW[o + e * krow] = __fmul_rn(sc, (float)(int)r);
        }
    }
}

template <int NB, int KB, int NW, int D>
int launch(WsmallArgs &a, hipStream_t s)
{
    constexpr int PG = NB == 1 ? 32 : 32 * NB + 32, PX = KB == 1 ? 32 : 32 * KB + 32, STAGE = 32 * (PG + PX);
    constexpr size_t lds = (size_t)NW * (NB * KB * 4096 > STAGE ? NB * KB * 4096 : STAGE) + 4 * 32 * (NB + KB);
    a.ctiles = (a.C + 32 * KB - 1) / (32 * KB);
    a.magic_ctiles = hq_magic32((unsigned)a.ctiles);
    a.xt = a.taps * a.ctiles;
    const int blocks = a.xt * ((a.N + 32 * NB - 1) / (32 * NB));
    a.ride.first = blocks;
    auto kern = hq_wgrad_small_kernel<NB, KB, NW, D>;
    static std::atomic<unsigned long long> allowed{0};
    if (!hq_allow_lds(kern, lds, allowed)) return HQ_E_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(blocks + a.ride.n)), dim3(NW * 64), lds, s, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

} // namespace

int hq_try_launch_wgrad_small(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                              const hq_qparams *gq, float *dW, int32_t *dW_acc, hipStream_t stream, const HqRideAlong *ride)
{
    if (p->C < 16) return HQ_E_BADSHAPE;                 // (first layers: packed columns)
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    const unsigned long long M = (unsigned long long)p->B * OH * OW, lim = 1ull << 32;
    const unsigned long long kt = (unsigned long long)p->R * p->S * ((p->C + 31) / 32);
    if ((M + 1024) * (unsigned)(OH > OW ? OH : OW) >= lim || kt * ((p->C + 31) / 32) >= lim || kt * ((p->Cout + 31) / 32) >= (1u << 30))
        return HQ_E_BADSHAPE;                            // operands of hq_magic_div, workgroups
    WsmallArgs a = {};
    a.X = X; a.G = dY; a.xq = xq; a.gq = gq; a.dW = dW; a.dW_acc = dW_acc;
    a.M = (int)M; a.N = p->Cout; a.C = p->C; a.taps = p->R * p->S; a.S = p->S; a.H = p->H; a.W = p->W; a.OH = OH; a.OW = OW;
    a.stride = p->stride; a.pad = p->pad;
    a.g16 = a.N % 16 == 0; a.x16 = a.C % 16 == 0;
    a.magic_OW = hq_magic32((unsigned)OW); a.magic_OH = hq_magic32((unsigned)OH); a.magic_S = hq_magic32((unsigned)p->S);
    if (ride) a.ride = *ride;
    auto tiles = [&](int tn, int tk) { return (long)((a.N + tn - 1) / tn) * a.taps * ((a.C + tk - 1) / tk); };
    // At most 16 steps: four wavefronts have enough to do, and the store of G_W is most of the time (from 2304 tiles on
    // 64 x 64 tiles, half the reads).  More steps: as long as the tiles run side by side and each reads less than about 10 us
    // worth; beyond, the split-K kernels (a 7 x 7 x 512 layer at batch 32 23 -> 9 us, 8192 pixels under 36 tiles 16 -> 12,
    // 12544 pixels under 128 tiles 22 -> 31).  Rows off 16 bytes are read by words and reach that point earlier.
    // The time here grows with the pixels alone (8.2 us for 4700, 9.2 for 6000, 11.2 for 8000), that of the split-K kernels with
    // the work: small gradients turn over earlier (3x3 16 -> 16 at 8000 pixels 11.1 us against 9.4).  3x3 layers of unit stride whose channels are multiples
    // of 64, against the framed kernel, at 8192 pixels: 64 -> 64 11.5 / 12.9, 64 -> 256 13.2 / 15.8, 128 -> 128 15.2 / 15.6, 64 -> 448 16.9 / 18.4; at 9016 128 -> 128
    // 17.1 / 15.7, 64 -> 256 14.3 / 15.9.  Of 594 such layers those past 200 tiles and 6300 pixels are on the wrong side, by up to 9 % (192 -> 128 at 8192
    // 19.1 / 17.6).
    // And every XCD reads all pixels it has a tile of, of whole 128-byte lines (with 256 channels half of them: eight tiles of
    // 32 channels, one per XCD): once they do not fit its L2 the time jumps (3x3 stride 2, 128 -> 64: 4.0 MB 10.1 us, 4.2 MB 15.9
    // against 13.1; but 96 -> 128, where the split-K kernel needs two tiles, 17.1 against 22.5).
    if (a.M <= 512) {
        if (tiles(32, 32) <= 2304) return launch<1, 1, 4, 4>(a, stream);
        return a.M <= 256 ? launch<2, 2, 4, 2>(a, stream) : HQ_E_BADSHAPE;
    }
    if (a.M <= 2048 && tiles(32, 32) <= 256) return launch<1, 1, 8, 4>(a, stream);
    if (a.M <= 2048 && tiles(32, 64) <= 256) return launch<1, 2, 8, 2>(a, stream);
    auto worth_it = [&] {
        if (a.M <= 5120) return true;
        const unsigned long long image = (unsigned long long)p->B * p->H * p->W, x = (image < M * a.taps ? image : M * a.taps) * a.C;
        const unsigned long long per_xcd = ((a.C + 31) / 32 % 8 == 0 ? x / 2 : x) + M * a.N, weights = (unsigned long long)a.N * a.taps * a.C;
        const unsigned least = a.taps == 1 ? (a.M <= 6400 ? 0 : 8192) : (a.M <= 6400 ? 6400 : a.M <= 7168 ? 12800 : 20480);
        return weights >= least && (per_xcd <= (4u << 20) || (a.N >= 128 && a.C >= 96));
    };
    if (a.M <= 8192 && tiles(32, 32) <= 256 && a.g16 && a.x16 && worth_it())
        return launch<1, 1, 16, 2>(a, stream);
    return HQ_E_BADSHAPE;
}
