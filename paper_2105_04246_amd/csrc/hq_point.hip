// Short reductions (at most 192 channels or features: 1x1 layers and linear layers; forward, input gradient of unit stride, pass 1 of the
// dynamic baseline): a pixel's channels go from global memory straight into MFMA operands, up to 78 KB of weights stay in LDS.
//
// Such a layer has one MFMA for every 16 to 192 requantized values of a lane: it is bound by memory or by the requantization (about
// 100 vector instructions a tile of 32 pixels x 32 channels), never by the matrix cores, and what other kernels do for those, staging pixels
// through LDS and meeting at barriers, only stands in the way.  Here a wavefront works alone: it loads the fragments of 32 pixels (lane l has
// 16 channels of pixel l % 32), the next 32 pixels' before it works on these, walks the blocks of 32 output channels and stores 16 codes a lane.
// Sixteen wavefronts a compute unit keep memory and vector ALU busy.  Weights lie in LDS as fragments in the order of their lanes (no bank
// conflicts, immediate offsets), loaded straight from global memory.
//
// Measured, before -> now (us), 401,408 pixels: 32 -> 192 channels 35.2 -> 24.3 (90 MB: 3.7 TB/s; 16 at the rate of a copy), its input
// gradient 22.8 -> 16.3, 192 -> 32 22.4 -> 15.8, its input gradient 36.3 -> 24.3 (stochastic 75.5 -> 60.4), 48 -> 144 40.3 -> 21.5, 64 -> 64 19.9 -> 12.8;
// 16,900 pixels, 192 -> 192 15.3 -> 5.8; stride 2 on 256 x 56 x 56, 64 -> 128 17.3 -> 14.0; 8192 x 192 x 4096 22.4 -> 18.5; 32-bit outputs 20 to 30 % less.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int PT_THREADS = 512, PT_WAVES = PT_THREADS / 64;
constexpr int PT_MANY = 2048;                                            // blocks of 32 pixels that fill the chip (256 units, 8 wavefronts)
constexpr int PT_LDS = 78 * 1024;                                        // two workgroups on a compute unit

struct PointArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, N, K;
    int nper, nparts, runs;        // blocks of 32 channels of a workgroup; such parts; workgroups per part
    int stride, H, W, OW, image;   // of a strided layer: source rows and columns, output columns and pixels of an image
    HqDivisor per_image, line;     // image and OW
    HqSr sr;
};

template <int KS, int MODE>
__global__ __launch_bounds__(PT_THREADS, 4) void hq_point_kernel(const PointArgs a)
{
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];       // fragments in the order of their lanes, 1 KB each; biases
    __shared__ int red[4 * PT_WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, r32 = lane & 31;
    const int run = __builtin_amdgcn_readfirstlane(blockIdx.x / a.nparts), part = blockIdx.x - run * a.nparts;
    const int n0 = 32 * a.nper * part, nblocks = min(a.nper, (a.N - n0 + 31) / 32);
    const int all = (a.M + 31) / 32;
    const int begin = (int)((long)all * run / a.runs), end = (int)((long)all * (run + 1) / a.runs);
    int *bias = reinterpret_cast<int *>(smem + 1024 * KS * a.nper);

    // ---- weights: row i of a fragment is channel hq_sigma32(i), so that a lane ends up with 16 consecutive output channels; channel i
    // for 32-bit outputs, whose products are formed transposed
    for (int f = wave; f < nblocks * KS; f += PT_WAVES) {
        const int nb = f / KS, k = 32 * (f - nb * KS) + 16 * half, n = n0 + 32 * nb + (MODE == 0 ? r32 : hq_sigma32(r32));
        const int8_t *src = a.Bw + (size_t)n * a.K + k;
        asm("" : "+v"(src));                                            // (selected, not branched around)
        hq_global_to_lds16(n < a.N && k < a.K ? src : reinterpret_cast<const int8_t *>(hq_fill_rows.w[0]), smem + 1024 * f);
    }

    // ---- a block of 32 pixels: lane's pixel, 16 channels of every 32.  What is read for channels past the last (K an odd number of 16)
    // meets weights of 0; pixels past the last repeat it.
    auto fetch = [&](int block, v4i (&af)[KS]) __attribute__((always_inline)) {
        unsigned m = (unsigned)min(32 * block + r32, a.M - 1);
        if (a.stride > 1) {
            const unsigned b = hq_quot(m, a.per_image), rem = m - b * (unsigned)a.image, y = hq_quot(rem, a.line);
            m = (b * (unsigned)a.H + y * (unsigned)a.stride) * (unsigned)a.W + (rem - y * (unsigned)a.OW) * (unsigned)a.stride;
        }
        const int8_t *p = a.A + (size_t)m * a.K;
#pragma unroll
        for (int ks = 0; ks < KS; ks++) af[ks] = *reinterpret_cast<const v4i *>(p + min(32 * ks + 16 * half, a.K - 16));
    };
    // (beside the random bits 9 and 23 registers would spill.  Without them one does under 161 to 192 channels, and the next pixels on their way are
    // worth it: 100,352 x 192 -> 32 5.9 us, 6.2 without)
    constexpr bool AHEAD = MODE != 2 || KS < 5;
    v4i afA[KS], afB[AHEAD ? KS : 1];
    int block = begin + wave;
    if (block < end) fetch(block, afA);
    const int za = a.aq->zero_point;
    for (int i = tid; i < 32 * nblocks; i += PT_THREADS) bias[i] = n0 + i < a.N ? -za * a.bsum[n0 + i] : 0;
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();

    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    auto body = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        auto process = [&](int block, const v4i (&af)[KS]) __attribute__((always_inline)) {
            const int first = 32 * block, pixel = first + r32;
            const bool whole = first + 32 <= a.M;
            for (int nb = 0; nb < nblocks; nb++) {
                const int8_t *frag = smem + 1024 * KS * nb + 16 * lane;
                v16i acc;
                if constexpr (MODE == 0) {
                    const int b = bias[32 * nb + r32];
#pragma unroll
                    for (int e = 0; e < 16; e++) acc[e] = b;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const v4i b = *reinterpret_cast<const v4i *>(bias + 32 * nb + 16 * half + 4 * k);
#pragma unroll
                        for (int e = 0; e < 4; e++) acc[4 * k + e] = b[e];
                    }
                }
#pragma unroll
                for (int ks = 0; ks < KS; ks++) {
                    const v4i wf = *reinterpret_cast<const v4i *>(frag + 1024 * ks);
                    acc = MODE == 0 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(af[ks], wf, acc, 0, 0, 0)
                                    : __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, af[ks], acc, 0, 0, 0);
                }
                int c[16];
#pragma unroll
                for (int e = 0; e < 16; e++) c[e] = acc[e];
                if constexpr (MODE == 0) {
                    // a lane holds one channel of 16 pixels: a store of the wavefront writes whole lines of two pixels
                    const int n = n0 + 32 * nb;
                    const unsigned mine = (unsigned)(4 * half * a.N + r32);
                    int32_t *out = a.out32 + (size_t)(unsigned)first * a.N + n;
                    if (n + r32 < a.N) {
                        if (whole) hq_minmax_group<16>(c, mn, mx);
#pragma unroll
                        for (int e = 0; e < 16; e++) {
                            asm("" : "+s"(out));                        // (a uniform address and the lane's part)
                            if (whole) out[mine] = c[e];
                            else if (first + 8 * (e >> 2) + (e & 3) + 4 * half < a.M) { out[mine] = c[e]; mn = min(mn, c[e]); mx = max(mx, c[e]); }
                            out += e % 4 == 3 ? 5 * a.N : a.N;
                        }
                    }
                } else {
                    const int n = n0 + 32 * nb + 16 * half;
                    if (pixel < a.M && n < a.N) {
                        const size_t o = (size_t)(unsigned)pixel * a.N + n;
                        int w[4];
                        if constexpr (MODE == 2) hq_requant_group_sr<16, FULL, 16>(c, ep, a.sr, o, mn, mx, nlo, nhi, w);
                        else                     hq_requant_group<16, FULL>(c, ep, mn, mx, nlo, nhi, w);
                        *reinterpret_cast<v4i *>(a.out8 + o) = v4i{w[0], w[1], w[2], w[3]};
                    }
                }
            }
        };
        if constexpr (!AHEAD) {
            for (; block < end; block += PT_WAVES) {
                process(block, afA);
                if (block + PT_WAVES < end) fetch(block + PT_WAVES, afA);
            }
        } else while (block < end) {                                    // the next block is on its way while this one is worked on
            if (block + PT_WAVES < end) fetch(block + PT_WAVES, afB);
            process(block, afA);
            block += PT_WAVES;
            if (block >= end) break;
            if (block + PT_WAVES < end) fetch(block + PT_WAVES, afA);
            process(block, afB);
            block += PT_WAVES;
        }
    };
    if (MODE == 0 || ep.full_grid) body(std::true_type()); else body(std::false_type());
    hq_block_stats_commit_n<PT_THREADS>(mn, mx, nlo, nhi, a.st, red);
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.N);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

template <int KS> int point_launch(const PointArgs &a, int mode, size_t lds, hipStream_t stream)
{
    auto kern = mode == 0 ? hq_point_kernel<KS, 0> : mode == 2 ? hq_point_kernel<KS, 2> : hq_point_kernel<KS, 1>;
    static std::atomic<unsigned long long> allowed[3];
    if (!hq_allow_lds(kern, PT_LDS, allowed[mode])) return HQ_E_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.runs * a.nparts)), dim3(PT_THREADS), lds, stream, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

} // namespace

int hq_try_launch_point(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                        const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8, int32_t *out32,
                        hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    const bool linear = p->kind == HQ_LINEAR;
    if (!linear && (p->kind != HQ_CONV2D || p->R != 1 || p->S != 1 || p->pad != 0)) return HQ_E_BADSHAPE;
    if (dgrad && p->stride != 1) return HQ_E_BADSHAPE;
    const int K = dgrad ? p->Cout : p->C, N = dgrad ? p->C : p->Cout;
    if (K % 16 != 0 || N % 16 != 0 || K > 192) return HQ_E_BADSHAPE;
    const int OH = (p->H - 1) / p->stride + 1, OW = (p->W - 1) / p->stride + 1;
    const unsigned long long M = (unsigned long long)p->B * OH * OW;
    if ((unsigned long long)p->B * p->H * p->W >= (1ull << 31) - 4096) return HQ_E_BADSHAPE;
    if (sr_seed && out32) return HQ_E_BADARG;
    PointArgs a = {};
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    a.M = (int)M; a.N = N; a.K = K;
    a.stride = p->stride; a.H = p->H; a.W = p->W; a.OW = OW; a.image = OH * OW;
    a.per_image = hq_divisor((unsigned)a.image); a.line = hq_divisor((unsigned)OW);
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    const int ks = (K + 31) / 32, blocks = (N + 31) / 32, most = PT_LDS / (1024 * ks + 128);
    const int all = (int)((M + 31) / 32);
    // 128 channels are two whole stages of the general kernel.  Where all of its 128 x 128 tiles are resident at once, four to a compute unit, and are
    // more than a round and a third, the two are level (general / this, us: 12,000 x 512 7.6 / 7.5, 24,000 x 256 7.6 / 7.6, 16,000 x 512 7.9 / 7.4, 24,000 x
    // 384 9.4 / 9.4, 11,729 x 864 9.4 / 9.6, 32,000 x 384 9.8 / 10.5, 12,000 x 928 9.7 / 10.7, 34,932 x 352 11.6 / 12.1, 16,805 x 768 11.3 / 10.9, 32,000 x 512 12.1 /
    // 11.1) and it stays there.  With fewer or more tiles this kernel is ahead (12,000 x 256 6.5 / 5.5, 7010 x 752 7.8 / 7.2; 45,184 x 400 16.4 / 15.9,
    // 24,021 x 1664 23.7 / 22.2, 63,257 x 928 33.7 / 29.0; 47 layers 0.90 of the time, one 3 % slower), and so it is with 112 channels (9852 x 288 6.7 / 5.3,
    // 6294 x 1888 10.0 / 9.7, 27,522 x 1088 20.2 / 15.9; 32 layers 0.83) and under stochastic rounding (24,000 x 512 15.7 / 14.7; 64 layers 0.88, one 4 % slower).
    const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
    if (K == 128 && N >= 256 && mode == 1 && tiles > 340 && tiles <= 1024) return HQ_E_BADSHAPE;
    // Where there are blocks of pixels for every wavefront a workgroup takes all the channels whose weights fit: split between workgroups the
    // lines of an output would be written in parts (401,408 x 32 x 192: 24 us in one part, 39 in three).  With fewer blocks the channels are
    // split, down to two blocks of 32, and the pixels dealt to as many workgroups as take least by this estimate: a wavefront's tiles one
    // after the other (5 units each) or the compute unit's on its four vector ALUs (2 wavefronts a unit), and 5 units to start a workgroup.
    // 8192 x 64 x 512: 10.5 us undivided, 4.8; 8192 x 128 x 1024 14.2, 7.6; 70000 x 128 x 512 24.9 in 274 workgroups, 21.6 in 512.
    // With stochastic rounding the vector ALUs bound every size: a tile is then mostly their work (3 units of latency), a SIMD's share comes in
    // whole blocks (every fourth of the workgroup's), one workgroup to a compute unit does not keep them busy, another number of workgroups for the
    // same split has to save an eighth, and channels are split under any number of pixels (100,244 x 64 x 944 90.0 us undivided, 72.9 in five parts).
    // Against the fastest of up to 60 splits each, 376 calls drawn at random: 4.9 % more time with rounding to nearest (a third at worst), 1.8 %
    // with stochastic rounding (18 % at worst; by the estimate for rounding to nearest 8.5 % and 45 %).
    const int least = (blocks + most - 1) / most;
    double best = 0.0;
    for (int nper = std::min(most, blocks); nper >= 1; nper--) {         // (at most 69 steps)
        const int nparts = (blocks + nper - 1) / nper;
        if ((blocks + nparts - 1) / nparts != nper) continue;            // (as many parts as with fewer blocks each)
        if (nparts != least && (nper < 2 || (mode != 2 && all >= PT_MANY))) continue;
        for (int want : {(all + PT_WAVES - 1) / PT_WAVES, 256 / nparts, 512 / nparts}) {
            const int runs = std::max(1, std::min({want, 512 / nparts, all}));
            const long share = (all + runs - 1) / runs, rounds = ((long)runs * nparts + 255) / 256, serial = (share + PT_WAVES - 1) / PT_WAVES * nper;
            const double load = 0.5 * (double)(rounds * nper) * (double)(mode == 2 ? (share + 3) / 4 * 4 : share);
            const double cost = std::max(mode == 2 ? 3.0 * serial : 5.0 * serial, mode == 2 && rounds == 1 ? 1.15 * load : load) + 5.0 * rounds;
            if (a.nper == 0 || (mode == 2 && nper == a.nper ? 1.125 : 1.0) * cost < best) { best = cost; a.nparts = nparts; a.nper = nper; a.runs = runs; }
        }
    }
    const size_t lds = (size_t)a.nper * (1024 * ks + 128);
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    switch (ks) {
    case 1: return point_launch<1>(a, mode, lds, stream);
    case 2: return point_launch<2>(a, mode, lds, stream);
    case 3: return point_launch<3>(a, mode, lds, stream);
    case 4: return point_launch<4>(a, mode, lds, stream);
    case 5: return point_launch<5>(a, mode, lds, stream);
    default: return point_launch<6>(a, mode, lds, stream);
    }
}
