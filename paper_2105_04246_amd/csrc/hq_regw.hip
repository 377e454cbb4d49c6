// 3x3, stride 1, padding 1 with 64 reduced channels (forward, input gradient as the stencil with mirrored taps, pass 1 of
// the dynamic baseline): the weights of 64 output channels live in REGISTERS for the whole launch.
//
// With both MFMA operands read from LDS a 64 x 64 wavefront tile needs 1 KB per MFMA, all that LDS delivers, and whatever
// else a phase does comes on top (the weights-in-LDS kernel: 28 us for 128 x 56 x 56 x 64 against 7 us of matrix work).
// 64 channels x 576 reduced bytes are 144 registers per lane; then only the pixels come from LDS, 1 KB for two MFMAs.
// A compute unit holds two wavefronts per SIMD: while one requantizes, the other multiplies.
// A unit is 256 consecutive output pixels, 32 per wavefront, of the tensor's [image][row][column] order, whatever rows and
// images it spans.  The input rows it needs are copied to LDS in padded-image order (a row of padding above and below
// every image), one patch row per wavefront and turn, while the unit before is multiplied; pixels have a pitch of
// 80 bytes, which spreads the fragment reads (32 pixels at one 16-byte chunk) over the banks (conflicts: 18 % of LDS's busy cycles)
// and lets a tap be a constant offset from the pixel's address.
// Measured: 24 us at that size, 6 or 7 units to a workgroup: 8 for a launch of one unit each, 2.6 for each further one (1.2 of them
// matrix work); 61 x 37 x 23 x 64, whose rows fit no band of the other kernel, 16 -> 8.5 us.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int RW_THREADS = 512, RW_UNIT = 256, RW_PITCH = 80, RW_LOADS = 10;   // loads: 64 slots of 16 bytes of a patch row each

struct RegwArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, N, H, W, PW;            // output pixels, channels; image; patch row W + 2 pixels
    int flip;
    int units, nparts, runs;       // units of 256 pixels; blocks of 64 channels; workgroups per channel block
    int prows;                     // most patch rows of a unit
    unsigned magic_W, magic_H, magic_H2;   // of W, H, H + 2
    float inv_W, inv_H;
    HqSr sr;
};

template <int MODE>
__global__ __launch_bounds__(RW_THREADS, 2) void hq_regw_kernel(const RegwArgs a)
{
    constexpr int CB = 64, KC = CB / 32, STORES = MODE == 0 ? 32 : 2;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    __shared__ __attribute__((aligned(16))) int bias[64];
    __shared__ int red[4 * (RW_THREADS / 64)];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;

    const int run = blockIdx.x / a.nparts, n0 = (blockIdx.x - run * a.nparts) * 64;
    const int u_begin = (int)((long)a.units * run / a.runs), u_end = (int)((long)a.units * (run + 1) / a.runs);
    const int za = a.aq->zero_point;
    const int rowpitch = a.PW * RW_PITCH;
    const int bufbytes = a.prows * rowpitch + 1024;                  // (a row's last load may end past it)

    // ---- staging plan: slot q of a patch row is 16-byte chunk q % 5 of pixel q / 5 (chunk 4: the padding of the pitch)
    const int nload = (a.PW * 5 + 63) / 64;
    unsigned loff[RW_LOADS];
    unsigned lmask = 0;
#pragma unroll
    for (int k = 0; k < RW_LOADS; k++) {
        const int q = lane + 64 * k, px = q / 5, ch = q - 5 * px;
        const bool ok = px >= 1 && px <= a.W && ch < 4;
        loff[k] = ok ? (unsigned)((px - 1) * CB + ch * 16) : 0u;
        lmask |= ok ? 1u << k : 0u;
    }
    auto locate = [&](int p, int &g, int &b) {                       // row and image of an output pixel (uniform)
        g = (int)hq_magic_div((unsigned)p, a.magic_W);
        b = (int)hq_magic_div((unsigned)g, a.magic_H);
    };
    // patch rows wave, wave + 8, ... of unit u
    auto stage = [&](int u, int buf) {
        int g0, b0, g1, b1;
        locate(u * RW_UNIT, g0, b0);
        locate(min(a.M, (u + 1) * RW_UNIT) - 1, g1, b1);
        const int rows = g1 - g0 + 2 * (b1 - b0) + 3;
        for (int pr = wave; pr < rows; pr += RW_THREADS / 64) {
            const int pad = g0 + 2 * b0 + pr;                        // row of the padded images
            const int img = (int)hq_magic_div((unsigned)pad, a.magic_H2), y = pad - img * (a.H + 2) - 1;
            const bool in = y >= 0 && y < a.H;
            const int8_t *src = in ? a.A + ((size_t)img * a.H + y) * a.W * CB : reinterpret_cast<const int8_t *>(hq_fill_rows.w[za & 0xff]);
            int8_t *dst = smem + buf * bufbytes + pr * rowpitch;
#pragma unroll
            for (int k = 0; k < RW_LOADS; k++)
            {
                if (k >= nload) break;
                if ((lmask >> k) & 1) hq_global_to_lds16(src, in ? loff[k] : 0u, dst + 1024 * k);
            }
        }
    };

    const int bz = tid < 64 ? a.bsum[n0 + tid] : 0;
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);
    if (u_begin < u_end) stage(u_begin, 0);
    // padding columns of a buffer's patch rows: never written again
    auto pad_columns = [&](int buf) {
        const unsigned f = (unsigned)(za & 0xff) * 0x01010101u;
        const v4i fv = {(int)f, (int)f, (int)f, (int)f};
        for (int i = tid; i < a.prows * 8; i += RW_THREADS) {
            const int ch = i & 3, side = (i >> 2) & 1, pr = i >> 3;
            *reinterpret_cast<v4i *>(smem + buf * bufbytes + pr * rowpitch + (side ? (a.W + 1) * RW_PITCH : 0) + 16 * ch) = fv;
        }
    };
    pad_columns(0);
    if (tid < 64) bias[tid] = -za * bz;
    // Weights of this workgroup's 64 channels.  A fragment's 32 rows lie far apart, so loading them costs 64 cache lines a
    // KB: every wavefront fetches an eighth of the 36 fragments into LDS, where all read them from.  Row i of a fragment is
    // channel hq_sigma32(i), so that a lane ends up with 16 consecutive output channels; channel i for 32-bit outputs, whose
    // products are formed transposed (see finish).
    v4i wf[9][KC][2];
    {
        int8_t *frags = smem + bufbytes;                             // the second buffer is not needed yet
        const int8_t *wrow = a.Bw + (size_t)(n0 + (MODE == 0 ? lane & 31 : hq_sigma32(lane & 31))) * 9 * CB + 16 * half;
        for (int f = wave; f < 9 * KC * 2; f += RW_THREADS / 64) {
            const int nb = f & 1, kc = (f >> 1) % KC, t = (f >> 1) / KC;
            hq_global_to_lds16(wrow + (size_t)32 * nb * 9 * CB + (a.flip ? 8 - t : t) * CB + 32 * kc, frags + 1024 * f);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 9; t++)
#pragma unroll
            for (int kc = 0; kc < KC; kc++)
#pragma unroll
                for (int nb = 0; nb < 2; nb++) wf[t][kc][nb] = *reinterpret_cast<const v4i *>(frags + 1024 * ((t * KC + kc) * 2 + nb) + 16 * lane);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
    }
    pad_columns(1);
    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;

    auto body = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        v16i acc[2];
        auto multiply = [&](int u, int buf) {
            int g0, b0;
            locate(u * RW_UNIT, g0, b0);
            // row and image relative to the unit's first, from small numbers (exact: the error of the product is far
            // below the distance to the next integer of (q + 1/2) / W)
            const int q = min(u * RW_UNIT + wave * 32 + (lane & 31), a.M - 1) - g0 * a.W;
            const int rr = (int)(((float)q + 0.5f) * a.inv_W), x = q - rr * a.W;
            const int bb = (int)(((float)(g0 - b0 * a.H + rr) + 0.5f) * a.inv_H);
            const int8_t *p0 = smem + buf * bufbytes + (rr + 2 * bb) * rowpitch + x * RW_PITCH + 16 * half;
#pragma unroll
            for (int nb = 0; nb < 2; nb++)
                if constexpr (MODE == 0) {
                    const int bz = bias[32 * nb + (lane & 31)];
#pragma unroll
                    for (int e = 0; e < 16; e++) acc[nb][e] = bz;
                } else
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const v4i bz = *reinterpret_cast<const v4i *>(bias + 32 * nb + 16 * half + 4 * k);
#pragma unroll
                    for (int e = 0; e < 4; e++) acc[nb][4 * k + e] = bz[e];
                }
            // the next tap's fragments are requested before this tap's MFMAs
            v4i af[2][KC];
            auto fetch = [&](int t, v4i (&f)[KC]) {
                const int8_t *pr = p0 + t / 3 * rowpitch + t % 3 * RW_PITCH;
#pragma unroll
                for (int kc = 0; kc < KC; kc++) f[kc] = *reinterpret_cast<const v4i *>(pr + 32 * kc);
            };
            fetch(0, af[0]);
#pragma unroll
            for (int t = 0; t < 9; t++) {
                if (t < 8) fetch(t + 1, af[(t + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int kc = 0; kc < KC; kc++)
#pragma unroll
                    for (int nb = 0; nb < 2; nb++)
                        acc[nb] = MODE == 0 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(af[t & 1][kc], wf[t][kc][nb], acc[nb], 0, 0, 0)
                                            : __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[t][kc][nb], af[t & 1][kc], acc[nb], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        // 32-bit outputs: a lane holds one channel of 16 pixels, so a store of the wavefront writes two whole 128-byte lines
        // (with 16 channels of one pixel a lane it would touch 64 lines, a quarter of each: 44 us against 30 for
        // 128 x 56 x 56 x 64).
        auto finish32 = [&](int u) {
            const int P0 = u * RW_UNIT + wave * 32, left = a.M - P0;
            const unsigned lo = (unsigned)(4 * half * a.N + (lane & 31));
#pragma unroll
            for (int nb = 0; nb < 2; nb++) {
                int c[16];
#pragma unroll
                for (int e = 0; e < 16; e++) c[e] = acc[nb][e];
                if (left >= 32) hq_minmax_group<16>(c, mn, mx);
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int row = 8 * (e >> 2) + (e & 3);
                    int32_t *dst = a.out32 + (size_t)(P0 + row) * a.N + n0 + 32 * nb;
                    if (left >= 32) dst[lo] = c[e];
                    else if (row + 4 * half < left) { dst[lo] = c[e]; mn = min(mn, c[e]); mx = max(mx, c[e]); }
                }
            }
        };
        auto finish = [&](int u) {
            if constexpr (MODE == 0) { finish32(u); return; }
            const int P = u * RW_UNIT + wave * 32 + (lane & 31);
            if (P >= a.M) return;
#pragma unroll
            for (int nb = 0; nb < 2; nb++) {
                int c[16];
#pragma unroll
                for (int e = 0; e < 16; e++) c[e] = acc[nb][e];
                const size_t o = (size_t)P * a.N + n0 + 32 * nb + 16 * half;
                int w[4];
                if constexpr (MODE == 2) hq_requant_group_sr<16, FULL, 16>(c, ep, a.sr, o, mn, mx, nlo, nhi, w);
                else                     hq_requant_group<16, FULL>(c, ep, mn, mx, nlo, nhi, w);
                *reinterpret_cast<v4i *>(a.out8 + o) = v4i{w[0], w[1], w[2], w[3]};
            }
        };
        // Between two barriers one of a SIMD's two wavefronts multiplies first and requantizes then, the other (`late`)
        // requantizes its unit before and then multiplies, so that the matrix cores and the vector ALU both have work.
        const bool late = wave >= RW_THREADS / 128;
        for (int u = u_begin; u < u_end; u++) {
            const int buf = (u - u_begin) & 1;
            // this wavefront's rows of unit u are in LDS once only the stores issued after them are under way
            if (u == u_begin || (late && u == u_begin + 1)) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            else                                           asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STORES) : "memory");
            __syncthreads();
            if (u + 1 < u_end) stage(u + 1, buf ^ 1);
            if (late && u > u_begin) finish(u - 1);
            multiply(u, buf);
            if (!late) finish(u);
        }
        if (late && u_end > u_begin) finish(u_end - 1);
    };
    if (MODE == 0 || ep.full_grid) body(std::true_type()); else body(std::false_type());
    hq_block_stats_commit_n<RW_THREADS>(mn, mx, nlo, nhi, a.st, red);
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.N);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

} // namespace

int hq_try_launch_regw(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8, int32_t *out32,
                       hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    if (p->kind != HQ_CONV2D || p->R != 3 || p->S != 3 || p->stride != 1 || p->pad != 1) return HQ_E_BADSHAPE;
    const int Cs = dgrad ? p->Cout : p->C, N = dgrad ? p->C : p->Cout;
    if (Cs != 64 || N % 64 != 0) return HQ_E_BADSHAPE;
    const unsigned long long M = (unsigned long long)p->B * p->H * p->W;
    const int H = p->H, W = p->W;
    // operands of hq_magic_div and the exactness of the float divisions
    if ((M + RW_UNIT) * (unsigned)((H > W ? H : W) + 2) >= (1ull << 32) || H > 4096 || W > 4096) return HQ_E_BADSHAPE;
    RegwArgs a = {};
    a.PW = W + 2;
    if ((a.PW * 5 + 63) / 64 > RW_LOADS) return HQ_E_BADSHAPE;
    const int rows = (RW_UNIT + W - 2) / W + 1;                      // most output rows a unit touches
    a.prows = rows + 2 + 2 * ((rows + H - 2) / H);
    const size_t buf = (size_t)a.prows * a.PW * RW_PITCH + 1024;
    const size_t lds = buf + std::max(buf, (size_t)36 * 1024);
    if (lds > 156 * 1024) return HQ_E_BADSHAPE;
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    a.M = (int)M; a.N = N; a.H = H; a.W = W; a.flip = dgrad;
    a.units = (int)((M + RW_UNIT - 1) / RW_UNIT);
    a.nparts = N / 64;
    a.runs = 256 / a.nparts;
    if (a.runs < 1) a.runs = 1;
    if (a.runs > a.units) a.runs = a.units;
    a.magic_W = hq_magic32((unsigned)W); a.magic_H = hq_magic32((unsigned)H); a.magic_H2 = hq_magic32((unsigned)(H + 2));
    a.inv_W = 1.0f / (float)W; a.inv_H = 1.0f / (float)H;
    if (sr_seed && out32) return HQ_E_BADARG;
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    auto kern = mode == 0 ? hq_regw_kernel<0> : mode == 2 ? hq_regw_kernel<2> : hq_regw_kernel<1>;
    static std::atomic<unsigned long long> allowed[3];
    if (!hq_allow_lds(kern, 156 * 1024, allowed[mode])) return HQ_E_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.runs * a.nparts)), dim3(RW_THREADS), lds, stream, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}
