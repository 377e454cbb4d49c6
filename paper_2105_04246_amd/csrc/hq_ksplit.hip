// Small launches of hq_gemm_fwd / hq_gemm_dgrad and of pass 1 of the dynamic baseline: layers whose output has so few
// tiles that the tile kernels leave most compute units idle while each tile walks its whole reduction stage by
// stage (batch-1 inference, small images under many channels, fully connected layers, ragged layers).
//
// What bounds such a launch is the latency of one tile's serial chain: load, wait, barrier, multiply, once per stage
// (about 1 us each; 46 us for 7x7x512 -> 512 at batch 1).  Here the wavefronts of a workgroup share a small
// output tile and split its reduction: wavefront w takes the 64-byte steps w, w + NW, ... and meets the others only once, when
// the partial sums are added through LDS.  There is no barrier inside the reduction.  Aligned form: each wavefront brings its
// steps into LDS of its own (direct-to-LDS loads of whole lines, D steps ahead), D x (TMB + TNB) KB in flight, and reads the MFMA
// fragments from there.  4-byte form (channel counts off 16): fragments straight from global memory into registers.  The price is
// that an operand byte is fetched once per tile instead of once per larger tile, so the rate is bound by the 64 bytes a clock a
// compute unit loads: (TM + TN) x K / 64 clocks per tile.  Measured (forward, before -> now): 7x7x512 -> 512 at batch 1 45 -> 8.4 us,
// 14x14x256 25 -> 7.3, 28x28x128 16 -> 6.9; 256 x 512 -> 1000 with 1000 reduced 30 -> 10; 4x4x512 at batch 128 24 -> 17 us.
// What is left is fixed: of the 16 K cycles a 56x56x64 launch then took (clock stamps), 1.1 K were its loads and matrix work, the
// rest arguments and operands fetched one miss after the other (2 + 1.2 K), a mask of every pixel's taps (5 K), loads of steps
// past the end, divisions and statistics (2 K).  Those are gone, requested together, or moved under the first loads: 10 K
// cycles, ResNet-18's forward pass at batch 1 155 -> 119 us, its step on 32 images of 64x64 525 -> 438 us.
//
// Both operations are  out[m][n] = sum_{tap,c} A[pix(m,tap)][c] * Bw[n][tap][c]  as in the gather kernel, with the
// same class form for strided input gradients (an output pixel's class fixes its taps; everything else is one class).
// A lane holds, per 16x16 block, 16 bytes of the reduction of one pixel and of one channel; the weights are the first
// operand, so that a lane ends up with 4 consecutive channels of one pixel.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

struct KsClass {
    int ph, pw, Hc, Wc;            // pixels (ph + ostep * y, pw + ostep * x) of the output image, y < Hc, x < Wc
    int ns, taps;                  // taps per row of the class's tap grid, taps in all
    int dh, dw;                    // source pixel of tap (0, 0) for y = x = 0
    int w0;                        // weight tap of tap (0, 0)
    unsigned magic_Wc, magic_Hc, magic_ns;
};

struct KsArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, N, B;
    int Cs, cpt;                   // reduced channels per tap; 16-byte chunks per tap (aligned form)
    unsigned magic_div;            // of cpt (aligned) or Cs
    size_t wrow;                   // bytes per weight row
    int Hs, Ws, Ho, Wo;            // source image, output image
    int istep, ostep, sgn;         // source pixel = istep * y + dh + sgn * tr;  ostep: class stride in the output
    int wr, wc;                    // weight tap = w0 + wr * tr + wc * ts
    int m_tiles, n_tiles, m_fast;  // m_fast: consecutive workgroups share their weights, not their pixels
    int classed, ncls;             // classed: the zero-point term is summed from the class's own weights
    HqSr sr;
    int tile0[16];                 // first row tile of each class
    KsClass cls[16];
};

// TMB, TNB: 16-pixel and 16-channel blocks of the tile.  NW wavefronts, D steps in flight.  MODE as in the gather kernel:
// 0 32-bit outputs, 1 round to nearest even, 2 stochastic rounding.  ALIGNED: Cs % 16 == 0, a 16-byte chunk is of one tap;
// otherwise 4-byte words (Cs % 4 == 0).
template <int TMB, int TNB, int NW, int D, bool ALIGNED, int MODE>
__global__ __launch_bounds__(NW * 64) void hq_ksplit_kernel(const KsArgs a)
{
    constexpr int TM = 16 * TMB, TN = 16 * TNB;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    constexpr int BUF = NW * 1024 * (TMB * TNB > D * (TMB + TNB) ? TMB * TNB : D * (TMB + TNB));
    v4i *sums = reinterpret_cast<v4i *>(smem);                           // [NW][TNB][TMB][64]
    int *bzs = reinterpret_cast<int *>(smem + BUF);                      // [TN]
    int *red = bzs + TN;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    // Aligned form: a 1 KB block of a step, 16 rows of 64 bytes, goes to LDS directly.  Lane l of such a load lands at
    // 16 * l, so consecutive lanes fetch consecutive chunks of one row (fragments loaded as the MFMA wants them, 16
    // rows side by side, come at a quarter of the rate); the chunks of a row are XOR-swizzled by the row, which keeps the
    // fragment reads free of bank conflicts.  4-byte form: fragments straight into registers.
    const int lrow = ALIGNED ? lane >> 2 : r16;                          // row of the lane's loads in a block
    const int lchunk = ALIGNED ? (lane & 3) ^ ((lrow >> 1) & 3) : g;     // and its 16-byte chunk of the step
    const int frag = r16 * 64 + 16 * (g ^ ((r16 >> 1) & 3));

    // The arguments span several cache lines; asked for where they are used they arrive one after the other, a miss each.
    const KsClass &c0 = a.cls[0];
    int m_tiles = a.m_tiles;
    asm("" : "+s"(m_tiles) : "s"(a.A), "s"(a.aq), "s"(a.st), "s"(a.M), "s"(a.wrow), "s"(a.istep), "s"(a.sr.k1), "s"(a.tile0[0]),
        "s"(a.tile0[15]), "s"(c0.ph), "s"(c0.magic_ns));
    int tile_m, tile_n;
    if (a.m_fast) { tile_n = blockIdx.x / m_tiles; tile_m = blockIdx.x - tile_n * m_tiles; }
    else          { tile_m = blockIdx.x / a.n_tiles; tile_n = blockIdx.x - tile_m * a.n_tiles; }
    int ci = 0;
    while (ci + 1 < a.ncls && tile_m >= a.tile0[ci + 1]) ci++;
    const KsClass &cl = a.cls[ci];
    const int m0 = (tile_m - a.tile0[ci]) * TM, n0 = tile_n * TN;
    int w0 = cl.w0;
    unsigned magic_ns = cl.magic_ns, magic_div = a.magic_div;
    asm("" : "+s"(w0), "+s"(magic_ns), "+s"(magic_div));                 // (kept, not read again for every load)
    const int Wc = cl.Wc, Hc = cl.Hc, ns = cl.ns, taps = cl.taps, Mrows = a.B * Hc * Wc;
    const int units = ALIGNED ? taps * a.cpt : taps * a.Cs / 4;          // 16-byte chunks / 4-byte words of the reduction
    auto decode = [&](int m, int &x, int &y, int &b) {
        const unsigned t = hq_magic_div((unsigned)m, cl.magic_Wc), bb = hq_magic_div(t, cl.magic_Hc);
        x = (int)((unsigned)m - t * (unsigned)Wc); y = (int)(t - bb * (unsigned)Hc); b = (int)bb;
    };

    const int za = a.aq->zero_point;
    const int8_t *fill = reinterpret_cast<const int8_t *>(hq_fill_rows.w[za & 0xff]);
    const int8_t *zero = reinterpret_cast<const int8_t *>(hq_fill_rows.w[0]);
    if (a.classed && tid < TN) bzs[tid] = 0;

    // per pixel of the lane: its source pixel and address of tap (0, 0)
    const int8_t *arow[TMB];
    int ay[TMB], ax[TMB];
#pragma unroll
    for (int i = 0; i < TMB; i++) {
        const int m = m0 + 16 * i + lrow;
        int x, y, b;
        decode(m < Mrows ? m : 0, x, y, b);              // rows past the end repeat row 0; nothing of them is stored
        ay[i] = y * a.istep + cl.dh; ax[i] = x * a.istep + cl.dw;
        arow[i] = a.A + ((ptrdiff_t)((ptrdiff_t)b * a.Hs + ay[i]) * a.Ws + ax[i]) * a.Cs;
    }
    const int8_t *brow[TNB];
#pragma unroll
    for (int j = 0; j < TNB; j++) {
        const int n = n0 + 16 * j + lrow;
        brow[j] = a.Bw + (size_t)(n < a.N ? n : 0) * a.wrow;
    }

    // What the epilogue reads is requested before the reduction: fetched after it, a launch's last memory round trip (1.2 K of
    // 16 K cycles) would be its own.
    constexpr int UPT = TMB * TNB > NW ? TMB * TNB / NW : 1;             // groups of 4 channels of one pixel per thread
    float scale_a = a.aq->scale, scale_b = a.bq->scale;
    hq_range range = {};
    if (MODE != 0) range = *a.range;
    v4i bz[UPT];
#pragma unroll
    for (int k = 0; k < UPT; k++) {
        const int u = tid + k * NW * 64, n = n0 + 16 * ((u >> 6) / TMB) + 4 * ((u & 63) >> 4);
        bz[k] = v4i{0, 0, 0, 0};
        if (!a.classed && u < TMB * TNB * 64 && n < a.N) bz[k] = *reinterpret_cast<const v4i *>(a.bsum + n);
    }

    // unit u (chunk or word): its tap's source pixel relative to tap (0, 0), its offsets from a pixel's tap (0, 0) and from a
    // weight row.  A tap has a source where that pixel lies in the image: two compares a load, where a mask of the taps worked
    // out beforehand costs a launch of nine taps 1.7 K cycles for every pixel of a lane before its first load.
    auto locate = [&](int u, int &dy, int &dx, int &aoff, int &woff) {
        const int per = ALIGNED ? a.cpt : a.Cs;
        const int k = ALIGNED ? u : 4 * u;
        const int tap = (int)hq_magic_div((unsigned)k, magic_div);
        const int tr = (int)hq_magic_div((unsigned)tap, magic_ns), ts = tap - tr * ns;
        const int c = (k - tap * per) * (ALIGNED ? 16 : 1);
        dy = a.sgn * tr; dx = a.sgn * ts;
        aoff = (dy * a.Ws + dx) * a.Cs + c;
        woff = (w0 + tr * a.wr + ts * a.wc) * a.Cs + c;
    };
    auto inside = [&](int i, int dy, int dx) { return (unsigned)(ay[i] + dy) < (unsigned)a.Hs && (unsigned)(ax[i] + dx) < (unsigned)a.Ws; };
    int8_t *const stage0 = smem + wave * D * (TMB + TNB) * 1024;         // [D][TMB + TNB][1024], this wavefront's own
    auto load_lds = [&](int step, int d) {
        const int u = 4 * step + lchunk;
        const bool ok = u < units;
        int dy, dx, aoff, woff;
        locate(u, dy, dx, aoff, woff);
        int8_t *dst = stage0 + d * (TMB + TNB) * 1024;
#pragma unroll
        for (int i = 0; i < TMB; i++) hq_global_to_lds16(ok && inside(i, dy, dx) ? arow[i] + aoff : fill, dst + 1024 * i);
#pragma unroll
        for (int j = 0; j < TNB; j++) hq_global_to_lds16(ok ? brow[j] + woff : zero, dst + 1024 * (TMB + j));
    };
    auto load_regs = [&](int step, v4i (&af)[TMB], v4i (&bf)[TNB]) {
#pragma unroll
        for (int d = 0; d < 4; d++) {
            const int u = 16 * step + 4 * lchunk + d;
            const bool ok = u < units;
            int dy, dx, aoff, woff;
            locate(u, dy, dx, aoff, woff);
#pragma unroll
            for (int i = 0; i < TMB; i++) af[i][d] = *reinterpret_cast<const int *>(ok && inside(i, dy, dx) ? arow[i] + aoff : fill);
#pragma unroll
            for (int j = 0; j < TNB; j++) bf[j][d] = *reinterpret_cast<const int *>(ok ? brow[j] + woff : zero);
        }
    };

    v4i acc[TNB][TMB];
#pragma unroll
    for (int j = 0; j < TNB; j++)
#pragma unroll
        for (int i = 0; i < TMB; i++) acc[j][i] = v4i{0, 0, 0, 0};
    int wsum[TNB] = {};
    const bool own_sums = a.classed && za != 0;

    // (4-byte form: steps past the end read the fill rows and add nothing, so the loads need no branch)
    const int nsteps = (units + (ALIGNED ? 3 : 15)) / (ALIGNED ? 4 : 16);
    auto multiply = [&](const v4i (&af)[TMB], const v4i (&bf)[TNB]) {
        if (own_sums)
#pragma unroll
            for (int j = 0; j < TNB; j++)
#pragma unroll
                for (int e = 0; e < 4; e++) wsum[j] = __builtin_amdgcn_sdot4(bf[j][e], 0x01010101, wsum[j], false);
#pragma unroll
        for (int j = 0; j < TNB; j++)
#pragma unroll
            for (int i = 0; i < TMB; i++)
                acc[j][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(bf[j], af[i], acc[j][i], 0, 0, 0);
    };
    float acc_scale;
    HqEpilogue ep = {1.0f, 0.0f, 0.0f, 0.0f, true};
    auto requant_constants = [&]() {                     // (the empty statements keep their divisions behind the first loads,
        auto behind = [](auto x) {                       // and before the reduction)
            int v = __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x));
            asm volatile("" : "+s"(v));
            return __builtin_bit_cast(decltype(x), v);
        };
        acc_scale = __fmul_rn(behind(scale_a), behind(scale_b));
        if (MODE != 0) {
            range.qp.scale = behind(range.qp.scale); range.qp.zero_point = behind(range.qp.zero_point);
            range.qlo = behind(range.qlo); range.qhi = behind(range.qhi);
            ep = hq_make_epilogue(acc_scale, &range);
            asm volatile("" : "+v"(ep.mult), "+v"(ep.flo), "+v"(ep.fhi), "+v"(ep.zoff), "+v"(ep.c_lo), "+v"(ep.c_hi));
        }
    };
    if constexpr (ALIGNED) {
#pragma unroll
        for (int d = 0; d < D; d++)
            if (wave + NW * d < nsteps) load_lds(wave + NW * d, d);
        requant_constants();
        int d = 0;
        for (int s = wave; s < nsteps; s += NW) {
            // this wavefront's own loads only: no barrier.  D - 1 later steps are in flight; at the end fewer, and all are
            // waited for.
            if (s + NW * (D - 1) < nsteps) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * (TMB + TNB)) : "memory");
            else                           asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const int8_t *src = stage0 + d * (TMB + TNB) * 1024 + frag;
            v4i af[TMB], bf[TNB];
#pragma unroll
            for (int i = 0; i < TMB; i++) af[i] = *reinterpret_cast<const v4i *>(src + 1024 * i);
#pragma unroll
            for (int j = 0; j < TNB; j++) bf[j] = *reinterpret_cast<const v4i *>(src + 1024 * (TMB + j));
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the stage has been read: it can be filled again
            if (s + NW * D < nsteps) load_lds(s + NW * D, d);
            multiply(af, bf);
            d = d + 1 == D ? 0 : d + 1;
        }
    } else {
        v4i af[D][TMB], bf[D][TNB];
        // (not where a wavefront has no step: three of four tiles of a strided input gradient under a 1x1 filter have no tap, and
        // loading fill rows for them was a sixth of the launch: 439 x 29 x 29 x 12 <- 124 29.7 -> 24.6 us)
        if (wave < nsteps) {
#pragma unroll
            for (int d = 0; d < D; d++) load_regs(wave + NW * d, af[d], bf[d]);
        }
        requant_constants();
        for (int s = wave; s < nsteps; s += NW * D) {
#pragma unroll
            for (int d = 0; d < D; d++) {
                multiply(af[d], bf[d]);
                load_regs(s + NW * (d + D), af[d], bf[d]);
            }
        }
    }
    __syncthreads();                                     // the stages make room for the partial sums
#pragma unroll
    for (int j = 0; j < TNB; j++)
#pragma unroll
        for (int i = 0; i < TMB; i++) sums[((wave * TNB + j) * TMB + i) * 64 + lane] = acc[j][i];
    if (own_sums)
#pragma unroll
        for (int j = 0; j < TNB; j++) atomicAdd(bzs + 16 * j + r16, wsum[j]);
    __syncthreads();

    // ---- epilogue: a thread = 4 consecutive channels of one pixel
    // (waited for here: left to the epilogue, threads without a group would wait for the others' stores with them)
#pragma unroll
    for (int k = 0; k < UPT; k++) asm volatile("" : "+v"(bz[k]));
    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    auto epilogue = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
#pragma unroll
        for (int k = 0; k < UPT; k++) {
            const int u = tid + k * NW * 64;
            if (u >= TMB * TNB * 64) break;
            const int l = u & 63, i = (u >> 6) % TMB, j = (u >> 6) / TMB;
            int m = m0 + 16 * i + (l & 15);
            const int nc = 16 * j + 4 * (l >> 4), n = n0 + nc;
            if (m >= Mrows || n >= a.N) continue;        // N % 4 == 0
            v4i c = sums[u];
#pragma unroll
            for (int w = 1; w < NW; w++) c += sums[w * (TMB * TNB * 64) + u];
            if (a.classed) {
                if (za != 0) c -= za * *reinterpret_cast<const v4i *>(bzs + nc);
                int x, y, b;
                decode(m, x, y, b);
                m = (b * a.Ho + cl.ph + a.ostep * y) * a.Wo + cl.pw + a.ostep * x;
            } else {
                c -= za * bz[k];
            }
            const int cc[4] = {c[0], c[1], c[2], c[3]};
            const size_t o = (size_t)m * a.N + n;
            if constexpr (MODE == 0) {
                hq_minmax_group<4>(cc, mn, mx);
                *reinterpret_cast<v4i *>(a.out32 + o) = c;
            } else {
                int w;
                if constexpr (MODE == 2) hq_requant_group_sr<4, FULL>(cc, ep, a.sr, o, mn, mx, nlo, nhi, &w);
                else                     hq_requant_group<4, FULL>(cc, ep, mn, mx, nlo, nhi, &w);
                *reinterpret_cast<int *>(a.out8 + o) = w;
            }
        }
    };
    if (ep.full_grid) epilogue(std::true_type()); else epilogue(std::false_type());
    hq_block_stats_commit_n<NW * 64>(mn, mx, nlo, nhi, a.st, red);
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.N);
        if (MODE != 0) *a.outq = range.qp;
    }
}

template <int TMB, int TNB, int NW, int D, bool ALIGNED, int MODE>
int launch3(KsArgs &a, hipStream_t s)
{
    int t = 0;
    for (int c = 0; c < a.ncls; c++) {
        a.tile0[c] = t;
        t += (a.B * a.cls[c].Hc * a.cls[c].Wc + 16 * TMB - 1) / (16 * TMB);
    }
    a.m_tiles = t;
    a.n_tiles = (a.N + 16 * TNB - 1) / (16 * TNB);
    const size_t lds = (size_t)NW * 1024 * (TMB * TNB > D * (TMB + TNB) ? TMB * TNB : D * (TMB + TNB)) + 4 * 16 * TNB + 16 * NW;
    auto kern = hq_ksplit_kernel<TMB, TNB, NW, D, ALIGNED, MODE>;
    static std::atomic<unsigned long long> allowed{0};
    if (!hq_allow_lds(kern, lds, allowed)) return HQ_E_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.m_tiles * a.n_tiles)), dim3(NW * 64), lds, s, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

template <int TMB, int TNB, int NW, int D, bool ALIGNED>
int launch2(KsArgs &a, int mode, hipStream_t s)
{
    if (mode == 0) return launch3<TMB, TNB, NW, D, ALIGNED, 0>(a, s);
    if (mode == 1) return launch3<TMB, TNB, NW, D, ALIGNED, 1>(a, s);
    return launch3<TMB, TNB, NW, D, ALIGNED, 2>(a, s);
}

} // namespace

int hq_try_launch_ksplit(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                         const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                         int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    if (p->kind == HQ_DEPTHWISE || (!dgrad && p->C < 8)) return HQ_E_BADSHAPE;      // (first layers have their own kernels)
    const int OH = (p->H + 2 * p->pad - p->R) / p->stride + 1, OW = (p->W + 2 * p->pad - p->S) / p->stride + 1;
    KsArgs a;
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st; a.B = p->B;
    const int taps = p->R * p->S;
    if (!dgrad) { a.N = p->Cout; a.Cs = p->C; a.Hs = p->H; a.Ws = p->W; a.Ho = OH; a.Wo = OW; }
    else        { a.N = p->C; a.Cs = p->Cout; a.Hs = OH; a.Ws = OW; a.Ho = p->H; a.Wo = p->W; }
    const unsigned long long M = (unsigned long long)a.B * a.Ho * a.Wo, lim = 1ull << 32;
    a.wrow = (size_t)taps * a.Cs;
    // operands of hq_magic_div: pixels, offsets in a weight row, taps
    if (M * (unsigned)(a.Ho > a.Wo ? a.Ho : a.Wo) >= lim || (a.wrow + 64) * a.Cs >= lim || (a.wrow + 64) / a.Cs * p->S >= lim) return HQ_E_BADSHAPE;
    // 32-bit offsets from a pixel's tap (0, 0)
    if (((unsigned long long)p->R * a.Ws + p->S) * a.Cs >= lim / 2) return HQ_E_BADSHAPE;
    a.M = (int)M;
    const bool aligned = a.Cs % 16 == 0;
    a.cpt = a.Cs / 16;
    a.magic_div = hq_magic32((unsigned)(aligned ? a.cpt : a.Cs));
    a.classed = dgrad && !(p->stride == 1 && p->R == p->S);
    if (!a.classed) {
        a.ncls = 1; a.ostep = 1; a.sgn = 1;
        a.istep = dgrad ? 1 : p->stride;
        KsClass &c = a.cls[0];
        c.ph = c.pw = 0; c.Hc = a.Ho; c.Wc = a.Wo; c.ns = p->S; c.taps = taps;
        c.dh = c.dw = dgrad ? -(p->R - 1 - p->pad) : -p->pad;
        c.w0 = dgrad ? taps - 1 : 0; a.wr = dgrad ? -p->S : p->S; a.wc = dgrad ? -1 : 1;
        c.magic_Wc = hq_magic32((unsigned)c.Wc); c.magic_Hc = hq_magic32((unsigned)c.Hc); c.magic_ns = hq_magic32((unsigned)c.ns);
    } else {
        const int S = p->stride;
        if (S > 4) return HQ_E_BADSHAPE;
        a.ncls = S * S; a.ostep = S; a.sgn = -1; a.istep = 1; a.wr = S * p->S; a.wc = S;
        for (int k = 0; k < a.ncls; k++) {
            KsClass &c = a.cls[k];
            c.ph = k / S; c.pw = k % S;
            c.Hc = (a.Ho - c.ph + S - 1) / S; c.Wc = (a.Wo - c.pw + S - 1) / S;
            const int r0 = (c.ph + p->pad) % S, s0 = (c.pw + p->pad) % S;
            const int nr = r0 < p->R ? (p->R - r0 + S - 1) / S : 0;
            c.ns = s0 < p->S ? (p->S - s0 + S - 1) / S : 0;
            c.taps = nr * c.ns;
            if (c.ns == 0) c.ns = 1;
            c.dh = (c.ph + p->pad - r0) / S; c.dw = (c.pw + p->pad - s0) / S;
            c.w0 = r0 * p->S + s0;
            c.magic_Wc = hq_magic32((unsigned)(c.Wc > 0 ? c.Wc : 1)); c.magic_Hc = hq_magic32((unsigned)(c.Hc > 0 ? c.Hc : 1));
            c.magic_ns = hq_magic32((unsigned)c.ns);
        }
    }
    if (sr_seed && out32) return HQ_E_BADARG;
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    a.m_fast = (size_t)a.N * a.wrow > (size_t)a.B * a.Hs * a.Ws * a.Cs;
    // Which tile.  While a launch is one round of tiles that run side by side its time is one tile's: the smallest tile that gives
    // every compute unit at most one is the fastest (over 1350 launches within 0.4 % of the best of the five).  Beyond one round the
    // tile kernels' larger tiles fetch fewer bytes per multiply-add.  (Strided input gradients of at most 64 channels would be
    // 256-pixel tiles over the whole reduction: 32 of them for 16x16x64 <- 8x8x128 at batch 32, 17 -> 7.6 us.)
    const size_t k = a.wrow / (a.classed ? (size_t)p->stride * p->stride : 1);      // reduction of an average tile
    auto tiles = [&](int tm, int tn) {
        unsigned long long m = 0;
        for (int c = 0; c < a.ncls; c++) m += ((unsigned long long)a.B * a.cls[c].Hc * a.cls[c].Wc + tm - 1) / tm;
        return m * (unsigned long long)((a.N + tn - 1) / tn);
    };
    if (!aligned) {
        // Microseconds of a launch by its rounds of 256 tiles and its reduction, for the tiles here and for the tile kernel (64-byte
        // stages of 4-byte loads, with few channels 256-pixel tiles), fitted to 830 launches of 1 .. 121 taps, 8 .. 2044 reduced and 4 ..
        // 2048 output channels in the three rounding modes: the choice costs 0.6 % over always the fastest, 2 launches in 100 are on
        // the wrong side by more than 5 %.  Forward, this / tile kernel: one tap, 2058 pixels -> 760, 244 reduced 10.6 / 11.8 us, 12996
        // -> 252, four taps of 120: 25.7 / 18.7; nine taps, 3136 -> 160, 5364 reduced 40.6 / 129, 11956 -> 252, 6840: 205 / 167; 49 taps,
        // 1152 -> 320, 392 reduced 6.8 / 16.6.
        const bool strided = a.classed && p->stride > 1;
        const double t32 = (double)tiles(32, 32);
        if (t32 <= (strided ? 512 : 256)) return launch2<2, 2, 8, 1, false>(a, mode, stream);
        if (!strided) {
            if (a.N > 64 && tiles(64, 64) > 512) return HQ_E_BADSHAPE;       // (98 launches: level in the mean)
            auto us = [&](int tm, int tn, double start, double round, double byte) {
                return start + (double)((tiles(tm, tn) + 255) / 256) * (round + byte * (double)k);
            };
            const double s32 = us(32, 32, 3.5, 1.25, 0.0054), s64x32 = us(64, 32, 4.5, 0.95, 0.0058), s64 = us(64, 64, 3.6, 2.0, 0.0076);
            const double sr = mode == 2 ? 1.0 : 0.0;
            const double tile = a.N <= 32 ? 6.9 + 0.036 * (double)k + 4.6 * sr : a.N <= 64 ? 5.5 + 0.034 * (double)k + 2.5 * sr :
                                k > 240 ? 6.6 + 0.0225 * (double)k + 2.9 * sr : us(128, 128, 5.9, 1.2, 0.0193) + 2.4 * sr;
            if (std::min({s32, s64x32, s64}) > tile) return HQ_E_BADSHAPE;
            if (s32 <= s64x32 && s32 <= s64) return launch2<2, 2, 8, 1, false>(a, mode, stream);
            if (s64x32 <= s64) return launch2<4, 2, 4, 1, false>(a, mode, stream);
            return launch2<4, 4, 4, 1, false>(a, mode, stream);
        }
        // Strided input gradients: the tile kernel walks every tap with a division test per word, so the line lies at short reductions.
        // The two sides are in proportion to what is left of a launch without its start-up (8 of 390 launches are on the wrong
        // side by more than 5 %).  1x1, 401408 pixels of 32, 36 reduced 28.2 / 26.9 us, 100: 30.0 / 42.5; 3x3, 119168 pixels of 128, 20
        // channels 56 / 31, 36: 56 / 57, 100: 69 / 114.
        const double t = (double)tiles(64, a.N <= 32 ? 32 : 64), stages = (double)((a.wrow + 63) / 64);
        const double g = (double)(a.N <= 64 ? tiles(256, 64) : tiles(128, 128)), per_class = (double)taps / (p->stride * p->stride);
        const double tile = std::max(1.0, g / 400) * ((mode == 1 ? 0 : 0.95) + (a.N <= 64 ? 9.8 : 6.2) * stages);
        const double split = std::max(1.0, t / (a.N <= 32 ? 100 : 80)) *
                             ((a.N <= 32 ? 0.55 : 1.0) + 0.43 * std::min(1.0, per_class) + 0.11 * per_class);
        if (split > tile) return HQ_E_BADSHAPE;
        if (a.N <= 32) return launch2<4, 2, 4, 1, false>(a, mode, stream);
        return launch2<4, 4, 4, 1, false>(a, mode, stream);
    }
    if (tiles(16, 16) <= 256) return launch2<1, 1, 8, 4, true>(a, mode, stream);
    if (tiles(16, 32) <= 256) return launch2<1, 2, 8, 4, true>(a, mode, stream);
    if (tiles(32, 32) <= 256) return launch2<2, 2, 8, 2, true>(a, mode, stream);
    if (tiles(32, 64) <= 256) return launch2<2, 4, 8, 2, true>(a, mode, stream);
    // One round is faster than the tile kernels whatever the reduction (this / tile kernel: nine taps of 16, 12887 pixels -> 64 5.7 /
    // 10.7 us, 25 taps of 96, 3840 -> 256 9.0 / 19.1, 49 taps of 16, 7584 -> 128 7.0 / 18.3; one tap of 64, 886 -> 1024 5.7 / 5.7, of 768, 1024
    // -> 1000 6.7 / 7.1), except for one tap of two or three 128-byte stages of the gather kernel's own 64 x 64 tiles (3136 -> 256, 256
    // reduced 5.8 / 5.0, 384: 6.1 / 5.5; 7056 -> 80, 560: 6.5 / 6.6).
    if (tiles(64, 64) <= 256 && !(taps == 1 && !a.classed && a.N > 64 && a.Cs >= 256 && a.Cs < 512))
        return launch2<4, 4, 8, 2, true>(a, mode, stream);
    // A second round where the tile kernels have 256-pixel tiles for it, as long as the reduction is long (19845 pixels -> 32, 1024 reduced
    // 8.7 / 14.1 us, 25480 -> 32, 256: 8.0 / 7.0; 24354 -> 64, 1024: 12.2 / 17.1, 32000 -> 64, 256: 10.3 / 8.7).
    if (a.N <= 64 && tiles(64, 64) <= 512 && k >= 1024)
        return a.N <= 32 ? launch2<2, 2, 8, 2, true>(a, mode, stream) : launch2<4, 4, 8, 2, true>(a, mode, stream);
    return HQ_E_BADSHAPE;
}
