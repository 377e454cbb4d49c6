// 3x3 layers of stride 1 and padding 1 with 128 or more channels on both sides, the reduced ones a multiple of 64: hq_gemm_fwd,
// hq_gemm_dgrad and pass 1 of the dynamic baseline.
//
//   out[m][n] = sum_{tap,c} A[pix(m,tap)][c] * Bw[n][tap][c]    (weight taps mirrored for the input gradient)
//
// What bounded these layers was the path into LDS: a gather kernel fetches every input byte once per tap, 64 bytes a clock of matrix
// work at 128 x 128 tiles, of which loads bring 28; row tiles fetch it once, but leave up to a quarter of a tile's rows empty.  Here
// a tile is any run of pixels, and its input is staged once per 64 channels as positions of framed images: a row has one position more
// than pixels, an image one row more, which hold the zero point's code and are the border on both sides, so that every tap is one offset
// for all pixels (a pixel's position is worked out once per tile, no tap is ever tested).  A workgroup of eight wavefronts owns 128 to 512
// pixels x 128 channels, one to a compute unit; a wavefront 32 to 128 pixels x 64 channels, so that a step of 32 channels reads 3 to 6
// fragments for 2 to 8 MFMAs.  A stage is one filter row x 64 channels, 24 KB of weights in one of three buffers, requested a stage ahead;
// the next 64 channels of the patch go into the other of two buffers two stages ahead.  All loads go straight to LDS, a few per step;
// one barrier per stage, 12 to 48 MFMAs of a wavefront apart.  A workgroup with another tile requests its first stages before it
// quantizes this one.
//
// Measured (before, with hq_ring_kernel or row tiles / now): 3x3 on 256 x 28 x 28 x 128 -> 128 50.3 / 38.7 us, batch 128 27.9 / 20.4, with
// stochastic rounding 33.6 / 27.9, 256 x 14 x 14 x 256 -> 256 42.7 / 31.0, 256 x 7 x 7 x 512 -> 512 38.4 / 32.4, 128 x 16 x 16 x 256 -> 256 25.1 /
// 22.5, 64 x 14 x 14 x 384 -> 384 29.7 / 21.3, 5 x 93 x 93 x 320 -> 320 90.9 / 49.7; 207 calls of 70 layers drawn at random 0.80 of the time.
// What bounds it now (256 x 14 x 14 x 256, tiles of 448): 6.2 K cycles until the first stage has arrived, 39.9 K of stages with 32.3 K of
// MFMAs per SIMD (34.1 K without the loads), 7.5 K of quantization (vector instructions), at 1.87 GHz, of which 2.2 to 2.3 are left where few
// compute units have a tile: the rest is the power that MFMAs on random bytes draw.  Smaller tiles read more LDS per MFMA: a stage takes
// 1.2 times its MFMAs at 512 pixels, 1.3 at 256, 1.9 at 128.  The barrier or the loads elsewhere in the stage, or the loads of a SIMD's two
// wavefronts apart, make no difference.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int FR_THREADS = 512, FR_BN = 128;
constexpr int FR_WSTAGE = 3 * FR_BN * 64;                               // weights of a stage: three taps x 128 filters x 64 channels

struct FrameArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    int M, N;                      // output pixels, channels
    int Cs, chunks;                // reduced channels; Cs / 64
    int B, H, W;
    int PW, image;                 // positions of a row and of an image of the frame: W + 1, (H + 1) * PW
    int blocks;                    // 16-position blocks of a tile's patch
    int w0, wr, wc;                // weight tap = w0 + wr * tap row + wc * tap column (mirrored: from the last one down)
    unsigned wrow;                 // bytes per weight row
    unsigned magic_W, magic_H;
    HqDivisor by_image, by_row;    // image and PW
    int m_tiles, n_tiles;
    HqSr sr;
};

// Four rows of two wavefronts; a wavefront has MA (rows 0, 1) or MB (rows 2, 3) 32-pixel blocks x 64 channels.  KA: patch blocks it loads.
template <int MODE, int MA, int MB, int KA>
__global__ __launch_bounds__(FR_THREADS) void hq_frame_kernel(const FrameArgs a)
{
    constexpr int BM = 64 * (MA + MB), NW = FR_THREADS / 64;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];       // [3] weights of a stage, [2] patch; no other LDS
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, r32 = lane & 31;
    const int wm = wave >> 1, wn = wave & 1;
    const unsigned patch0 = 3 * FR_WSTAGE, patch_bytes = 1024u * a.blocks;
    const int za = __builtin_amdgcn_readfirstlane(a.aq->zero_point);
    const int stages = 3 * a.chunks, tiles = a.m_tiles * a.n_tiles;

    auto frame = [&](int m) __attribute__((always_inline)) {            // position of an output pixel
        const unsigned t = hq_magic_div((unsigned)m, a.magic_W), b = hq_magic_div(t, a.magic_H);
        return (int)b * a.image + (int)(t - b * (unsigned)a.H) * a.PW + (int)((unsigned)m - t * (unsigned)a.W);
    };

    // ---- loads of a tile.  Weights: wavefront w loads filters 16 w .. of every tap; patch: 16 positions x 64 channels per load; lane l
    // lands at 16 * l, i.e. in row l / 4, the chunks of a row swizzled by bits 2 and 3 of its number
    const unsigned swizzled = 16u * ((unsigned)(lane & 3) ^ (unsigned)(lane >> 4 & 3));
    int m0, n0, p0;
    unsigned boff, wdst, pdst, ok;
    int lr, lc;                                                         // tap row and channel chunk of the next stage to load
    const int8_t *wb, *src[KA];
    auto next_weights = [&]() __attribute__((always_inline)) {
        wb = a.Bw + (ptrdiff_t)((a.w0 + lr * a.wr) * a.Cs + lc * 64);
        wdst = wdst >= 2 * FR_WSTAGE ? wdst - 2 * FR_WSTAGE : wdst + FR_WSTAGE;
        if (++lr == 3) { lr = 0; lc++; }
    };
    auto load_weights = [&](int s) __attribute__((always_inline)) { hq_lds_load16(wb + (ptrdiff_t)(s * a.wc) * a.Cs, boff, wdst + s * (FR_BN * 64)); };
    auto load_patch = [&](int k) __attribute__((always_inline)) {
        // (past the last block the first one again: every wavefront has KA loads in flight)
        const int kk = wave + NW * k < a.blocks ? k : 0;
        hq_lds_load16(src[k], pdst + 8192 * kk);
        src[k] += (ok >> k & 1) * 64;
    };
    auto begin_tile = [&](int t) __attribute__((always_inline)) {
        // consecutive workgroups go to the 8 XCDs in turn: each XCD gets a run of tiles, channel blocks of the same pixels together
        const int per = tiles / 8;
        if (t < per * 8) t = (t & 7) * per + (t >> 3);
        const int tile_m = t / a.n_tiles;
        m0 = tile_m * BM; n0 = (t - tile_m * a.n_tiles) * FR_BN;
        p0 = frame(m0);
        const int row = 16 * wave + (lane >> 2), n = n0 + (row & ~31) + hq_sigma32(row & 31);
        boff = (unsigned)(n < a.N ? n : 0) * a.wrow + swizzled;
        lr = 0; lc = 0; wdst = 2 * FR_WSTAGE + 1024u * wave; pdst = patch0 + 1024u * wave; ok = 0;
        next_weights();
#pragma unroll
        for (int s = 0; s < 3; s++) load_weights(s);
#pragma unroll
        for (int k = 0; k < KA; k++) {
            const int block = wave + NW * k < a.blocks ? wave + NW * k : wave;
            const unsigned q = (unsigned)(p0 + 16 * block + (lane >> 2) + a.image - a.PW - 1);
            const unsigned b1 = hq_quot2(q, a.by_image), rem = q - b1 * (unsigned)a.image;
            const unsigned y = hq_quot2(rem, a.by_row), x = rem - y * (unsigned)a.PW;
            const bool in = (b1 - 1u < (unsigned)a.B) & (y < (unsigned)a.H) & (x < (unsigned)a.W);
            src[k] = hq_source(in, a.A, (unsigned long long)(((b1 - 1u) * (unsigned)a.H + y) * (unsigned)a.W + x) * (unsigned)a.Cs + swizzled, hq_fill_rows.w[za & 0xff]);
            ok |= in ? 1u << k : 0u;
            load_patch(k);
        }
        pdst += patch_bytes;
        next_weights();
#pragma unroll
        for (int s = 0; s < 3; s++) load_weights(s);
    };
    begin_tile(blockIdx.x);

    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {1.0f, 0.0f, 0.0f, 0.0f, true};
    if (MODE != 0) ep = hq_make_epilogue(acc_scale, a.range);
    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;

    auto run = [&](auto blocks, int first) __attribute__((always_inline)) {     // of the wavefront: its 32-pixel blocks, the first one
        constexpr int MW = decltype(blocks)::value;
        unsigned woff[2];
#pragma unroll
        for (int ks = 0; ks < 2; ks++) woff[ks] = (64 * wn + r32) * 64 + 16 * ((2 * ks + half) ^ (r32 >> 2 & 3));
        auto lds = [&](unsigned off) __attribute__((always_inline)) { return *(const LDS_PTR(v4i))(off); };
        for (int tile = blockIdx.x;;) {
            // accumulators start at what the zero point adds to every output of a channel
            v16i acc[MW][2];
#pragma unroll
            for (int j = 0; j < 2; j++) {
                const int nb = n0 + 64 * wn + 32 * j + 16 * half;
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    const v4i bz = *reinterpret_cast<const v4i *>(a.bsum + (nb < a.N ? nb : 0) + 4 * g);     // (N % 16 == 0)
#pragma unroll
                    for (int e = 0; e < 4; e++)
#pragma unroll
                        for (int i = 0; i < MW; i++) acc[i][j][4 * g + e] = -za * bz[e];
                }
            }
            // fragments: row of the patch under tap (0, 0), a chunk of 16 channels
            unsigned arow[MW], addr[MW];
#pragma unroll
            for (int i = 0; i < MW; i++) arow[i] = (unsigned)(frame(min(m0 + 32 * (first + i) + r32, a.M - 1)) - p0) * 64 + 16 * half;
            v4i af[2][MW], wf[2][2];
            // pixel fragment i of k-step ks of a tap (its address is worked out with the first); weight fragment j
            auto read_a = [&](int ks, int i, unsigned tap) __attribute__((always_inline)) {
                if (ks == 0) { const unsigned t = arow[i] + tap; addr[i] = t ^ (t >> 4 & 0x30u); }
                af[ks][i] = lds(ks == 0 ? addr[i] : addr[i] ^ 32u);
            };
            auto read_w = [&](int ks, int j, unsigned wtap) __attribute__((always_inline)) { wf[ks][j] = lds(woff[ks] + wtap + j * 2048); };

            unsigned wcur = 0, pcur = patch0;
            asm volatile("s_waitcnt vmcnt(3)" ::: "memory");           // (and what the accumulators start from)
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MW; i++) read_a(0, i, pcur);
#pragma unroll
            for (int j = 0; j < 2; j++) read_w(0, j, wcur);

            int r = 0, c = 0;
            bool patches = false;                                       // the stage before requested a patch behind its weights
            for (int st = 0; st < stages; st++) {
                const unsigned tap0 = pcur + (unsigned)(r * a.PW) * 64;
                const bool last_row = r == 2, more_w = st + 2 < stages, more_p = r == 0 && c + 1 < a.chunks;
                const unsigned wnext = wcur + FR_WSTAGE >= 3 * FR_WSTAGE ? 0 : wcur + FR_WSTAGE;
                const unsigned pnext = last_row ? (pcur == patch0 ? patch0 + patch_bytes : patch0) : pcur;
                const unsigned tapn = pnext + (unsigned)((last_row ? 0 : r + 1) * a.PW) * 64;
#pragma unroll
                for (int step = 0; step < 6; step++) {
                    const int s = step >> 1, ks = step & 1, kn = ks ^ 1;    // the next step's fragments are read between the MFMAs
                    const unsigned tap = ks == 0 ? tap0 + 64 * s : s < 2 ? tap0 + 64 * (s + 1) : tapn;
                    const unsigned wtap = ks == 0 ? wcur + 8192 * s : s < 2 ? wcur + 8192 * (s + 1) : wnext;
#pragma unroll
                    for (int i = 0; i < MW; i++)
#pragma unroll
                        for (int j = 0; j < 2; j++) {
                            __builtin_amdgcn_sched_barrier(0);
                            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[ks][j], af[ks][i], acc[i][j], 0, 0, 0);
                            __builtin_amdgcn_sched_barrier(0);
                            if (j == 0) read_a(kn, i, tap);
                            else if (i < 2) read_w(kn, i, wtap);
                            if (MW == 1 && j == 1) read_w(kn, 1, wtap);
                        }
                    if (step == 1) {
                        // The next stage, requested one stage ago, is visible behind the barrier, and the stage before this one is free.  A
                        // patch, requested under tap row 0, is needed two stages later.
                        if (patches) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KA) : "memory");
                        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                        __syncthreads();
                        if (more_w) next_weights();
                        patches = more_p;
                    }
                    // (a few at a time: a wavefront that finds the path to LDS busy holds up its MFMAs)
                    if (step >= 1 && step <= 3 && more_w) load_weights(step - 1);
                    if (step >= 4 && more_p) {
#pragma unroll
                        for (int k = 0; k < KA; k++) if (k * 2 / KA == step - 4) load_patch(k);
                        if (step == 5) pdst = pdst >= patch0 + patch_bytes ? pdst - patch_bytes : pdst + patch_bytes;
                    }
                }
                wcur = wnext; pcur = pnext;
                if (last_row) { r = 0; c++; } else r++;
            }
            // the next tile's first loads run under this tile's epilogue (32-bit outputs need LDS for themselves)
            __syncthreads();
            const int me = m0, ne = n0;
            tile += gridDim.x;
            if (MODE != 0 && tile < tiles) begin_tile(tile);

            // 32 pixels x 32 channels: 16 consecutive channels of a pixel per lane
            auto epilogue = [&](auto full) __attribute__((always_inline)) {
                constexpr bool FULL = decltype(full)::value;
#pragma unroll
                for (int i = 0; i < MW; i++) {
                    const int m = me + 32 * (first + i) + r32;
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        const int nb = ne + 64 * wn + 32 * j + 16 * half;
                        int v[16];
#pragma unroll
                        for (int e = 0; e < 16; e++) v[e] = acc[i][j][e];
                        const bool in = m < a.M && nb < a.N;             // N % 16 == 0
                        const size_t o = (size_t)m * a.N + nb;
                        if constexpr (MODE == 0) {
                            // 32-bit outputs leave as whole lines: the block is turned in 4 KB of LDS, 16-byte pieces swizzled by the pixel
                            if (in) hq_minmax_group<16>(v, mn, mx);
                            v4i *turn = reinterpret_cast<v4i *>(smem) + wave * 256;
#pragma unroll
                            for (int g = 0; g < 4; g++) turn[r32 * 8 + ((4 * half + g) ^ (r32 & 7))] = v4i{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                            __builtin_amdgcn_wave_barrier();             // (LDS serves a wavefront's accesses in order)
                            const int piece = lane & 7, n = ne + 64 * wn + 32 * j + 4 * piece;
#pragma unroll
                            for (int t = 0; t < 4; t++) {
                                const int px = 8 * t + (lane >> 3), mt = me + 32 * (first + i) + px;
                                const v4i w = turn[px * 8 + (piece ^ (px & 7))];
                                if (mt < a.M && n < a.N) *reinterpret_cast<v4i *>(a.out32 + (size_t)mt * a.N + n) = w;
                            }
                            __builtin_amdgcn_wave_barrier();
                        } else if (in) {
                            int w[4];
                            if constexpr (MODE == 2) hq_requant_group_sr<16, FULL, 16>(v, ep, a.sr, o, mn, mx, nlo, nhi, w);
                            else                     hq_requant_group<16, FULL>(v, ep, mn, mx, nlo, nhi, w);
                            *reinterpret_cast<v4i *>(a.out8 + o) = v4i{w[0], w[1], w[2], w[3]};
                        }
                    }
                }
            };
            if (MODE == 0 || ep.full_grid) epilogue(std::true_type()); else epilogue(std::false_type());
            if (tile >= tiles) break;
            if (MODE == 0) { __syncthreads(); begin_tile(tile); }
        }
    };
    if constexpr (MA == MB) run(std::integral_constant<int, MA>(), MA * wm);
    else if (wm < 2) run(std::integral_constant<int, MA>(), MA * wm);
    else run(std::integral_constant<int, MB>(), 2 * MA + MB * (wm - 2));
    if (MODE == 0) __syncthreads();                                     // (otherwise behind the last tile's fragments: LDS is free for the statistics)
    hq_block_stats_commit_n<FR_THREADS>(mn, mx, nlo, nhi, a.st, reinterpret_cast<int *>(smem));
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)a.M * (unsigned long long)a.N);
        if (MODE != 0) *a.outq = a.range->qp;
    }
}

// 16-position blocks of the patch of any tile of `bm` pixels: its pixels, the extra column of every row and the extra row of every
// image that ends among them, and two rows and two positions for the taps.
int patch_blocks(const FrameArgs &a, int bm)
{
    const long rows = bm + ((bm - 2) / a.W + 1) + (long)a.PW * ((bm - 2) / ((long)a.H * a.W) + 1) + 2 * a.PW + 3;
    return (int)((rows + 15) / 16);
}

template <int MODE, int MA, int MB, int KA> int launch(FrameArgs &a, hipStream_t s)
{
    a.blocks = patch_blocks(a, 64 * (MA + MB));
    a.m_tiles = (a.M + 64 * (MA + MB) - 1) / (64 * (MA + MB));
    const size_t lds = 3 * FR_WSTAGE + 2048 * (size_t)a.blocks;
    static std::atomic<unsigned long long> allowed{0};
    if (!hq_allow_lds(hq_frame_kernel<MODE, MA, MB, KA>, 160 * 1024, allowed)) return HQ_E_HIP;
    hipLaunchKernelGGL((hq_frame_kernel<MODE, MA, MB, KA>), dim3((unsigned)std::min(a.m_tiles * a.n_tiles, 256)), dim3(FR_THREADS), lds, s, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}

template <int MODE> int launch_s(FrameArgs &a, int size, hipStream_t s)
{
    switch (size) {
    case 2: return launch<MODE, 1, 1, 4>(a, s);
    case 3: return launch<MODE, 2, 1, 4>(a, s);
    case 4: return launch<MODE, 2, 2, 5>(a, s);
    case 6: return launch<MODE, 3, 3, 5>(a, s);
    case 7: return launch<MODE, 4, 3, 6>(a, s);
    default: return launch<MODE, 4, 4, 6>(a, s);
    }
}

} // namespace

int hq_try_launch_frame(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                        const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8, int32_t *out32,
                        hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed)
{
    if (p->kind != HQ_CONV2D || p->R != 3 || p->S != 3 || p->stride != 1 || p->pad != 1) return HQ_E_BADSHAPE;
    FrameArgs a = {};
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    a.B = p->B; a.H = p->H; a.W = p->W;
    a.Cs = dgrad ? p->Cout : p->C; a.N = dgrad ? p->C : p->Cout;
    if (a.Cs % 64 != 0 || a.Cs < 128 || a.N % 16 != 0 || a.N < 128) return HQ_E_BADSHAPE;
    const unsigned long long M = (unsigned long long)p->B * p->H * p->W, lim = 1ull << 32;
    const unsigned long long positions = (unsigned long long)(p->B + 2) * (p->H + 1) * (p->W + 1);
    // operands of the divisions, 32-bit offsets into the weights
    if (M * (unsigned)std::max(a.H, a.W) >= lim || positions >= lim / 4 || (unsigned long long)a.N * 9 * a.Cs >= lim) return HQ_E_BADSHAPE;
    a.M = (int)M;
    a.chunks = a.Cs / 64;
    a.PW = a.W + 1; a.image = (a.H + 1) * a.PW;
    a.w0 = dgrad ? 8 : 0; a.wr = dgrad ? -3 : 3; a.wc = dgrad ? -1 : 1;
    a.wrow = 9u * (unsigned)a.Cs;
    a.magic_W = hq_magic32((unsigned)a.W); a.magic_H = hq_magic32((unsigned)a.H);
    a.by_image = hq_divisor((unsigned)a.image); a.by_row = hq_divisor((unsigned)a.PW);
    a.n_tiles = (a.N + FR_BN - 1) / FR_BN;
    if (sr_seed && out32) return HQ_E_BADARG;
    // The tile (64 s pixels) whose rounds of 256, one workgroup to a compute unit, take the fewest cycles: those of a stage and of a tile's end
    // from clock stamps.  Over 70 layers drawn at random the choice is within 4 % of the best size.
    static const int stage_cycles[9] = {0, 0, 1430, 1640, 2040, 0, 2940, 3340, 3700}, end_cycles[9] = {0, 0, 3700, 4100, 5500, 0, 7300, 7500, 9100};
    int size = 0;
    double best = 0.0;
    for (int s : {2, 3, 4, 6, 7, 8}) {
        if (patch_blocks(a, 64 * s) > (s >= 7 ? 44 : s >= 4 ? 40 : 32)) continue;        // LDS; blocks that eight wavefronts load
        const long tiles = (a.M + 64l * s - 1) / (64 * s) * a.n_tiles, rounds = (tiles + 255) / 256;
        const double t = (double)rounds * (3.0 * a.chunks * stage_cycles[s] + (sr_seed ? 3700.0 * s : end_cycles[s]));
        if (size == 0 || t < best) { size = s; best = t; }
    }
    if (size == 0) return HQ_E_BADSHAPE;
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    return out32 ? launch_s<0>(a, size, stream) : sr_seed ? launch_s<2>(a, size, stream) : launch_s<1>(a, size, stream);
}
