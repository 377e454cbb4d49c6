// 3x3, stride 1, padding 1 with 64 reduced channels (forward, input gradient as the stencil with mirrored taps, pass 1 of
// the dynamic baseline): the weights of 64 output channels live in REGISTERS for the whole launch.
//
// With both MFMA operands read from LDS a 64 x 64 wavefront tile needs 1 KB per MFMA, all that LDS delivers, and whatever
// else a phase does comes on top (the weights-in-LDS kernel: 28 us for 128 x 56 x 56 x 64 against 7 us of matrix work).
// 64 channels x 576 reduced bytes are 144 registers per lane; then only the pixels come from LDS, 1 KB for two MFMAs.
// A compute unit holds two wavefronts per SIMD: while one requantizes, the other multiplies.
//
// A unit is 256 consecutive output pixels, 32 per wavefront, of the tensor's [image][row][column] order, whatever rows and
// images it spans; a workgroup takes a run of units.  Their input is a stream of positions: image rows of W + 1 positions and images of
// H + 1 rows, one column and one row of padding between neighbours, so that every tap is a constant distance in the stream.  The
// positions go through a ring in LDS in blocks of 64, straight from global memory, as many as the next unit needs while this one is
// multiplied (the run's first pixel starts the ring; a position outside the images loads a row of the zero point).  The ring is four
// planes of 16 channels: a fragment's 32 positions are 512 consecutive bytes, without bank conflicts, and the taps of a filter row and the
// halves of the channels are immediate offsets from one address per filter row.  What the framed stream costs in positions (a unit
// of 3 x 3 images has 455) it costs only in loads: the matrix work is on pixels.  The ring holds two units of images up to 403 wide that have
// more than 510 pixels; every further image in two units is another extra row (one-row images: up to 241 wide, and 256 to 302).
//
// Before, patches of padded rows were copied through registers into two buffers, 1,000 of 4,950 clocks of a unit, for images up
// to 121 wide.  Measured, before -> now (us): 256 x 56 x 56 x 64 40.5 -> 38.3, 128 x 56 x 56 x 64 24.8 -> 23.2, 16 x 56 x 56 x 64 7.8 -> 7.2,
// 61 x 37 x 23 x 64 7.8 -> 7.2, 400 x 7 x 7 x 64 7.8 -> 6.7; wider images, then the general kernel's: 16 x 224 x 224 x 64 79.9 -> 36.4,
// 1 x 150 x 150 x 64 14.2 -> 6.8.  Bound by power where it fills the chip: with the requantization spread between the MFMAs a unit took
// 3,600 clocks instead of 4,600, and the launch as long as before, at a lower clock rate.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int RW_THREADS = 512, RW_UNIT = 256, RW_BLOCK = 64;           // pixels of a unit, 32 per wavefront; positions that are loaded together
constexpr int RW_RING = 1792;                                            // positions of the ring; its first block is repeated behind its end
constexpr int RW_PLANE = (RW_RING + RW_BLOCK) * 16;                     // bytes of a plane: 16 channels of every position
constexpr int RW_WEIGHTS = 64 * 9 * 64;

struct RegwArgs {
    const int8_t *A, *Bw;
    const int32_t *bsum;
    const hq_qparams *aq, *bq;
    const hq_range *range;
    int8_t *out8;
    int32_t *out32;
    hq_qparams *outq;
    hq_stats *st;
    HqFrame frame;
    int N;                         // output channels
    int flip;
    int units, nparts, runs;       // units; blocks of 64 channels; workgroups per channel block
    HqDivisor image, line;         // H * W and W
    HqFramePlace unit, loads;      // a unit's pixels as positions (p), rows and columns; four blocks of positions
    HqSr sr;
};

template <int MODE>
__global__ __launch_bounds__(RW_THREADS, 2) void hq_regw_kernel(const RegwArgs a)
{
    // four planes of 16 channels, the weights of 64 channels (chunks of 16 bytes swizzled by bits 2 and 3 of the row)
    extern __shared__ __attribute__((aligned(64))) int8_t smem[];
    __shared__ __attribute__((aligned(16))) int bias[64];
    __shared__ int red[4 * (RW_THREADS / 64)];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, r32 = lane & 31;

    const int run = __builtin_amdgcn_readfirstlane(blockIdx.x / a.nparts), n0 = (blockIdx.x - run * a.nparts) * 64;
    const int u_begin = (int)((long)a.units * run / a.runs), u_end = (int)((long)a.units * (run + 1) / a.runs);
    const unsigned lds0 = hq_lds_address(smem);
    constexpr unsigned wlds = 4 * RW_PLANE;

    // ---- weights of this workgroup's 64 channels: 36 KB in one piece
    {
        const int8_t *wsrc = a.Bw + (size_t)n0 * 576;
#pragma unroll
        for (int k = 0; k < 5; k++) {
            const int f = wave + 8 * k;                                  // 36 loads of 64 chunks
            const int q = 64 * f + lane, row = q / 36, ch = q - 36 * row;
            if (f < 36) hq_lds_load16(wsrc + row * 576 + 16 * (ch ^ (row >> 2 & 3)), lds0 + wlds + 1024u * f);
        }
    }

    // ---- input: 16 channels of 64 positions per load; a wavefront loads two planes of every fourth block.
    // The ring's place 0 is the first position under the run's first pixel, PW + 1 before the pixel's own.
    const HqFrame &f = a.frame;
    auto position = [&](unsigned k, int &y, int &x) __attribute__((always_inline)) {   // of a pixel
        const unsigned b = hq_quot(k, a.image), rem = k - b * (unsigned)(f.H * f.W);
        y = (int)hq_quot(rem, a.line);
        x = (int)(rem - (unsigned)y * (unsigned)f.W);
        return ((int)b * (f.H + 1) + y) * f.PW + x;
    };
    int y0, x0, oy, ox;
    const int origin = position((unsigned)(u_begin * RW_UNIT), y0, x0);
    unsigned place = (unsigned)(position((unsigned)(u_begin * RW_UNIT + 32 * wave + r32), oy, ox) - origin);     // of the lane's pixel's first tap
    auto needed = [&](int u) __attribute__((always_inline)) {           // blocks up to the unit's last position
        int y, x;
        return (unsigned)(position((unsigned)(min((u + 1) * RW_UNIT, f.M) - 1), y, x) + 2 * f.PW + 2 - origin) / RW_BLOCK + 1;
    };
    // the lane's next position to load
    HqFramePlace next = hq_frame_place(f, (unsigned)(origin + RW_BLOCK * (wave & 3) + lane));
    hq_frame_back(f, next);
    const int za = __builtin_amdgcn_readfirstlane(a.aq->zero_point);
    const int8_t *input = a.A + 32 * (wave >> 2);
    const int8_t *src;
    bool pending = true;                                                 // `src` has been used
    int second;                                                          // the other plane's distance: a position outside an image has one row of fill
    auto prepare = [&]() __attribute__((always_inline)) {
        const bool there = hq_frame_inside(f, next);
        src = hq_source(there, input, (unsigned long long)(unsigned)next.p * 64u, hq_fill_rows.w[za & 0xff]);
        second = there ? 16 : 0;
        hq_frame_advance(f, a.loads, next);
        pending = false;
    };
    unsigned block = wave & 3;                                           // the wavefront's next
    unsigned at = RW_BLOCK * (wave & 3);                                 // its place in the ring
    auto load = [&](unsigned end) __attribute__((always_inline)) {      // the wavefront's blocks before `end`, the first of them prepared
        while (block < end) {
            const unsigned to = lds0 + 2 * RW_PLANE * (wave >> 2) + at * 16;
            hq_lds_load16(src, to);
            hq_lds_load16(src + second, to + RW_PLANE);
            if (at == 0) {
                hq_lds_load16(src, to + RW_RING * 16);
                hq_lds_load16(src + second, to + RW_PLANE + RW_RING * 16);
            }
            at = at + 4 * RW_BLOCK >= RW_RING ? at + 4 * RW_BLOCK - RW_RING : at + 4 * RW_BLOCK;
            block += 4;
            pending = true;
            if (block < end) prepare();
        }
    };
    const int bz = tid < 64 ? a.bsum[n0 + tid] : 0;
    const float acc_scale = __fmul_rn(a.aq->scale, a.bq->scale);
    HqEpilogue ep = {};
    if (MODE != 0) {
        ep = hq_make_epilogue(acc_scale, a.range);
        auto uniform = [](auto &v) { v = __builtin_bit_cast(std::decay_t<decltype(v)>, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v))); };
        uniform(ep.mult); uniform(ep.flo); uniform(ep.fhi); uniform(ep.zoff); uniform(ep.c_hi); uniform(ep.c_lo);
    }
    prepare();
    load(needed(u_begin));
    if (pending) prepare();
    if (tid < 64) bias[tid] = -za * bz;

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const unsigned mine = lds0 + RW_PLANE * half;
    int mn = INT_MAX, mx = INT_MIN;
    unsigned nlo = 0, nhi = 0;
    int first = u_begin * RW_UNIT + 32 * wave;                           // the wavefront's first pixel of the unit that is finished next

    auto body = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;
        // (different statements keep the compiler from loading the weights ahead of the choice, where their registers would be laid out
        // for both forms of the loop at once, with spills in either)
        if (FULL) asm volatile("; whole grid" ::: "memory"); else asm volatile("; part of the grid" ::: "memory");
        constexpr int D = MODE == 2 ? 2 : 3;                             // fragment sets: taps ahead, and the one in use (3 would spill with the random bits)
        // Row i of a weight fragment is channel hq_sigma32(i), so that a lane ends up with 16 consecutive output channels; channel i for
        // 32-bit outputs, whose products are formed transposed (see finish32).
        v4i wf[9][2][2];
#pragma unroll
        for (int t = 0; t < 9; t++)
#pragma unroll
            for (int kc = 0; kc < 2; kc++)
#pragma unroll
                for (int nb = 0; nb < 2; nb++) {
                    const int row = 32 * nb + (MODE == 0 ? r32 : hq_sigma32(r32)), tap = a.flip ? 8 - t : t;
                    wf[t][kc][nb] = *reinterpret_cast<const v4i *>(smem + wlds + row * 576 + 16 * ((4 * tap + 2 * kc + half) ^ (row >> 2 & 3)));
                }
        v16i acc[2];
        v4i af[D][2];
        // the lane's place in its plane under the three filter rows; the taps of a row and the other half of the channels are constant distances
        unsigned row[3];
        auto rows = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int r = 0; r < 3; r++) {
                const unsigned k = place + (unsigned)(r * f.PW);
                row[r] = mine + 16 * min(k, k - RW_RING);               // (k < 2 * RW_RING)
            }
            ox += a.unit.x; oy += a.unit.y; place += (unsigned)a.unit.p;
            const bool cx = ox >= f.W;
            ox -= cx ? f.W : 0; oy += cx; place += cx;
            const bool cy = oy >= f.H;
            oy -= cy ? f.H : 0; place += cy ? (unsigned)f.PW : 0u;
            place = min(place, place - RW_RING);
        };
        auto fetch = [&](int t) __attribute__((always_inline)) {
            LDS_PTR(const int8_t) q = (LDS_PTR(const int8_t))(size_t)row[t / 3] + t % 3 * 16;
            af[t % D][0] = *(LDS_PTR(const v4i))q;
            af[t % D][1] = *(LDS_PTR(const v4i))(q + 2 * RW_PLANE);
        };
        auto begin = [&](int nb) __attribute__((always_inline)) {
            if constexpr (MODE == 0) {
                const int b = bias[32 * nb + r32];
#pragma unroll
                for (int e = 0; e < 16; e++) acc[nb][e] = b;
            } else
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const v4i b = *reinterpret_cast<const v4i *>(bias + 32 * nb + 16 * half + 4 * k);
#pragma unroll
                for (int e = 0; e < 4; e++) acc[nb][4 * k + e] = b[e];
            }
        };
        auto multiply = [&]() __attribute__((always_inline)) {
            rows();
            begin(0); begin(1);
#pragma unroll
            for (int t = 0; t < D - 1; t++) fetch(t);
#pragma unroll
            for (int t = 0; t < 9; t++) {
                if (t + D - 1 < 9) fetch(t + D - 1);
#pragma unroll
                for (int kc = 0; kc < 2; kc++)
#pragma unroll
                    for (int nb = 0; nb < 2; nb++) {
                        __builtin_amdgcn_sched_barrier(0);
                        acc[nb] = MODE == 0 ? __builtin_amdgcn_mfma_i32_32x32x32_i8(af[t % D][kc], wf[t][kc][nb], acc[nb], 0, 0, 0)
                                            : __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[t][kc][nb], af[t % D][kc], acc[nb], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        // the next address is worked out while the matrix cores are busy
                        if (t == 4 && kc == 0 && nb == 0 && pending) prepare();
                    }
            }
        };
        // 32-bit outputs: a lane holds one channel of 16 pixels, so a store of the wavefront writes two whole 128-byte lines (with 16
        // channels of one pixel a lane it would touch 64 lines, a quarter of each: 44 us against 30 for 128 x 56 x 56 x 64).
        auto finish32 = [&]() __attribute__((always_inline)) {
            const unsigned mine32 = (unsigned)(4 * half * a.N + r32);
            const bool whole = first + 32 <= f.M;
#pragma unroll
            for (int nb = 0; nb < 2; nb++) {
                int c[16];
#pragma unroll
                for (int e = 0; e < 16; e++) c[e] = acc[nb][e];
                int32_t *out = a.out32 + (size_t)(unsigned)first * a.N + n0 + 32 * nb;
                if (whole) hq_minmax_group<16>(c, mn, mx);
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    asm("" : "+s"(out));                                // (a uniform address and the lane's part, not 16 addresses)
                    if (whole) out[mine32] = c[e];
                    else if (first + 8 * (e >> 2) + (e & 3) + 4 * half < f.M) { out[mine32] = c[e]; mn = min(mn, c[e]); mx = max(mx, c[e]); }
                    out += e % 4 == 3 ? 5 * a.N : a.N;
                }
            }
        };
        // Returns whether all the wavefront's stores were issued.
        auto finish = [&]() __attribute__((always_inline)) {
            const bool whole = first + 32 <= f.M;
            const int pixel = first + r32;
            if constexpr (MODE == 0) {
                finish32();
            } else if (pixel < f.M) {
#pragma unroll
                for (int nb = 0; nb < 2; nb++) {
                    int c[16];
#pragma unroll
                    for (int e = 0; e < 16; e++) c[e] = acc[nb][e];
                    const size_t o = (size_t)(unsigned)pixel * a.N + n0 + 32 * nb + 16 * half;
                    int w[4];
                    if constexpr (MODE == 2) hq_requant_group_sr<16, FULL, 16>(c, ep, a.sr, o, mn, mx, nlo, nhi, w);
                    else                     hq_requant_group<16, FULL>(c, ep, mn, mx, nlo, nhi, w);
                    *reinterpret_cast<v4i *>(a.out8 + o) = v4i{w[0], w[1], w[2], w[3]};
                }
            }
            first += RW_UNIT;
            return whole;
        };
        // Between two barriers one of a SIMD's two wavefronts multiplies first and requantizes then, the other (`late`)
        // requantizes its unit before and then multiplies, so that the matrix cores and the vector ALU both have work.
        const bool late = wave >= RW_THREADS / 128;
        bool stored = false;                                            // a unit's stores since the last loads
        for (int u = u_begin; u < u_end; u++) {
            // this wavefront's blocks of the unit are in LDS once only the stores issued after them are under way
            if (stored) asm volatile("s_waitcnt vmcnt(%0)" :: "n"(MODE == 0 ? 32 : 2) : "memory");
            else        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (u + 1 < u_end) load(needed(u + 1));
            stored = false;
            if (late && u > u_begin) stored = finish();
            multiply();
            if (!late) stored = finish();
        }
        if (late && u_end > u_begin) finish();
    };
    if (MODE == 0 || ep.full_grid) body(std::true_type()); else body(std::false_type());
    hq_block_stats_commit_n<RW_THREADS>(mn, mx, nlo, nhi, a.st, red);
    if (blockIdx.x == 0 && tid == 0) {
        a.st->acc_scale = acc_scale;
        atomicAdd((unsigned long long *)&a.st->count, (unsigned long long)f.M * (unsigned long long)a.N);
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
    if ((unsigned long long)p->B * (H + 1) * (W + 1) >= (1ull << 31) - 4096) return HQ_E_BADSHAPE;      // (positions are ints)
    // the ring holds a unit's positions and the next one's, blocks loaded as wholes
    const int lines = (2 * RW_UNIT - 2) / W + 1, images = (2 * RW_UNIT - 2) / (H * W) + 1;
    if (2 * RW_UNIT + lines + images * (W + 1) + 2 * (W + 1) + 2 + RW_BLOCK > RW_RING) return HQ_E_BADSHAPE;
    RegwArgs a = {};
    a.frame = hq_frame(p->B, H, W);
    a.A = A; a.Bw = Bw; a.bsum = bsum; a.aq = aq; a.bq = bq; a.range = range;
    a.out8 = out8; a.out32 = out32; a.outq = outq; a.st = st;
    a.N = N; a.flip = dgrad;
    a.units = (int)((M + RW_UNIT - 1) / RW_UNIT);
    a.nparts = N / 64;
    a.runs = 256 / a.nparts;
    if (a.runs < 1) a.runs = 1;
    if (a.runs > a.units) a.runs = a.units;
    const int image = H * W;
    a.image = hq_divisor((unsigned)image); a.line = hq_divisor((unsigned)W);
    a.unit.y = RW_UNIT % image / W; a.unit.x = RW_UNIT % image % W;
    a.unit.p = RW_UNIT / image * (H + 1) * (W + 1) + a.unit.y * (W + 1) + a.unit.x;
    a.loads = hq_frame_distance(a.frame, 4 * RW_BLOCK);
    if (sr_seed && out32) return HQ_E_BADARG;
    a.sr = sr_seed ? HqSr{(unsigned)*sr_seed, (unsigned)(*sr_seed >> 32)} : HqSr{0, 0};
    const int mode = out32 ? 0 : sr_seed ? 2 : 1;
    auto kern = mode == 0 ? hq_regw_kernel<0> : mode == 2 ? hq_regw_kernel<2> : hq_regw_kernel<1>;
    constexpr size_t lds = 4 * RW_PLANE + RW_WEIGHTS;
    static std::atomic<unsigned long long> allowed[3];
    if (!hq_allow_lds(kern, lds, allowed[mode])) return HQ_E_HIP;
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.runs * a.nparts)), dim3(RW_THREADS), lds, stream, a);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}
