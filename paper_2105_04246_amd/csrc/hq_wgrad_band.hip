// Weight gradient of 3x3 stride-1 layers (padding 1, channel counts multiples of 64): the shape of most layers of the paper's
// networks (Table 5; ResNet-18 basic blocks).
//
//   acc[n][tap][c] = sum_m  G[m][n] * Xg[m][tap][c]          m = (b, y, x) over all output pixels
//
// The reduction runs over positions of images with a frame: a row has one position more than the image has pixels, an image one row
// more, so that position k of the gradient meets position k + r * PW + s of the input under tap (r, s), PW = W + 1.  The extra
// column is the right border of its row and the left border of the next one, the extra row the lower border of its image and the
// upper border of the next one.  The gradient is 0 there, so those positions add nothing.  (Share of idle positions: 4 % for 56 x 56
// images, 7 % for 28 x 28, 13 % for 14 x 14, 23 % for 7 x 7.)  What this buys: the nine views are plain offsets, without a table, and the
// three taps of a filter row are the same bytes shifted by one: a lane reads 24 consecutive positions of its channel through the
// transposing read (ds_read_b64_tr_b8, three of them) and forms the fragments of all three taps with byte shifts, where each
// tap takes two transposing reads of its own otherwise.
//
// A workgroup owns a 64 (Cout) x 32 (C) block of G_W for all nine taps and walks a run of positions in chunks of 384.  Twelve wavefronts,
// three to a SIMD: two groups take alternate 32-position steps; a wavefront of a group owns one filter row and one 32-block of Cout:
// 5 transposing reads, 8 byte shifts and 3 MFMAs a step.  Chunks come from global memory straight into LDS, the input into a ring (every
// position is fetched once per run; the ring's start is repeated behind its end, so that a chunk's addresses are constants), the
// gradient into three buffers, requested one chunk before they are needed; gradient rows of 64 bytes, whose two 32-byte halves are
// swapped in every second group of four rows, so that the 16 rows x 32 bytes of a transposing read meet all banks.  There is one barrier
// per chunk, behind its first step: it makes the next chunk visible and frees the chunk before.
//
// Measured (whole call; before, with a table of patch rows, 64 x 64 blocks and an exchange of 147 KB at the end / now): 3x3 on
// 256 x 56 x 56 x 64 -> 64 60.5 / 43.8 us, batch 128 40.6 / 28.9, 256 x 28 x 28 x 128 -> 128 67.3 / 43.7, 256 x 14 x 14 x 256 -> 256
// 58.0 / 44.8, 256 x 7 x 7 x 512 -> 512 59.0 / 50.1, 64 x 14 x 14 x 384 -> 384 64.4 / 32.8, 3 x 112 x 112 x 64 -> 64 25.4 / 15.1.  What bounds
// it now (first shape, 38 us in this kernel): 46 K cycles of steps, of which the matrix pipes are busy for 29 K, at 1.75 GHz: without
// its loads the loop takes 35 K cycles, but at 1.71 GHz, i.e. it draws all the power there is; 6 K cycles until the first chunk has
// arrived, 4 K to add the groups and store.  64 x 64 blocks take 3 K cycles less in the loop, but twice the partial sums cost that and
// 3 us more (46.9 us); requesting loads two chunks ahead changes nothing.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace {

constexpr int WB_WAVES = 12, WB_THREADS = 64 * WB_WAVES;
constexpr int GROUPS = 2;                     // groups of six wavefronts that take the 32-position steps in turn
constexpr int STEPS = 6;                      // steps of a group per chunk
constexpr int L = 32 * STEPS * GROUPS;        // positions per chunk
constexpr int UNIT = 64 * GROUPS, UNITS = STEPS / 2;     // positions of two steps of either group; a chunk's units
constexpr int XROW = 32, GROW = 64;           // bytes of a row: 32 channels of the input, 64 of dY
constexpr int XLOAD = 1024 / XROW, GLOAD = 1024 / GROW;  // positions of a wavefront's load
constexpr int GLOADS = L / GLOAD / WB_WAVES;  // loads of the gradient per wavefront and chunk
constexpr int TAIL = L + 64;                  // rows of the ring's start that are repeated behind its end
constexpr unsigned GBYTES = 3 * L * GROW;     // the three buffers of the gradient
constexpr int SLOT_V4 = 2 * 9 * 4 * 64;       // 16-byte words of one workgroup's partial sums
constexpr int SUMS = 64 + 9 * 32;             // column sums that a workgroup may form: dY [64], input [9][32]
constexpr int EXCHANGE = WB_WAVES * 6 * 1024; // LDS bytes in which the groups' sums meet
static_assert(L == XLOAD * WB_WAVES && GLOADS * GLOAD * WB_WAVES == L, "one load of the input per wavefront and chunk");

struct WbandArgs {
    const int8_t *X, *G;
    const hq_qparams *xq, *gq;
    int32_t *partial;              // [slot][SLOT_V4] 16-byte words: a workgroup's 64 x 9 x 32 sums
    int32_t *gsums, *xsums;        // [run][N], [run][9][C]: column sums of dY and of the input taps
    HqFrame frame;
    int C, N;                      // channels of input and gradient
    HqFramePlace gstep, xstep;     // from one load to the next
    int units, per_block, splits;  // runs are cut at units of two steps of every group
    int cparts, nparts;            // C / 32, N / 64
    int lead;                      // chunks by which the input is ahead of the gradient: those of 2 * PW + 2 positions and a read's overhang
    unsigned ring;                 // bytes of the input's ring: (lead + 3) chunks
};

__global__ __launch_bounds__(WB_THREADS) void hq_wgrad_band_kernel(const WbandArgs a)
{
    // input ring, gradient buffers, [3][L] position masks.  The kernel has no other LDS, so offsets from its start are addresses.
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave / 6, gw = wave - 6 * grp, fr = gw >> 1, nblk = gw & 1;     // group, filter row, 32-block of Cout

    // workgroup -> (output block, run of chunks); the blocks of one run sit on one XCD
    int part, split;
    {
        const int per = a.cparts * a.nparts, total = per * a.splits;
        const int full = (total / (8 * per)) * (8 * per);
        if ((int)blockIdx.x < full) {
            const int g8 = blockIdx.x / (8 * per), r = blockIdx.x % (8 * per);
            split = g8 * 8 + (r & 7); part = r >> 3;
        } else {
            const int r = blockIdx.x - full;
            split = full / per + r / per; part = r % per;
        }
    }
    const int cp = part % a.cparts, np = part / a.cparts;
    const int units = min(a.units - split * a.per_block, a.per_block), n = (units + UNITS - 1) / UNITS;     // of this run, at least 1; chunks
    const unsigned begin = (unsigned)(split * a.per_block) * UNIT;

    // ---- loads: a wavefront brings 16 positions x 64 channels of dY, 1 KB of the input; lane l lands at 16 * l
    const int grow = lane >> 2, xrow = lane / (XROW / 16);
    const int gchunk = 16 * ((lane & 3) ^ (grow & 4 ? 2 : 0)), xchunk = 16 * (lane & 1);
    // the lane's next position, of the gradient and of the input, PW + 1 positions before
    HqFramePlace gpl = hq_frame_place(a.frame, begin + (unsigned)(GLOAD * wave + grow));
    HqFramePlace xpl = hq_frame_place(a.frame, begin + (unsigned)(XLOAD * wave + xrow));
    hq_frame_back(a.frame, xpl);
    const unsigned gbase = a.ring + TAIL * XROW, mbase = gbase + GBYTES;
    const int zx = __builtin_amdgcn_readfirstlane(a.xq->zero_point);
    const int8_t *xfill = reinterpret_cast<const int8_t *>(hq_fill_rows.w[zx & 0xff]), *gfill = reinterpret_cast<const int8_t *>(hq_fill_rows.w[0]);
    const int8_t *Xc = a.X + cp * XROW, *Gn = a.G + np * 64;
    // a column sum is only ever multiplied by the other operand's zero point (the finalize kernel's correction terms): with that
    // zero point at 0 it is not formed at all
    const bool do_gsum = cp == 0 && fr == 0 && zx != 0, xsums = np == 0 && __builtin_amdgcn_readfirstlane(a.gq->zero_point) != 0;
    unsigned xdst = 1024u * wave, gdst = gbase + 1024u * wave;         // where the wavefront's next loads go
    // A load is worked out in the shadow of the matrix cores, long before it is requested: behind the barrier, where all wavefronts
    // request theirs at once, that arithmetic would hold up the MFMAs.
    const int8_t *xsrc, *gsrc[GLOADS];
    bool gin[GLOADS];
    auto prepare_x = [&]() __attribute__((always_inline)) {
        xsrc = hq_source(hq_frame_inside(a.frame, xpl), Xc, (unsigned long long)(unsigned)xpl.p * (unsigned)a.C + (unsigned)xchunk, xfill);
        hq_frame_advance(a.frame, a.xstep, xpl);
    };
    auto prepare_g = [&](int i) __attribute__((always_inline)) {
        gin[i] = hq_frame_inside(a.frame, gpl);
        gsrc[i] = hq_source(gin[i], Gn, (unsigned long long)(unsigned)gpl.p * (unsigned)a.N + (unsigned)gchunk, gfill);
        hq_frame_advance(a.frame, a.gstep, gpl);
    };
    auto load_x = [&]() __attribute__((always_inline)) {
        hq_lds_load16(xsrc, xdst);
        if (xdst < TAIL * XROW) hq_lds_load16(xsrc, xdst + a.ring);
        xdst += L * XROW;
        xdst = xdst >= a.ring ? xdst - a.ring : xdst;
    };
    auto load_g = [&](bool masks) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GLOADS; i++) {
            hq_lds_load16(gsrc[i], gdst);
            if (masks && (lane & 3) == 0) smem[mbase + (gdst - gbase) / 64 + grow] = gin[i];
            gdst += GLOAD * WB_WAVES * GROW;
            gdst = gdst >= mbase ? gdst - GBYTES : gdst;
        }
    };
    auto prepare_gs = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GLOADS; i++) prepare_g(i);
    };
    prepare_gs();
    load_g(xsums);
    for (int i = 0; i <= a.lead; i++) { prepare_x(); load_x(); }
    prepare_x();
    load_x();
    prepare_gs();
    load_g(xsums);                                                      // (past the run: the next run's, or fill rows)
    prepare_x();
    prepare_gs();

    v16i acc[3];
#pragma unroll
    for (int s = 0; s < 3; s++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[s][e] = 0;
    int gsv = 0, xsv[3] = {0, 0, 0};

    // ---- fragments.  Lane l takes channel l % 32 and the 16 positions of half l / 32; it hands in row j / 2 of eight, 8 bytes of it.
    // (rows of 64 bytes: their halves are swapped by bit 2 of the row's number, which steps of 8 positions and the rings' lengths leave
    // alone).  The step's place in the ring is the same for all lanes; a lane is at most 39 rows behind it, hence the ring's tail.
    const int j16 = lane & 15, half = lane >> 5, row = 16 * half + (j16 >> 1), fcol = 16 * ((lane >> 4) & 1) + 8 * (j16 & 1);
    const int xfirst = 32 * grp + fr * a.frame.PW;
    const unsigned xlane = row * XROW + fcol;
    const unsigned glane = gbase + (32 * grp + row) * 64 + 32u * ((unsigned)nblk ^ ((unsigned)row >> 2 & 1)) + fcol;
    unsigned xat = (unsigned)xfirst * XROW, gat = 0, mat = 0;           // the chunk's places in the ring and in the buffers
    auto tr = [&](unsigned off) __attribute__((always_inline)) { return __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(off)); };
    unsigned xo, go;
    auto next_chunk = [&](int k) __attribute__((always_inline)) {
        xat += k * L * XROW;
        xat = min(xat, xat - a.ring);                                   // (below twice the ring: the smaller one is the place in it)
        gat = gat + k * L * 64 == GBYTES ? 0 : gat + k * L * 64;
        xo = xlane + xat; go = glane + gat;
    };
    auto fragments = [&](int k, v4i &g, unsigned (&w)[5]) __attribute__((always_inline)) {      // of the chunk's k-th step of this group
        const int dx = k * GROUPS * 32 * XROW, dg = k * GROUPS * 32 * 64;
        const tr_v2i g0 = tr(go + dg), g1 = tr(go + dg + 8 * 64), x0 = tr(xo + dx), x1 = tr(xo + dx + 8 * XROW), x2 = tr(xo + dx + 16 * XROW);
        g = v4i{g0[0], g0[1], g1[0], g1[1]};
        w[0] = (unsigned)x0[0]; w[1] = (unsigned)x0[1]; w[2] = (unsigned)x1[0]; w[3] = (unsigned)x1[1]; w[4] = (unsigned)x2[0];
    };
    // GS, XS: the wavefront forms the column sums of dY / of its input taps (behind the MFMAs of their own fragments, in the shadow
    // of the matrix cores)
    // One step.  Between two MFMAs stands what runs while the first is carried out; nothing moves across.
    auto step = [&](auto gs, auto xs, int k, const v4i &g, const unsigned (&w)[5], v4i &gn, unsigned (&wn)[5]) __attribute__((always_inline)) {
        constexpr bool GS = decltype(gs)::value, XS = decltype(xs)::value;
        v4i mask = {0, 0, 0, 0}, xf;
        if (XS) mask = *reinterpret_cast<const v4i *>(smem + mbase + mat + 32 * (k * GROUPS + grp) + 16 * half);
#pragma unroll
        for (int s = 0; s < 3; s++) {
#pragma unroll
            for (int d = 0; d < 4; d++) xf[d] = s == 0 ? (int)w[d] : (int)__builtin_amdgcn_alignbyte(w[d + 1], w[d], s);
            __builtin_amdgcn_sched_barrier(0);
            acc[s] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g, xf, acc[s], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (s == 0) fragments((k + 1) % STEPS, gn, wn);
            if (s == 1 && k == 1) prepare_x();
            if (s == 1 && k == 4) prepare_g(0);
            if (s == 1 && k == 5 && GLOADS == 2) prepare_g(GLOADS - 1);
            if (XS) {
#pragma unroll
                for (int d = 0; d < 4; d++) xsv[s] = __builtin_amdgcn_sdot4(xf[d], mask[d], xsv[s], false);
            }
            if (GS && s == 1) {
#pragma unroll
                for (int d = 0; d < 4; d++) gsv = __builtin_amdgcn_sdot4(g[d], 0x01010101, gsv, false);
            }
        }
    };
    v4i gA, gB;
    unsigned wA[5], wB[5];
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(1 + GLOADS) : "memory");
    __syncthreads();
    next_chunk(0);
    fragments(0, gA, wA);
    auto walk = [&](auto gs, auto xs) __attribute__((always_inline)) {
        constexpr bool XS = decltype(xs)::value;
        const int full = units / UNITS, rest = units - full * UNITS;
        for (int c = 0; c < full; c++) {
            const bool more = c + 2 < n;
#pragma unroll
            for (int k = 0; k < STEPS; k += 2) {
                step(gs, xs, k, gA, wA, gB, wB);
                if (k == 0) {
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the next chunk, requested one chunk ago
                    __syncthreads();
                    if (more) load_x();
                }
                // (not all at once: a wavefront whose load finds the path to LDS busy holds up its MFMAs)
                if (k == 2 && more) load_g(XS);
                if (k + 2 == STEPS) next_chunk(1);
                step(gs, xs, k + 1, gB, wB, gA, wA);                    // (behind the last step fragments that are never used)
            }
            if (XS) mat = mat + L == 3 * L ? 0 : mat + L;
        }
        // the run's last, incomplete chunk
        for (int r = 0; r < rest; r++) {
            step(gs, xs, 0, gA, wA, gB, wB);
            step(gs, xs, 1, gB, wB, gA, wA);
            xo += 2 * GROUPS * 32 * XROW; go += 2 * GROUPS * 32 * 64; mat += 2 * GROUPS * 32;
        }
    };
    if (xsums) walk(std::true_type(), std::true_type());               // (an asymmetric gradient; sums nobody reads are dropped)
    else if (do_gsum) walk(std::true_type(), std::false_type());
    else walk(std::false_type(), std::false_type());

    // ---- two groups are added through LDS, each finishing half of the sums, and a workgroup's sums go to a slot of its own with plain
    // 16-byte stores: partial[slot][32-block of Cout][tap][r / 4][lane / 32][c][r % 4].  The finalize kernel adds the slots; merging with
    // atomics instead would queue every workgroup of the launch on the same lines.
    const size_t slot = (size_t)split * (a.cparts * a.nparts) + part;
    v4i *pout = reinterpret_cast<v4i *>(a.partial) + slot * SLOT_V4 + ((nblk * 9 + 3 * fr) * 4) * 64 + half * 32 + (lane & 31);
    auto quad = [&](int k) __attribute__((always_inline)) {
        return v4i{acc[k >> 2][4 * (k & 3)], acc[k >> 2][4 * (k & 3) + 1], acc[k >> 2][4 * (k & 3) + 2], acc[k >> 2][4 * (k & 3) + 3]};
    };
    int *csum = reinterpret_cast<int *>(smem + EXCHANGE);            // [GROUPS][SUMS]
    // A run shorter than a chunk has not waited for the second set of loads that was requested for it, which may land where the sums
    // meet (the barrier does not wait for them); every other run has none under way.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (do_gsum) {
        const int sm = gsv + __shfl_xor(gsv, 32);
        if (lane < 32) csum[grp * SUMS + nblk * 32 + lane] = sm;
    }
    if (xsums && nblk == 0) {
#pragma unroll
        for (int s = 0; s < 3; s++) {
            const int sm = xsv[s] + __shfl_xor(xsv[s], 32);
            if (lane < 32) csum[grp * SUMS + 64 + (3 * fr + s) * 32 + lane] = sm;
        }
    }
    v4i *xch = reinterpret_cast<v4i *>(smem);                           // [12 wavefronts][6][64]
    const int other = wave + (grp ? -6 : 6);
#pragma unroll
    for (int k = 0; k < 6; k++) xch[(other * 6 + k) * 64 + lane] = grp ? quad(k) : quad(6 + k);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 6; k++) pout[(6 * grp + k) * 64] = (grp ? quad(6 + k) : quad(k)) + xch[(wave * 6 + k) * 64 + lane];
    // (what was not formed is neither read by the finalize kernel)
    if ((cp == 0 && zx != 0) || xsums)
        for (int i = tid; i < SUMS; i += WB_THREADS) {
            int sm = 0;
#pragma unroll
            for (int g = 0; g < GROUPS; g++) sm += csum[g * SUMS + i];
            const int x = i - 64;
            if (x < 0) { if (cp == 0) a.gsums[(size_t)split * a.N + np * 64 + i] = sm; }
            else if (xsums) a.xsums[((size_t)split * 9 + (x >> 5)) * a.C + cp * 32 + (x & 31)] = sm;
        }
}

// Adds the workgroups' partial sums (64 threads along C, TY taking every TY-th slot), removes the zero points and scales.
// One thread owns 4 consecutive output channels of one (tap, c): the 16 bytes a lane of the band kernel stored.
template <int TY>
__global__ __launch_bounds__(64 * TY) void wband_finalize_kernel(const int32_t *partial, const int32_t *gsums, const int32_t *xsums,
                                                              const hq_qparams *xq, const hq_qparams *gq, unsigned M,
                                                              int N, int C, int splits, float *dW, int32_t *dW_acc,
                                                              const HqRideAlong ride)
{
    if (hq_ride_along(ride)) return;
    __shared__ v4i sh[TY][64];
    __shared__ int shx[TY][64], shg[TY][4];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int cparts = C / 32, parts = cparts * (N / 64);
    const size_t o = (size_t)blockIdx.x * 64 + tx;                 // (n / 4, tap, c), c fastest
    const int c = (int)(o % C), tap = (int)((o / C) % 9), n0 = (int)(o / ((size_t)9 * C)) * 4;
    const int cp = c / 32, cc = c & 31, np = n0 / 64, i = (n0 >> 5) & 1, rq = (n0 >> 3) & 3, lh = (n0 >> 2) & 1;
    const v4i *src = reinterpret_cast<const v4i *>(partial) + (size_t)(np * cparts + cp) * SLOT_V4 +
                     ((i * 9 + tap) * 4 + rq) * 64 + lh * 32 + cc;
    const int *xsrc = xsums + (size_t)tap * C + c, *gsrc = gsums + n0;
    // a column sum is only ever multiplied by the other operand's zero point: with that at 0 it is neither formed
    // by the band kernel nor read here (uniform branches)
    const bool need_xs = gq->zero_point != 0, need_gs = xq->zero_point != 0;
    v4i gs = {0, 0, 0, 0};                                         // (the same four for the whole workgroup, whose threads share the slots)
    if (need_gs)
        for (int s = threadIdx.x; s < splits; s += 64 * TY) gs += *reinterpret_cast<const v4i *>(gsrc + (size_t)s * N);
    v4i sum = {0, 0, 0, 0};
    int xs = 0;
#pragma unroll 4
    for (int s = ty; s < splits; s += TY) sum += src[(size_t)s * parts * SLOT_V4];
    if (need_xs)
        for (int s = ty; s < splits; s += TY) xs += xsrc[(size_t)s * 9 * C];
    if (need_gs) {
#pragma unroll
        for (int e = 0; e < 4; e++) gs[e] = hq_wave_reduce(gs[e], HqAdd());
    }
    sh[ty][tx] = sum; shx[ty][tx] = xs;
    if (tx < 4) shg[ty][tx] = tx == 0 ? gs[0] : tx == 1 ? gs[1] : tx == 2 ? gs[2] : gs[3];
    __syncthreads();
    if (ty != 0) return;
    int g4[4] = {0, 0, 0, 0};
#pragma unroll
    for (int y = 1; y < TY; y++) { sum += sh[y][tx]; xs += shx[y][tx]; }
#pragma unroll
    for (int y = 0; y < TY; y++)
#pragma unroll
        for (int e = 0; e < 4; e++) g4[e] += shg[y][e];
    const unsigned zx = (unsigned)xq->zero_point, zg = (unsigned)gq->zero_point;
    const float sc = __fmul_rn(xq->scale, gq->scale);
    const size_t K = (size_t)9 * C, k = (size_t)tap * C + c;
    const unsigned xterm = zg * (unsigned)xs, both = M * zx * zg;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const unsigned v = (unsigned)sum[e] - zx * (unsigned)g4[e] - xterm + both;
        const size_t idx = (size_t)(n0 + e) * K + k;
        if (dW_acc) dW_acc[idx] = (int)v;
        dW[idx] = __fmul_rn(sc, (float)(int)v);
    }
}

// Geometry of the band kernel for one layer (host, pure); covered == false: the tile kernel takes it.  Its workspace is one slot per run and
// block of G_W and nothing else: up to 256 slots (18.9 MB and the column sums) while blocks are split, and with one run for every block the
// size of G_W and its column sums, what the tile kernel's accumulator takes, so that a bounded workspace holds the same layers for both.
struct WbandPlan {
    bool covered;
    int units, per_block, splits, parts, lead;
    unsigned ring;
    size_t lds, partial_bytes, gsums_bytes, xsums_bytes;
};

WbandPlan wband_plan(const hq_problem *p)
{
    WbandPlan pl = {};
    if (p->kind != HQ_CONV2D || p->R != 3 || p->S != 3 || p->stride != 1 || p->pad != 1) return pl;
    if (p->C % 64 != 0 || p->Cout % 64 != 0) return pl;
    const unsigned long long positions = (unsigned long long)p->B * (p->H + 1) * (p->W + 1);
    if (positions >= 1ull << 30) return pl;                           // (hq_quot2, with room for what is requested past the end)
    pl.lead = (2 * (p->W + 1) + 10 + L - 1) / L;
    pl.ring = (unsigned)(pl.lead + 3) * L * XROW;
    pl.lds = std::max((size_t)pl.ring + TAIL * XROW + GBYTES + 3 * L, (size_t)EXCHANGE + GROUPS * SUMS * 4);
    if (pl.lds > 160 * 1024) return pl;
    pl.parts = (p->C / 32) * (p->Cout / 64);
    pl.units = (int)((positions + UNIT - 1) / UNIT);
    // One workgroup per compute unit; but a unit takes 0.5 us and another slot of partial sums, written and read back, 0.03 us, so that
    // runs shorter than sqrt(0.04 * slots per run length of one) cost more in slots than they save.
    const int fill = std::max(1, 256 / pl.parts), even = (pl.units + fill - 1) / fill;
    pl.per_block = std::max(even, (int)std::sqrt(0.06 * pl.parts * (double)pl.units));
    pl.splits = (pl.units + pl.per_block - 1) / pl.per_block;
    pl.per_block = (pl.units + pl.splits - 1) / pl.splits;
    pl.partial_bytes = (size_t)pl.parts * pl.splits * SLOT_V4 * 16;
    pl.gsums_bytes = (size_t)pl.splits * p->Cout * 4;
    pl.xsums_bytes = (size_t)pl.splits * 9 * p->C * 4;
    pl.covered = true;
    return pl;
}

} // namespace

size_t hq_wgrad_band_bytes(const hq_problem *p)
{
    const WbandPlan pl = wband_plan(p);
    return pl.partial_bytes + pl.gsums_bytes + pl.xsums_bytes;
}

int hq_try_launch_wgrad_band(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY, const hq_qparams *gq,
                             float *dW, int32_t *dW_acc, void *ws, hipStream_t stream, const HqRideAlong *ride)
{
    const WbandPlan pl = wband_plan(p);
    if (!pl.covered) return HQ_E_BADSHAPE;
    WbandArgs a = {};
    a.X = X; a.G = dY; a.xq = xq; a.gq = gq;
    // every workgroup stores its sums to a slot of its own: nothing to zero, no atomics
    a.partial = static_cast<int32_t *>(ws);
    a.gsums = reinterpret_cast<int32_t *>(static_cast<char *>(ws) + pl.partial_bytes);
    a.xsums = reinterpret_cast<int32_t *>(static_cast<char *>(ws) + pl.partial_bytes + pl.gsums_bytes);
    a.frame = hq_frame(p->B, p->H, p->W);
    a.C = p->C; a.N = p->Cout;
    a.units = pl.units; a.per_block = pl.per_block; a.splits = pl.splits;
    a.cparts = p->C / 32; a.nparts = p->Cout / 64;
    a.lead = pl.lead; a.ring = pl.ring;
    a.gstep = hq_frame_distance(a.frame, GLOAD * WB_WAVES); a.xstep = hq_frame_distance(a.frame, L);
    static std::atomic<unsigned long long> allowed{0};
    if (!hq_allow_lds(hq_wgrad_band_kernel, 160 * 1024, allowed)) return HQ_E_HIP;
    hipLaunchKernelGGL(hq_wgrad_band_kernel, dim3((unsigned)(pl.parts * pl.splits)), dim3(WB_THREADS), pl.lds, stream, a);
    const size_t quads = (size_t)p->Cout / 4 * 9 * p->C;               // multiple of 64 (C % 64 == 0)
    HqRideAlong ra = ride ? *ride : HqRideAlong{nullptr, nullptr, 0, 0};
    ra.first = (int)(quads / 64);
    const dim3 fgrid((unsigned)(quads / 64) + (unsigned)ra.n);
    auto finalize = [&](auto kernel, int ty) {
        hipLaunchKernelGGL(kernel, fgrid, dim3(64 * ty), 0, stream, a.partial, a.gsums, a.xsums, xq, gq, (unsigned)a.frame.M, a.N, a.C, pl.splits, dW, dW_acc, ra);
    };
    if (pl.splits >= 48) finalize(wband_finalize_kernel<16>, 16);
    else if (pl.splits >= 12) finalize(wband_finalize_kernel<4>, 4);
    else finalize(wband_finalize_kernel<1>, 1);
    return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP;
}
