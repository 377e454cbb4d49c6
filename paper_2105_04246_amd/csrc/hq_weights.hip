// Weight side of a layer, run once per optimizer update: Q_W (hq_weight_quantize) and the re-laying of
// the codes for the input gradient with the zero-point sums (hq_weight_prepare).
//
// A network's update calls both for every layer, and most layers hold so few weights (10^4 .. 10^6) that
// a launch costs more than its memory traffic: what bounds these entry points is the number of launches
// and the longest serial chain in each.  Hence one launch for hq_weight_prepare (two beyond COL_ONE lines), one for
// hq_weight_quantize up to QW_ONE elements, two beyond.  All weights of ResNet-18 (21 layers, 11.7 M): 167 launches before, 51 now.
#include "hq_device.h"
#include "hq_internal.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

inline bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }
inline int launch_status() { return hipGetLastError() == hipSuccess ? HQ_OK : HQ_E_HIP; }

// ---------------------------------------------------------------------------------------
// Q_W
// ---------------------------------------------------------------------------------------
constexpr int QW_THREADS = 1024;
// One launch: every workgroup reads the whole tensor for its maximum (from L2 after the first) and quantizes
// its share.  A compute unit reads about 64 bytes a clock, so 160 K elements are 10 K clocks, about what a
// second launch costs behind the first.
constexpr size_t QW_ONE = 160 * 1024;
constexpr int QW_PARTS = 512;                        // workgroups of the maximum pass of larger tensors

__device__ inline unsigned abs_bits(float w) { return __float_as_uint(w) & 0x7fffffffu; }

// Maximum of |w| over elements first, first + step, ... (groups of four where `vec`), as non-negative float bits: a NaN is
// above every number there and reaches scale_of.
__device__ inline unsigned absmax_bits(const float *__restrict__ w, size_t n, size_t first, size_t step, bool vec)
{
    unsigned m = 0;
    if (vec) {
        const size_t quads = n / 4;
        const v4f *w4 = reinterpret_cast<const v4f *>(w);
        size_t i = first;
        for (; i + 3 * step < quads; i += 4 * step) {
            v4f v[4];
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] = w4[i + k * step];
#pragma unroll
            for (int k = 0; k < 4; k++)
                m = max(m, max(max(abs_bits(v[k][0]), abs_bits(v[k][1])), max(abs_bits(v[k][2]), abs_bits(v[k][3]))));
        }
        for (; i < quads; i += step) {
            const v4f v = w4[i];
            m = max(m, max(max(abs_bits(v[0]), abs_bits(v[1])), max(abs_bits(v[2]), abs_bits(v[3]))));
        }
        if (first < n - 4 * quads) m = max(m, abs_bits(w[4 * quads + first]));
    } else {
        for (size_t i = first; i < n; i += step) m = max(m, abs_bits(w[i]));
    }
    return m;
}

// Maximum over the workgroup, in every thread.
__device__ inline unsigned block_max(unsigned m, unsigned *red)
{
    m = (unsigned)hq_wave_reduce((int)m, HqMax());       // bits of non-negative floats order like signed integers
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    unsigned r = red[threadIdx.x & (QW_THREADS / 64 - 1)];
    return (unsigned)hq_wave_reduce((int)r, HqMax());
}

__device__ inline float scale_of(unsigned bits)
{
    const float amax = __uint_as_float(bits);
    return amax > 0.0f ? __fdiv_rn(amax, 127.0f) : 1.0f;
}

// code of w: rne(w / s) with the division rounded once.  w * (1 / s) differs from that quotient by less than 4e-5
// (|quotient| <= 127, two roundings of 2^-24 each), so its rounding is the quotient's unless it lies that
// close to a half; only then is the division carried out (about two values in 10^4).
__device__ inline int code_of(float w, float s, float inv)
{
    const float q = __fmul_rn(w, inv);
    float r = rintf(q);
    // (a reciprocal that is not finite or lost bits to underflow fails the second comparison)
    if (!(fabsf(__fsub_rn(q, r)) < 0.4999f) || !(inv < 1e37f && inv > 1e-37f)) r = rintf(__fdiv_rn(w, s));
    return (int)__builtin_amdgcn_fmed3f(r, -127.0f, 127.0f);
}

// Codes of elements [lo, hi), dealt to threads t = tid, tid + step, ... by groups of four where `vec` (lo % 4 == 0,
// 16-byte aligned source, 4-byte aligned destination).
__device__ inline void quantize_span(const float *__restrict__ w, int8_t *__restrict__ out, size_t lo, size_t hi,
                                     size_t tid, size_t step, bool vec, float s)
{
    const float inv = __fdiv_rn(1.0f, s);
    if (vec) {
        const size_t q1 = hi / 4;
        for (size_t i = lo / 4 + tid; i < q1; i += step) {
            const v4f v = reinterpret_cast<const v4f *>(w)[i];
            reinterpret_cast<unsigned *>(out)[i] =
                hq_pack4(code_of(v[0], s, inv), code_of(v[1], s, inv), code_of(v[2], s, inv), code_of(v[3], s, inv));
        }
        lo = max(lo, 4 * q1);
    }
    for (size_t i = lo + tid; i < hi; i += step) out[i] = (int8_t)code_of(w[i], s, inv);
}

__global__ __launch_bounds__(QW_THREADS) void weight_quantize_one_kernel(const float *__restrict__ w, size_t n, int vec,
                                                                         int8_t *__restrict__ out, hq_qparams *wq)
{
    __shared__ unsigned red[QW_THREADS / 64];
    const unsigned m = block_max(absmax_bits(w, n, threadIdx.x, QW_THREADS, vec), red);
    const float s = scale_of(m);
    if (blockIdx.x == 0 && threadIdx.x == 0) { wq->scale = s; wq->zero_point = 0; }
    const size_t share = ((n + gridDim.x - 1) / gridDim.x + 3) & ~(size_t)3;
    const size_t lo = min(n, share * blockIdx.x), hi = min(n, lo + share);
    quantize_span(w, out, lo, hi, threadIdx.x, QW_THREADS, vec, s);
}

// Larger tensors.  The maxima of the first launch's workgroups wait at the start of `out` (aligned to 4 bytes);
// the second launch's workgroups read them, quantize everything behind them, and the last one to finish -- all
// have read the maxima by then -- quantizes the elements whose codes belong there.  wq->zero_point counts the
// finished workgroups in the meantime (cleared by the first launch).
__global__ __launch_bounds__(QW_THREADS) void weight_absmax_kernel(const float *__restrict__ w, size_t n, int vec,
                                                                   unsigned *parts, hq_qparams *wq)
{
    __shared__ unsigned red[QW_THREADS / 64];
    const size_t first = (size_t)blockIdx.x * QW_THREADS + threadIdx.x;
    const unsigned m = block_max(absmax_bits(w, n, first, (size_t)gridDim.x * QW_THREADS, vec), red);
    if (threadIdx.x == 0) parts[blockIdx.x] = m;
    if (blockIdx.x == 0 && threadIdx.x == 0) wq->zero_point = 0;
}

__global__ __launch_bounds__(QW_THREADS) void weight_quantize_kernel(const float *__restrict__ w, size_t n, int vec,
                                                                     const unsigned *parts, int nparts, size_t skip,
                                                                     int8_t *out, hq_qparams *wq)
{
    __shared__ unsigned red[QW_THREADS / 64];
    __shared__ unsigned arrived;
    const unsigned m = block_max((int)threadIdx.x < nparts ? parts[threadIdx.x] : 0u, red);
    const float s = scale_of(m);
    quantize_span(w, out, skip, n, (size_t)blockIdx.x * QW_THREADS + threadIdx.x, (size_t)gridDim.x * QW_THREADS, vec, s);
    // (the maxima were used before this barrier, so their loads are complete)
    __syncthreads();
    if (threadIdx.x == 0) arrived = (unsigned)atomicAdd(&wq->zero_point, 1);
    __syncthreads();
    if (arrived != gridDim.x - 1) return;
    quantize_span(w, out, 0, skip, threadIdx.x, QW_THREADS, vec, s);
    if (threadIdx.x == 0) { wq->scale = s; wq->zero_point = 0; }
}

// ---------------------------------------------------------------------------------------
// Re-laying and sums
// ---------------------------------------------------------------------------------------
// Lines that one workgroup takes (as 16-byte loads / with 256 channels or more, where the rest of the launch takes longer / by
// words), and at least when they are split.  One / two launches: 512 channels, 4608 lines 8.7 / 8.9 us, 9216 20.7 / 13.4; 1024
// channels, 6400 lines 19.9 / 22.7; 64 channels, 36864 lines 23.5 / 9.3; 100 channels, 3136 lines 9.3 / 9.8, 4608 10.8 / 8.9.
constexpr long COL_ONE = 5120, COL_ONE_WIDE = 8192, COL_ONE_WORDS = 4096, COL_PART = 1024;

struct PrepArgs {
    const int8_t *W;
    int8_t *Wd;
    int32_t *rowsum, *colsum, *colsum2;
    int rows, taps, C;              // W[rows][taps][C]
    int row_blocks, col_blocks;     // workgroups of the first two roles; the rest re-lay tiles
    int col_parts;                  // workgroups that share the lines of one column block, which meet by atomics if more than one
    int32_t *clear;                 // C words to clear for such a launch that follows
    int fold;                       // lines of fewer than 16 channels that are read as one
    int lines, share;               // (folded) lines; of a workgroup's part
    int tiles_n, tiles_c;           // 64 x 64 tiles per tap
    int in_align, out_align;        // 16, 4 or 1: what divides the address of W / of every line of Wd
};

// 16 codes at p, of which `n` exist; `align` (16, 4 or 1) divides both the address and n.
__device__ inline v4i load_codes16(const int8_t *p, int n, int align)
{
    v4i v = {0, 0, 0, 0};
    if (n >= 16 && align >= 16) {
        v = *reinterpret_cast<const v4i *>(p);
    } else if (align >= 4) {
#pragma unroll
        for (int d = 0; d < 4; d++)
            if (4 * d < n) v[d] = *reinterpret_cast<const int *>(p + 4 * d);
    } else {
#pragma unroll
        for (int e = 0; e < 16; e++)
            if (e < n) v[e >> 2] |= (int)((unsigned)(unsigned char)p[e] << (8 * (e & 3)));
    }
    return v;
}

// Three roles, by workgroup index, all reading W (from L2 after the first touch):
//   row sums      one wavefront per row of taps * C codes
//   column sums   a workgroup owns 16 channels and runs over all rows * taps lines, so that nothing has to be
//                 cleared beforehand and no atomics meet; four lines of a thread are in flight, since the lines lie in
//                 as many cache lines and the chain of loads is the longest of the launch
//   re-laying     64 x 64 tiles of one tap, transposed through LDS: W[n][tap][c] -> Wd[c][tap][n]
// Beyond COL_ONE lines the chain is longer than another launch: that one splits the lines over workgroups.
__global__ __launch_bounds__(HQ_THREADS) void weight_prepare_kernel(const PrepArgs a)
{
    __shared__ __attribute__((aligned(16))) int8_t tile[64 * 68];
    __shared__ int sums[HQ_THREADS / 64][16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const size_t len = (size_t)a.taps * a.C;
    int block = blockIdx.x;
    if (a.clear)
        for (int c = block * HQ_THREADS + tid; c < a.C; c += gridDim.x * HQ_THREADS) a.clear[c] = 0;
    if (block < a.row_blocks) {
        const int row = block * (HQ_THREADS / 64) + wave;
        if (row >= a.rows) return;
        const int8_t *w = a.W + (size_t)row * len;
        const int align = min(a.in_align, len % 16 == 0 ? 16 : len % 4 == 0 ? 4 : 1);
        int s = 0;
        for (size_t i = 16 * lane; i < len; i += 16 * 64) {
            const v4i v = load_codes16(w + i, (int)min((size_t)16, len - i), align);
#pragma unroll
            for (int d = 0; d < 4; d++) s = __builtin_amdgcn_sdot4(v[d], 0x01010101, s, false);
        }
        s = hq_wave_reduce(s, HqAdd());
        if (lane == 0) a.rowsum[row] = s;
        return;
    }
    block -= a.row_blocks;
    const int align = min(a.in_align, a.C % 16 == 0 ? 16 : a.C % 4 == 0 ? 4 : 1);
    if (block < a.col_blocks * a.col_parts) {
        const int width = a.C * a.fold, walign = min(a.in_align, width % 16 == 0 ? 16 : width % 4 == 0 ? 4 : 1);
        const int column = a.col_parts == 1 ? block : block / a.col_parts, part = block - column * a.col_parts;
        const int c0 = 16 * column, nc = min(16, width - c0);
        const int lo = a.share * part, lines = min(a.lines, lo + a.share);
        int s[16] = {};
        auto run = [&](auto al) {
            auto load = [&](int l) { return load_codes16(a.W + (size_t)l * width + c0, nc, decltype(al)::value); };
            auto add = [&](const v4i &v) {
#pragma unroll
                for (int e = 0; e < 16; e++) s[e] = __builtin_amdgcn_sdot4(v[e >> 2], 1 << (8 * (e & 3)), s[e], false);
            };
            int l = lo + tid;
            if (decltype(al)::value > 1)                 // (off 4 bytes: 16 loads a line are in flight anyway)
                for (int full = (lines - lo) / (4 * HQ_THREADS); full > 0; full--, l += 4 * HQ_THREADS) {
                    v4i v[4];
#pragma unroll
                    for (int k = 0; k < 4; k++) v[k] = load(l + k * HQ_THREADS);
#pragma unroll
                    for (int k = 0; k < 4; k++) add(v[k]);
                }
#pragma unroll 1
            for (; l < lines; l += HQ_THREADS) add(load(l));
        };
        if (walign == 16) run(std::integral_constant<int, 16>());
        else if (walign == 4) run(std::integral_constant<int, 4>());
        else run(std::integral_constant<int, 1>());
#pragma unroll
        for (int e = 0; e < 16; e++) {
            const int t = hq_wave_reduce(s[e], HqAdd());
            if (lane == 0) sums[wave][e] = t;
        }
        __syncthreads();
        if (tid < (a.fold > 1 ? a.C : nc)) {
            int t = 0;
            for (int j = tid; j < (a.fold > 1 ? nc : tid + 1); j += a.C) t += sums[0][j] + sums[1][j] + sums[2][j] + sums[3][j];
            if (a.col_parts > 1) {
                atomicAdd(a.colsum + c0 + tid, t);
            } else {
                if (a.colsum) a.colsum[c0 + tid] = t;
                if (a.colsum2) a.colsum2[c0 + tid] = t;
            }
        }
        return;
    }
    block -= a.col_blocks * a.col_parts;
    if (!a.Wd) return;
    const int tc = block % a.tiles_c, tn = block / a.tiles_c % a.tiles_n, tap = block / (a.tiles_c * a.tiles_n);
    const int c0 = 64 * tc, n0 = 64 * tn, r = tid >> 2, q = 16 * (tid & 3);
    {
        v4i v = {0, 0, 0, 0};
        if (n0 + r < a.rows && c0 + q < a.C)
            v = load_codes16(a.W + ((size_t)(n0 + r) * a.taps + tap) * a.C + c0 + q, min(16, a.C - c0 - q), align);
#pragma unroll
        for (int d = 0; d < 4; d++) *reinterpret_cast<int *>(tile + r * 68 + q + 4 * d) = v[d];
    }
    __syncthreads();
    if (c0 + r >= a.C || n0 + q >= a.rows) return;
    v4i v;
#pragma unroll
    for (int d = 0; d < 4; d++) {
        const int8_t *t = tile + (q + 4 * d) * 68 + r;
        v[d] = (int)hq_pack4(t[0], t[68], t[136], t[204]);
    }
    int8_t *dst = a.Wd + ((size_t)(c0 + r) * a.taps + tap) * a.rows + n0 + q;
    const int nn = min(16, a.rows - n0 - q);
    if (nn == 16 && a.out_align == 16) {
        *reinterpret_cast<v4i *>(dst) = v;
    } else if (a.out_align >= 4) {                       // rows % 4 == 0
#pragma unroll
        for (int d = 0; d < 4; d++)
            if (4 * d < nn) *reinterpret_cast<int *>(dst + 4 * d) = v[d];
    } else {
#pragma unroll
        for (int e = 0; e < 16; e++)
            if (e < nn) dst[e] = (int8_t)(v[e >> 2] >> (8 * (e & 3)));
    }
}

inline int align_of(const void *p) { return misaligned(p, 16) ? misaligned(p, 4) ? 1 : 4 : 16; }

} // namespace

int hq_launch_weight_prepare(const hq_problem *p, const int8_t *W, int8_t *Wd, int32_t *wsum, int32_t *wdsum, hipStream_t s)
{
    PrepArgs a = {};
    a.W = W; a.taps = p->R * p->S; a.C = p->C; a.in_align = align_of(W);
    if (p->kind == HQ_DEPTHWISE) {
        a.rows = 1; a.colsum = wsum; a.colsum2 = wdsum;
        a.col_blocks = wsum || wdsum ? (p->C + 15) / 16 : 0;
    } else {
        a.rows = p->Cout; a.Wd = Wd; a.rowsum = wsum; a.colsum = wdsum;
        a.row_blocks = wsum ? (p->Cout + 3) / 4 : 0;
        a.col_blocks = wdsum ? (p->C + 15) / 16 : 0;
        a.out_align = std::min(align_of(Wd), p->Cout % 16 == 0 ? 16 : 4);        // Cout % 4 == 0
    }
    a.tiles_n = (a.rows + 63) / 64; a.tiles_c = (a.C + 63) / 64;
    a.col_parts = 1;
    a.fold = a.C == 3 ? 4 : (long)a.rows * a.taps < 1024 ? 1 : a.C == 4 ? 4 : a.C == 8 ? 2 : 1;
    if ((long)a.rows * a.taps % a.fold != 0) a.fold = 1;
    const long lines = (long)a.rows * a.taps / a.fold;
    const int col_blocks = a.col_blocks;
    a.lines = a.share = (int)lines;
    const bool apart = a.colsum && !a.colsum2 &&
                       lines > (a.in_align != 16 || a.C * a.fold % 16 != 0 ? COL_ONE_WORDS : a.C >= 256 ? COL_ONE_WIDE : COL_ONE);
    if (apart) { a.col_blocks = 0; a.clear = a.colsum; }
    unsigned blocks = (unsigned)(a.row_blocks + a.col_blocks) + (a.Wd ? (unsigned)a.tiles_n * a.tiles_c * a.taps : 0u);
    if (apart && blocks == 0) blocks = (unsigned)((a.C + HQ_THREADS - 1) / HQ_THREADS);
    if (blocks == 0) return HQ_OK;
    hipLaunchKernelGGL(weight_prepare_kernel, dim3(blocks), dim3(HQ_THREADS), 0, s, a);
    if (apart) {
        a.clear = nullptr; a.Wd = nullptr; a.row_blocks = 0;
        a.col_blocks = col_blocks;
        a.col_parts = (int)std::min((lines + COL_PART - 1) / COL_PART, std::max(1L, 1024L / col_blocks));
        a.share = (int)((lines + a.col_parts - 1) / a.col_parts);
        hipLaunchKernelGGL(weight_prepare_kernel, dim3((unsigned)(a.col_blocks * a.col_parts)), dim3(HQ_THREADS), 0, s, a);
    }
    return launch_status();
}

int hq_launch_weight_quantize(const float *Wf, size_t n, int8_t *Wq, hq_qparams *wq, hipStream_t s)
{
    const int vec = !misaligned(Wf, 16) && !misaligned(Wq, 4);
    if (n <= QW_ONE) {
        // a share of at least 4 K elements: more workgroups would only read the tensor more often
        const unsigned blocks = (unsigned)((n + 4095) / 4096);
        hipLaunchKernelGGL(weight_quantize_one_kernel, dim3(blocks), dim3(QW_THREADS), 0, s, Wf, n, vec, Wq, wq);
        return launch_status();
    }
    // at least 16 elements per thread in the first launch and 4 in the second
    const size_t most = (n + 16 * QW_THREADS - 1) / (16 * QW_THREADS);
    const int nparts = (int)(most < QW_PARTS ? most : QW_PARTS);
    unsigned *parts = reinterpret_cast<unsigned *>((reinterpret_cast<uintptr_t>(Wq) + 3) & ~(uintptr_t)3);
    const size_t skip = 4 * (size_t)nparts + 4;          // elements whose codes share bytes with `parts`; multiple of 4
    const size_t quads = (n + 4 * QW_THREADS - 1) / (4 * QW_THREADS);
    hipLaunchKernelGGL(weight_absmax_kernel, dim3((unsigned)nparts), dim3(QW_THREADS), 0, s, Wf, n, vec, parts, wq);
    hipLaunchKernelGGL(weight_quantize_kernel, dim3((unsigned)(quads < 1024 ? quads : 1024)), dim3(QW_THREADS), 0, s,
                       Wf, n, vec, parts, nparts, skip, Wq, wq);
    return launch_status();
}
