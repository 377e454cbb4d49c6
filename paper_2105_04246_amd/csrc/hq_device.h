// Device-side helpers shared by the HIP kernels of the hq library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <limits.h>
#include <stddef.h>
#include "../../include/hq.h"

typedef int v4i  __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

#define HQ_THREADS 256                     // 4 wavefronts of 64 lanes; kernels with other sizes name their own

// x / d by multiplication, for d >= 1 and x * d < 2^32: magic = (unsigned)ceil(2^32 / d), which for
// d == 1 wraps to 0 and is then taken as "no division".  The host computes the constant.
__host__ __device__ inline unsigned hq_magic32(unsigned d) { return (unsigned)(((1ull << 32) + d - 1) / d); }
__device__ inline unsigned hq_magic_div(unsigned x, unsigned magic) { return magic ? __umulhi(x, magic) : x; }

// x / d by multiplication for every x < 2^31 and 1 <= d < 2^31 (Granlund and Montgomery): m = ceil(2^(31 + l) / d) with
// 2^(l - 1) < d <= 2^l, s = l - 1.  d = 1 is m = 0, "no division"; hq_quot2 is for divisors that are at least 2.
struct HqDivisor { unsigned m, s; };
inline HqDivisor hq_divisor(unsigned d)
{
    unsigned l = 1;
    while ((1ull << l) < d) l++;
    return d < 2 ? HqDivisor{0, 0} : HqDivisor{(unsigned)(((1ull << (31 + l)) + d - 1) / d), l - 1};
}
__device__ inline unsigned hq_quot2(unsigned x, HqDivisor d) { return __umulhi(x, d.m) >> d.s; }
__device__ inline unsigned hq_quot(unsigned x, HqDivisor d) { return d.m ? hq_quot2(x, d) : x; }

// ---------------------------------------------------------------------------------------
// Framed images: positions of rows of W + 1 and of images of H + 1 rows.  The extra column is the right border of its row and the left
// border of the next one, the extra row the lower border of its image and the upper border of the next one, so that every tap of a
// 3x3 filter is one distance in positions for all pixels.  A lane that walks such positions keeps pixel, row and column; the pixel counts as if
// the frame were not there, so that it is right where row and column lie inside the image.
// ---------------------------------------------------------------------------------------
struct HqFrame {
    int M, H, W;                   // pixels of the batch; image
    int PW;                        // positions of a row: W + 1
    HqDivisor image, row;          // (H + 1) * PW and PW
};
struct HqFramePlace { int p, y, x; };                        // pixel, row, column; of a distance: that many positions as such

inline HqFrame hq_frame(int B, int H, int W)
{
    return HqFrame{B * H * W, H, W, W + 1, hq_divisor((unsigned)(H + 1) * (unsigned)(W + 1)), hq_divisor((unsigned)W + 1)};
}
inline HqFramePlace hq_frame_distance(const HqFrame &f, int k)
{
    const int image = (f.H + 1) * f.PW, y = k % image / f.PW, x = k % image % f.PW;
    return HqFramePlace{(k / image * f.H + y) * f.W + x, y, x};
}
__device__ inline HqFramePlace hq_frame_place(const HqFrame &f, unsigned k)                 // of position k
{
    const unsigned image = (unsigned)(f.H + 1) * (unsigned)f.PW, b = hq_quot2(k, f.image), rem = k - b * image;
    HqFramePlace t;
    t.y = (int)hq_quot2(rem, f.row);
    t.x = (int)(rem - (unsigned)t.y * (unsigned)f.PW);
    t.p = ((int)b * f.H + t.y) * f.W + t.x;
    return t;
}
__device__ inline void hq_frame_back(const HqFrame &f, HqFramePlace &t)                     // PW + 1 positions: what the first tap meets
{
    t.p -= f.W + 1; t.y--; t.x--;
    if (t.x < 0) { t.x += f.PW; t.y--; t.p++; }
    if (t.y < 0) { t.y += f.H + 1; t.p += f.W; }
}
__device__ inline void hq_frame_advance(const HqFrame &f, const HqFramePlace &d, HqFramePlace &t)
{
    t.x += d.x; t.y += d.y; t.p += d.p;
    const bool cx = t.x >= f.PW;
    t.x -= cx ? f.PW : 0; t.y += cx; t.p -= cx;
    const bool cy = t.y > f.H;
    t.y -= cy ? f.H + 1 : 0; t.p -= cy ? f.W : 0;
}
__device__ inline bool hq_frame_inside(const HqFrame &f, const HqFramePlace &t)
{
    return ((unsigned)t.p < (unsigned)f.M) & (t.y < f.H) & (t.x < f.W);
}
// base + offset where `in`, otherwise `fill`: selected, not branched around.
__device__ inline const int8_t *hq_source(bool in, const int8_t *base, unsigned long long offset, const void *fill)
{
    unsigned long long p = (unsigned long long)(uintptr_t)base + offset;
    asm("" : "+v"(p));
    return reinterpret_cast<const int8_t *>((uintptr_t)(in ? p : (unsigned long long)(uintptr_t)fill));
}

// ---------------------------------------------------------------------------------------
// 3-byte pixels (RGB inputs): a lane's 4-byte word of the reduction starts at any byte address and
// can hold bytes of two taps.  Words are loaded unaligned and the unwanted bytes replaced under a
// byte mask.
// ---------------------------------------------------------------------------------------

// Bytes e of a 32-bit word with lo <= e < hi (little endian), as a mask of whole bytes.
__device__ inline unsigned hq_bytemask(int lo, int hi)
{
    lo = max(lo, 0); hi = min(hi, 4);
    if (hi <= lo) return 0u;
    const unsigned upto_hi = hi == 4 ? 0xffffffffu : (1u << (8 * hi)) - 1u;
    return upto_hi & ~((1u << (8 * lo)) - 1u);
}

// 16 consecutive bytes starting at p (any alignment) of a tensor that occupies [begin, end): aligned loads
// of the five 32-bit words that hold them (one 16-byte and one 4-byte load where all five lie inside the
// tensor, guarded single words at its first and last bytes), then a byte-wise funnel shift.  Unaligned
// word loads are served far more slowly.  Bytes outside the tensor arrive as anything: the caller masks them
// (they belong to taps outside the image).  An aligned word that holds the tensor's last byte is read
// whole, i.e. up to the next multiple of 4 of `end`.
__device__ inline v4i hq_load16_any(const int8_t *p, const int8_t *begin, const int8_t *end)
{
    // (pointer arithmetic only: a pointer rebuilt from an integer would lose its address space and every load
    // below would become a flat load, which the compiler can only wait for all at once)
    const unsigned sh = (unsigned)(reinterpret_cast<uintptr_t>(p) & 3);
    const int8_t *a = p - sh;
    const int8_t *end4 = end + ((4u - (unsigned)(reinterpret_cast<uintptr_t>(end) & 3)) & 3u);
    int w[5];
    // one uniform branch: wavefronts that touch neither end of the tensor (all but a few) take the two wide
    // loads; the others load word by word from addresses moved inside the tensor where they would fall outside
    const bool inner = a >= begin && a + 20 <= end4;
    if (__builtin_amdgcn_ballot_w64(!inner) == 0) {
        v4i x;
        __builtin_memcpy(&x, __builtin_assume_aligned(a, 4), 16);
        w[0] = x[0]; w[1] = x[1]; w[2] = x[2]; w[3] = x[3];
        w[4] = *reinterpret_cast<const int *>(a + 16);
    } else {
        const int8_t *safe = begin + ((4u - (unsigned)(reinterpret_cast<uintptr_t>(begin) & 3)) & 3u);
#pragma unroll
        for (int d = 0; d < 5; d++) {
            const int8_t *q = a + 4 * d;
            const bool in = q >= begin && q < end4;
            const int x = *reinterpret_cast<const int *>(in ? q : safe);
            w[d] = in ? x : 0;
        }
    }
    v4i v;
#pragma unroll
    for (int d = 0; d < 4; d++) v[d] = (int)__builtin_amdgcn_alignbyte((unsigned)w[d + 1], (unsigned)w[d], sh);
    return v;
}

// ---------------------------------------------------------------------------------------
// Quantizer arithmetic.  Each fp32 operation rounds once (no contraction), so that the
// result is a function of the operands alone.
// ---------------------------------------------------------------------------------------

// Quantizer of a range (qmin, qmax): asymmetric grids are widened to contain real zero.
__device__ inline hq_qparams hq_qparams_from_range(float qmin, float qmax, int symmetric, int qlo, int qhi)
{
    hq_qparams q;
    if (symmetric) {
        float amax = fmaxf(fabsf(qmin), fabsf(qmax));
        q.scale = amax > 0.0f ? __fdiv_rn(amax, (float)qhi) : 1.0f;
        q.zero_point = 0;
        return q;
    }
    float lo = fminf(qmin, 0.0f), hi = fmaxf(qmax, 0.0f);
    float width = __fsub_rn(hi, lo);
    float s = width > 0.0f ? __fdiv_rn(width, (float)(qhi - qlo)) : 1.0f;
    float z = rintf(__fsub_rn((float)qlo, __fdiv_rn(lo, s)));
    z = fminf(fmaxf(z, (float)qlo), (float)qhi);
    q.scale = s;
    q.zero_point = (int)z;
    return q;
}

// Order-preserving map between fp32 values and signed 32-bit keys (its own inverse on the bit
// pattern): integer min / max and their atomics then order real values.  Used by the statistics
// of real-valued tensors; -0 is made +0 first so that equal values have equal keys.
__device__ inline int hq_float_key(float x)
{
    const int b = __float_as_int(x + 0.0f);
    return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ inline float hq_key_float(int k) { return __int_as_float(k ^ ((k >> 31) & 0x7fffffff)); }

// ---------------------------------------------------------------------------------------
// eq. (2)-(3): q <- (1 - eta) * g + eta * q, each product and the sum rounded once.
// ---------------------------------------------------------------------------------------
__device__ inline void hq_ema_update(hq_range *r, float gmin, float gmax)
{
    if (!r->initialized) {
        r->qmin = gmin; r->qmax = gmax; r->initialized = 1;
    } else {
        const float w = __fsub_rn(1.0f, r->eta);
        r->qmin = __fadd_rn(__fmul_rn(w, gmin), __fmul_rn(r->eta, r->qmin));
        r->qmax = __fadd_rn(__fmul_rn(w, gmax), __fmul_rn(r->eta, r->qmax));
    }
    r->qp = hq_qparams_from_range(r->qmin, r->qmax, r->symmetric, r->qlo, r->qhi);
}

// ---------------------------------------------------------------------------------------
// Saturation-driven update (Sec. 4 names the saturation ratio as a statistic; the rule is this
// library's, stated with hq_range_update_saturation).
// ---------------------------------------------------------------------------------------

// ln x for a positive normal x by a fixed sequence of fp32 operations, each rounded once:
// x = m * 2^e, m in [sqrt(1/2), sqrt(2)), s = (m - 1) / (m + 1), ln x = e ln 2 + 2 s (1 + s^2/3 + s^4/5 + s^6/7).
__device__ inline float hq_ln_fixed(float x)
{
    const unsigned bits = __float_as_uint(x);
    int e = (int)((bits >> 23) & 0xffu) - 127;
    float m = __uint_as_float((bits & 0x007fffffu) | 0x3f800000u);
    if (m > 1.41421354f) { m = __fmul_rn(m, 0.5f); e += 1; }
    const float sq = __fdiv_rn(__fsub_rn(m, 1.0f), __fadd_rn(m, 1.0f));
    const float s2 = __fmul_rn(sq, sq);
    float p = __fmul_rn(s2, 1.0f / 7.0f);
    p = __fadd_rn(p, 0.2f);
    p = __fmul_rn(p, s2);
    p = __fadd_rn(p, 1.0f / 3.0f);
    p = __fmul_rn(p, s2);
    p = __fadd_rn(p, 1.0f);
    const float lm = __fmul_rn(__fmul_rn(2.0f, sq), p);
    return __fadd_rn(__fmul_rn((float)e, 0.693147182f), lm);
}

__device__ inline void hq_saturation_update(hq_range *r, hq_saturation *sat, unsigned long long clipped,
                                            unsigned long long count, float gmin, float gmax)
{
    if (!r->initialized) {
        r->qmin = gmin; r->qmax = gmax; r->initialized = 1;
        sat->streak = 0;
    } else {
        const float alpha = __fdiv_rn((float)clipped, (float)count);
        if (alpha >= sat->alpha_min && alpha <= sat->alpha_max) {
            sat->streak = 0;
        } else {
            sat->streak += 1;
            if (sat->streak > sat->tau) {
                const float fl = __fdiv_rn(0.5f, (float)count);
                const float ah = fminf(fmaxf(alpha, fl), 0.5f);
                const float rho = __fdiv_rn(hq_ln_fixed(sat->alpha_target), hq_ln_fixed(ah));
                r->qmin = __fmul_rn(rho, r->qmin);
                r->qmax = __fmul_rn(rho, r->qmax);
                sat->streak = 0;
            }
        }
    }
    r->qp = hq_qparams_from_range(r->qmin, r->qmax, r->symmetric, r->qlo, r->qhi);
}

// Everything the epilogue needs to turn a zero-point-corrected accumulator into a code.
struct HqRequant {
    float mult;        // (s_a * s_b) / s_out
    float flo, fhi;    // grid bounds relative to the zero point, as floats
    int   z;
};

__device__ inline HqRequant hq_make_requant(float acc_scale, hq_qparams out, int qlo, int qhi)
{
    HqRequant r;
    r.mult = __fdiv_rn(acc_scale, out.scale);
    r.flo = (float)(qlo - out.zero_point);
    r.fhi = (float)(qhi - out.zero_point);
    r.z = out.zero_point;
    return r;
}

// One fp32 multiply, round half to even, clamp in float, then the zero point.
__device__ inline int hq_requant(int c, const HqRequant &q, unsigned &nlo, unsigned &nhi)
{
    float r = rintf(__fmul_rn((float)c, q.mult));
    nlo += (r < q.flo) ? 1u : 0u;
    nhi += (r > q.fhi) ? 1u : 0u;
    r = fminf(fmaxf(r, q.flo), q.fhi);
    return (int)r + q.z;
}

// ---------------------------------------------------------------------------------------
// Fused epilogue of the MFMA kernels: a lane's zero-point-corrected accumulators -> codes,
// with min / max and exact clip counts folded in (Sec. 4, steps 1 and 2).
// Per value: convert, multiply, round (the requantization of the static quantizer), add the
// zero point, pack.  Clipped values are counted per lane from the rounded floats, and only in
// groups whose extreme accumulators may clip: requantization is monotone in the accumulator, so
// the extremes decide for the whole group, and two bounds on the accumulator, worked out once, decide for them.
// ---------------------------------------------------------------------------------------
struct HqEpilogue {
    float mult;          // (s_a * s_b) / s_out
    float flo, fhi;      // grid bounds relative to the zero point
    float zoff;          // zero point + 128: codes are formed as unsigned bytes, see below
    bool full_grid;      // grid is -128..127: the saturating pack is the whole clamp
    int c_lo, c_hi;      // accumulators in [c_lo, c_hi] surely do not clip under round to nearest
};

__device__ inline HqEpilogue hq_make_epilogue(float acc_scale, const hq_range *r)
{
    HqEpilogue e;
    e.mult = __fdiv_rn(acc_scale, r->qp.scale);
    e.flo = (float)(r->qlo - r->qp.zero_point);
    e.fhi = (float)(r->qhi - r->qp.zero_point);
    e.zoff = (float)(r->qp.zero_point + 128);
    e.full_grid = r->qlo == -128 && r->qhi == 127;
    // a value clips iff |c| * mult rounds past the bound, i.e. c > (fhi + 1/2) / mult up to the few roundings (2^-24
    // each) of that quotient, of float(c) and of the product: 1e-6 of it and one unit cover them
    const float hi = __fmul_rn(__fdiv_rn(e.fhi + 0.5f, e.mult), 0.999999f) - 1.0f;
    const float lo = __fmul_rn(__fdiv_rn(e.flo - 0.5f, e.mult), 0.999999f) + 1.0f;
    e.c_hi = hi < 2147483648.0f ? (int)hi : INT_MAX;
    e.c_lo = lo > -2147483648.0f ? (int)lo : INT_MIN;
    return e;
}

__device__ inline float hq_round_scaled(int c, float mult) { return rintf(__fmul_rn((float)c, mult)); }

// 16 bytes per lane from global memory straight into LDS (global_load_lds_dwordx4): lane l of the wavefront
// lands at wave_base + 16 * l.  Written as an asm statement because the compiler, once it has issued such a load
// itself, waits for every outstanding LDS read before using any of them (it stops counting them), which
// defeats fragment double buffering in the loops that follow.  The caller waits for the load with an explicit
// "s_waitcnt vmcnt(..)" before a barrier; the compiler's own counts stay safe because loads retire in order.
__device__ inline void hq_lds_load16(const void *src, unsigned dst)                        // (dst: LDS address, uniform)
{
    unsigned keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "v"(src), "s"(dst) : "memory");
}
// ... from a uniform base plus a lane's offset.
__device__ inline void hq_lds_load16(const int8_t *base, unsigned off, unsigned dst)
{
    unsigned keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "v"(off), "s"(base), "s"(dst) : "memory");
}
// ... to a pointer that is the same in all lanes.
__device__ inline unsigned hq_lds_address(void *wave_base)
{
    return __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void *)wave_base);
}
__device__ inline void hq_global_to_lds16(const void *src, void *wave_base) { hq_lds_load16(src, hq_lds_address(wave_base)); }
__device__ inline void hq_global_to_lds16(const int8_t *base, unsigned off, void *wave_base) { hq_lds_load16(base, off, hq_lds_address(wave_base)); }

// 16-byte rows of one repeated byte value, indexed by that value: what lanes of such a load read that have no source (outside the
// image: the zero-point code; past the reduction or the weights: 0), so that every lane has an address and a wavefront's count of
// outstanding loads does not depend on its data.
struct HqFillRows {
    unsigned w[256][4];
    constexpr HqFillRows() : w()
    {
        for (int v = 0; v < 256; v++)
            for (int k = 0; k < 4; k++) w[v][k] = (unsigned)v * 0x01010101u;
    }
};
static __device__ const HqFillRows hq_fill_rows = HqFillRows();

// Row of a 32-row operand block that LDS row i holds, so that a lane of the 32 x 32 MFMA's result has 16 consecutive channels.
__device__ inline int hq_sigma32(int i) { return ((i >> 2) & 1) * 16 + (i >> 3) * 4 + (i & 3); }

typedef __attribute__((__vector_size__(2 * sizeof(int)))) int tr_v2i;
#define LDS_PTR(T) __attribute__((address_space(3))) T *

// Fragment of one 32-channel x 32-pixel operand block for the 32x32x32 MFMA, read transposed (ds_read_b64_tr_b8) from LDS
// rows of one pixel's channels: lane l gets channel (l % 32) and the 16 pixels of half (l / 32).  `tile` points at row 0
// of the k-step and column 0 of the 32-channel block; P is the pitch of a row.
template <int P> __device__ inline v4i hq_read_frag_tr(const int8_t *tile, int lane)
{
    const int j = lane & 15, grp = (lane >> 4) & 1, half = lane >> 5;
    const int8_t *p = tile + (half * 16 + (j >> 1)) * P + 16 * grp + 8 * (j & 1);
    tr_v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(p));
    tr_v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((LDS_PTR(tr_v2i))(p + 8 * P));
    v4i f = {lo[0], lo[1], hi[0], hi[1]};
    return f;
}

// Three-operand integer minimum / maximum (v_min3_i32 / v_max3_i32).  The empty statement keeps the compiler from
// balancing a chain of minima into a tree of two-operand ones (12 instructions for 16 values instead of 8).  The
// instruction itself is left to the compiler: it knows how long the result of a dot product or an MFMA has to
// settle before it may be read, which it does not see inside an asm statement.
__device__ inline int hq_min3(int a, int b, int c)
{
    int r = min(min(a, b), c);
    asm("" : "+v"(r));
    return r;
}
__device__ inline int hq_max3(int a, int b, int c)
{
    int r = max(max(a, b), c);
    asm("" : "+v"(r));
    return r;
}

// N = 4, 8 or 16 accumulators -> N / 4 words of signed codes.  v_cvt_pk_u8_f32 saturates to
// 0..255, which after the flip of the top bits is the clamp to -128..127.
template <int N, bool FULL_GRID>
__device__ inline void hq_requant_group(const int *c, const HqEpilogue &ep, int &mn, int &mx,
                                        unsigned &w_lo, unsigned &w_hi, int *words)
{
    int gmn = c[0], gmx = c[0];
#pragma unroll
    for (int e = 1; e + 1 < N; e += 2) { gmn = hq_min3(gmn, c[e], c[e + 1]); gmx = hq_max3(gmx, c[e], c[e + 1]); }
    gmn = min(gmn, c[N - 1]); gmx = max(gmx, c[N - 1]);
    mn = min(mn, gmn); mx = max(mx, gmx);
    float f[N];
#pragma unroll
    for (int e = 0; e < N; e++) f[e] = hq_round_scaled(c[e], ep.mult);
    if (__any(gmx > ep.c_hi || gmn < ep.c_lo)) {
        // rounded values and bounds are whole numbers: clamping the difference to [0, 1] is the
        // indicator of a clipped value (a subtraction with the clamp modifier, no compare)
        float nh = 0.0f, nl = 0.0f;
#pragma unroll
        for (int e = 0; e < N; e++) {
            nh += __builtin_amdgcn_fmed3f(f[e] - ep.fhi, 0.0f, 1.0f);
            nl += __builtin_amdgcn_fmed3f(ep.flo - f[e], 0.0f, 1.0f);
        }
        w_hi += (unsigned)nh; w_lo += (unsigned)nl;
    }
#pragma unroll
    for (int g = 0; g < N / 4; g++) {
        unsigned w = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            float v = f[4 * g + e];
            if (!FULL_GRID) v = __builtin_amdgcn_fmed3f(v, ep.flo, ep.fhi);
            w = __builtin_amdgcn_cvt_pk_u8_f32(v + ep.zoff, e, w);
        }
        words[g] = (int)(w ^ 0x80808080u);
    }
}

// ---------------------------------------------------------------------------------------
// Stochastic rounding (the paper quantizes gradients with it, Sec. 5 experimental setup, after
// Gupta et al. 2015): the scaled accumulator x rounds up with probability x - floor(x).  Each
// output element draws its 24 random bits from a counter-based generator keyed on the element's
// linear index in its tensor and a 64-bit seed, so the result does not depend on how the launch
// is tiled.  The generator: the low index word through the finalizer of MurmurHash3, with the
// first key word added and the high index word (times an odd constant) plus the second key
// word folded in between its two rounds, closed by a multiply with the golden-ratio constant
// and a xor-shift.
// ---------------------------------------------------------------------------------------
struct HqSr { unsigned k0, k1; };          // low and high half of the seed

__device__ inline unsigned hq_sr_first(unsigned idx_lo, unsigned k0) { return (idx_lo ^ (idx_lo >> 16)) * 0x85ebca6bu + k0; }

__device__ inline unsigned hq_sr_rest(unsigned h, unsigned hi_term)      // hi_term = idx_hi * 0x85ebca77 + k1
{
    h ^= hi_term;
    h ^= h >> 13; h *= 0xc2b2ae35u; h ^= h >> 16;
    h *= 0x9e3779b1u; h ^= h >> 15;
    return h;
}

__device__ inline unsigned hq_sr_bits(unsigned idx_lo, unsigned hi_term, unsigned k0)
{
    return hq_sr_rest(hq_sr_first(idx_lo, k0), hi_term);
}

// hq_sr_first of the indices idx_lo .. idx_lo + N - 1, idx_lo a multiple of N = 4, 8 or 16.  The generator's integer
// multiplications run at a quarter of the rate and are what stochastic rounding costs; here one serves N elements.  All
// N share the bits above the lowest log2 N, so element e multiplies b ^ e, b that of element 0, and flipping bit k of b
// adds or takes 2^k: the products differ by sums of +-(constant << k).  (A step of 3x3 128 -> 128 on 28 x 28 at batch 128 with a
// stochastically rounded input gradient: 105.9 -> 103.8 us.)
template <int N> __device__ inline void hq_sr_first_n(unsigned idx_lo, unsigned k0, unsigned *h)
{
    static_assert(N == 4 || N == 8 || N == 16, "aligned groups");
    const unsigned b = idx_lo ^ (idx_lo >> 16);
    h[0] = b * 0x85ebca6bu + k0;
#pragma unroll
    for (int k = 1; k < N; k *= 2) {
        const unsigned up = 0x85ebca6bu * (unsigned)k, d = (b & (unsigned)k) ? 0u - up : up;
#pragma unroll
        for (int e = 0; e < k; e++) h[k + e] = h[e] + d;
    }
}

// One value (the depthwise stencil's epilogue): as hq_requant, with stochastic rounding.
__device__ inline int hq_requant_sr(int c, const HqRequant &q, const HqSr &sr, size_t idx, unsigned &nlo, unsigned &nhi)
{
    const unsigned bits = hq_sr_bits((unsigned)idx, (unsigned)(idx >> 32) * 0x85ebca77u + sr.k1, sr.k0);
    const float x = __fmul_rn((float)c, q.mult), fl = floorf(x);
    const float u = __fmul_rn((float)(bits >> 8), 1.0f / 16777216.0f);
    float r = __fsub_rn(x, fl) > u ? __fadd_rn(fl, 1.0f) : fl;
    nlo += (r < q.flo) ? 1u : 0u;
    nhi += (r > q.fhi) ? 1u : 0u;
    r = fminf(fmaxf(r, q.flo), q.fhi);
    return (int)r + q.z;
}

// As hq_requant_group, with stochastic rounding; idx0 is the tensor index of c[0], the N values
// are consecutive elements.  ALIGN (4, or N) divides idx0: channel counts are multiples of 4, and of 16 where a
// kernel takes 16 only.
template <int N, bool FULL_GRID, int ALIGN = 4>
__device__ inline void hq_requant_group_sr(const int *c, const HqEpilogue &ep, const HqSr &sr, size_t idx0, int &mn,
                                           int &mx, unsigned &w_lo, unsigned &w_hi, int *words)
{
    int gmn = c[0], gmx = c[0];
#pragma unroll
    for (int e = 1; e + 1 < N; e += 2) { gmn = hq_min3(gmn, c[e], c[e + 1]); gmx = hq_max3(gmx, c[e], c[e + 1]); }
    gmn = min(gmn, c[N - 1]); gmx = max(gmx, c[N - 1]);
    mn = min(mn, gmn); mx = max(mx, gmx);
    float f[N];
    unsigned h[N], term[N / ALIGN];
#pragma unroll
    for (int g = 0; g < N / ALIGN; g++) {                                // (no carry into the high word inside such a group)
        const size_t idx = idx0 + (size_t)(g * ALIGN);
        term[g] = (unsigned)(idx >> 32) * 0x85ebca77u + sr.k1;
        hq_sr_first_n<ALIGN>((unsigned)idx, sr.k0, h + g * ALIGN);
    }
#pragma unroll
    for (int e = 0; e < N; e++) {
        const unsigned bits = hq_sr_rest(h[e], term[e / ALIGN]);
        const float x = __fmul_rn((float)c[e], ep.mult), fl = floorf(x);
        const float u = __fmul_rn((float)(bits >> 8), 1.0f / 16777216.0f);
        f[e] = __fsub_rn(x, fl) > u ? __fadd_rn(fl, 1.0f) : fl;
    }
    // the rounded value lies in [floor(x), floor(x) + 1]: the group's extremes decide whether any can clip
    if (__any(__fadd_rn(floorf(__fmul_rn((float)gmx, ep.mult)), 1.0f) > ep.fhi || floorf(__fmul_rn((float)gmn, ep.mult)) < ep.flo)) {
        float nh = 0.0f, nl = 0.0f;
#pragma unroll
        for (int e = 0; e < N; e++) {
            nh += __builtin_amdgcn_fmed3f(f[e] - ep.fhi, 0.0f, 1.0f);
            nl += __builtin_amdgcn_fmed3f(ep.flo - f[e], 0.0f, 1.0f);
        }
        w_hi += (unsigned)nh; w_lo += (unsigned)nl;
    }
#pragma unroll
    for (int g = 0; g < N / 4; g++) {
        unsigned w = 0;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            float v = f[4 * g + e];
            if (!FULL_GRID) v = __builtin_amdgcn_fmed3f(v, ep.flo, ep.fhi);
            w = __builtin_amdgcn_cvt_pk_u8_f32(v + ep.zoff, e, w);
        }
        words[g] = (int)(w ^ 0x80808080u);
    }
}

// min / max alone (pass 1 of the dynamic baseline keeps the 32-bit values)
template <int N> __device__ inline void hq_minmax_group(const int *c, int &mn, int &mx)
{
#pragma unroll
    for (int e = 0; e + 1 < N; e += 2) { mn = hq_min3(mn, c[e], c[e + 1]); mx = hq_max3(mx, c[e], c[e + 1]); }
}

__device__ inline unsigned hq_pack4(int a, int b, int c, int d)
{
    return (unsigned)(a & 0xff) | ((unsigned)(b & 0xff) << 8) | ((unsigned)(c & 0xff) << 16) | ((unsigned)d << 24);
}

// ---------------------------------------------------------------------------------------
// Wavefront and workgroup reductions for the online statistics.
// ---------------------------------------------------------------------------------------

// The value of the lane's partner inside its row of 16 lanes, without LDS: lane ^ 1, lane ^ 2, the mirror image in the 8 lanes,
// the mirror image in the 16 lanes (K = 1, 2, 4, 8).  Applied one after the other they combine every lane with every other.
template <int K> __device__ inline int hq_lane_partner(int v)
{
    constexpr int ctrl = K == 1 ? 0xB1 : K == 2 ? 0x4E : K == 4 ? 0x141 : 0x140;
    return __builtin_amdgcn_update_dpp(0, v, ctrl, 0xf, 0xf, false);
}
template <int N, typename Op> __device__ inline int hq_row_reduce(int v, Op op)     // groups of N = 4, 8 or 16 lanes
{
    v = op(v, hq_lane_partner<1>(v));
    v = op(v, hq_lane_partner<2>(v));
    if (N > 4) v = op(v, hq_lane_partner<4>(v));
    if (N > 8) v = op(v, hq_lane_partner<8>(v));
    return v;
}

// All 64 lanes take part; the result is uniform.
template <typename Op> __device__ inline int hq_wave_reduce(int v, Op op)
{
    v = hq_row_reduce<16>(v, op);
    return op(op(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
              op(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

struct HqMin { __device__ int operator()(int a, int b) const { return a < b ? a : b; } };
struct HqMax { __device__ int operator()(int a, int b) const { return a > b ? a : b; } };
struct HqAdd { __device__ int operator()(int a, int b) const { return a + b; } };

// Merges one workgroup's statistics into the tensor's record: wavefront reduction, a
// second level through LDS, then one atomic per field from one lane, into the partial record
// chosen by the workgroup's index: consecutive workgroups land on different 128-byte lines, so
// a launch's atomics do not queue on one address.  `red` is LDS space for 4 * (NTHREADS / 64)
// ints.  Must be called by all NTHREADS threads of the workgroup; `block` is its index in the launch.
// It is the end of every launch's serial chain, so it is written for latency: exchanges inside rows of 16 lanes and scalar
// reads instead of LDS permutes, sums only where something was clipped, and the second level in one LDS read whose lanes
// hold one field each (2000 -> 1300 cycles of a small launch's 16 K).
template <int NTHREADS>
__device__ inline void hq_block_stats_commit_n(int mn, int mx, unsigned nlo, unsigned nhi,
                                               hq_stats *st, int *red, unsigned block = blockIdx.x)
{
    constexpr int NW = NTHREADS / 64;
    static_assert(NW == 4 || NW == 8 || NW == 16, "a field is a group of NW lanes");
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    mn = hq_wave_reduce(mn, HqMin());
    mx = hq_wave_reduce(mx, HqMax());
    if (__any((nlo | nhi) != 0)) {
        nlo = (unsigned)hq_wave_reduce((int)nlo, HqAdd());
        nhi = (unsigned)hq_wave_reduce((int)nhi, HqAdd());
    }
    if (lane == 0) { red[wave] = mn; red[NW + wave] = ~mx; red[2 * NW + wave] = (int)nlo; red[3 * NW + wave] = (int)nhi; }
    __syncthreads();
    if (wave == 0) {
        const int f = lane / NW, v = f < 4 ? red[lane] : 0;
        // ~ reverses the order: the smallest ~mx is that of the largest mx
        const int least = hq_row_reduce<NW>(v, HqMin()), sum = hq_row_reduce<NW>(v, HqAdd());
        int8_t *part = reinterpret_cast<int8_t *>(&st->part[block % HQ_STATS_PARTS]);
        // (a lane's own address: with a common one the compiler puts a loop over the lanes around an atomic that one lane does)
        static_assert(offsetof(hq_stats_part, acc_max) == 4 && offsetof(hq_stats_part, clip_lo) == 8 && offsetof(hq_stats_part, clip_hi) == 16, "");
        unsigned word = f < 2 ? 4u * f : 8u * (f - 1);
        asm volatile("" : "+v"(word));
        part += word;
        if (lane % NW == 0) {                              // (a workgroup without values adds none)
            if (f == 0 && least != INT_MAX) atomicMin(reinterpret_cast<int *>(part), least);
            if (f == 1 && least != INT_MAX) atomicMax(reinterpret_cast<int *>(part), ~least);
            if ((f == 2 || f == 3) && sum) atomicAdd(reinterpret_cast<unsigned long long *>(part), (unsigned long long)(unsigned)sum);
        }
    }
}

__device__ inline void hq_block_stats_commit(int mn, int mx, unsigned nlo, unsigned nhi, hq_stats *st, int *red,
                                             unsigned block = blockIdx.x)
{
    hq_block_stats_commit_n<HQ_THREADS>(mn, mx, nlo, nhi, st, red, block);
}

// Moves what the partial records hold into the record's leading fields and empties them.
// One wavefront (HQ_STATS_PARTS == 64 lanes, lane = partial record), registers only.  Lane 0
// writes the leading fields; every lane returns their new values.
struct HqStatsFolded { int acc_min, acc_max; unsigned long long clip_lo, clip_hi; };

__device__ inline unsigned long long hq_wave_sum64(unsigned long long v)
{
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
        const unsigned lo = (unsigned)__shfl_xor((int)(unsigned)v, k), hi = (unsigned)__shfl_xor((int)(unsigned)(v >> 32), k);
        v += ((unsigned long long)hi << 32) | lo;
    }
    return v;
}

__device__ inline HqStatsFolded hq_stats_fold_wave(hq_stats *st)
{
    static_assert(HQ_STATS_PARTS == 64, "one lane per partial record");
    const int lane = threadIdx.x & 63;
    hq_stats_part *p = &st->part[lane];
    const int pmn = p->acc_min, pmx = p->acc_max;
    const unsigned long long plo = p->clip_lo, phi = p->clip_hi;
    HqStatsFolded f;
    f.acc_min = st->acc_min; f.acc_max = st->acc_max; f.clip_lo = st->clip_lo; f.clip_hi = st->clip_hi;
    p->acc_min = INT_MAX; p->acc_max = INT_MIN; p->clip_lo = 0; p->clip_hi = 0;
    f.acc_min = min(f.acc_min, hq_wave_reduce(pmn, HqMin()));
    f.acc_max = max(f.acc_max, hq_wave_reduce(pmx, HqMax()));
    f.clip_lo += hq_wave_sum64(plo);
    f.clip_hi += hq_wave_sum64(phi);
    if (lane == 0) { st->acc_min = f.acc_min; st->acc_max = f.acc_max; st->clip_lo = f.clip_lo; st->clip_hi = f.clip_hi; }
    return f;
}

// eq. (2)-(3) for one quantizer, by one wavefront: folds the statistics record, moves the range,
// derives the quantizer, empties the record.  With count == 0 the range is left as it is.
__device__ inline void hq_range_update_wave(hq_range *r, hq_stats *st)
{
    // every load is issued before anything waits: one memory round trip
    hq_range rr = *r;
    const float acc_scale = st->acc_scale;
    const unsigned fp32_keys = st->fp32_keys;
    const unsigned long long count = st->count;
    const HqStatsFolded f = hq_stats_fold_wave(st);
    if ((threadIdx.x & 63) == 0) {
        if (count != 0) {
            if (fp32_keys) hq_ema_update(&rr, hq_key_float(f.acc_min), hq_key_float(f.acc_max));
            else hq_ema_update(&rr, __fmul_rn(acc_scale, (float)f.acc_min), __fmul_rn(acc_scale, (float)f.acc_max));
            *r = rr;
        }
        st->acc_min = INT_MAX; st->acc_max = INT_MIN; st->acc_scale = 0.0f; st->fp32_keys = 0;
        st->clip_lo = 0; st->clip_hi = 0; st->count = 0;           // the partial records are already empty
    }
}

// Range updates that ride along with another launch: the workgroups past `first` of that launch
// (one per quantizer, their first wavefront) run eq. (2)-(3) instead of the launch's own work.
struct HqRideAlong { hq_range *r; hq_stats *st; int n; int first; };

__device__ inline bool hq_ride_along(const HqRideAlong &ra)
{
    if (ra.n == 0 || (int)blockIdx.x < ra.first) return false;
    if (threadIdx.x < 64) hq_range_update_wave(ra.r + (blockIdx.x - ra.first), ra.st + (blockIdx.x - ra.first));
    return true;
}
