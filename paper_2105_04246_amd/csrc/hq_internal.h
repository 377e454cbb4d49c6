// Host-side launchers shared between the translation units of the hq library.
#pragma once
#include <hip/hip_runtime.h>
#include "../../include/hq.h"

#include <atomic>

// Lets `kernel` have `bytes` of dynamic LDS on the current GPU.  The attribute belongs to a kernel on one GPU; `devices` (a
// static of the caller, one for each kernel) has a bit for every GPU on which it has been set.
template <typename K> inline bool hq_allow_lds(K *kernel, size_t bytes, std::atomic<unsigned long long> &devices)
{
    if (bytes <= 48 * 1024) return true;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return false;
    const unsigned long long bit = dev < 64 ? 1ull << dev : 0;
    if (devices.load(std::memory_order_relaxed) & bit) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        return false;
    devices.fetch_or(bit, std::memory_order_relaxed);
    return true;
}

// sr_seed: NULL = round to nearest even; otherwise (host pointer) the seed of stochastic rounding.
int hq_launch_gemm(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                   const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                   int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed = nullptr);

// Launches with few output tiles (the wavefronts of a workgroup split the reduction); HQ_E_BADSHAPE: not covered.
// sr_seed as for hq_launch_gemm.
int hq_try_launch_ksplit(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                         const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                         int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream,
                         const uint64_t *sr_seed = nullptr);

// 3x3 stride-1 layers with 64 reduced channels (weights in registers); HQ_E_BADSHAPE: not covered.
// sr_seed as for hq_launch_gemm.
int hq_try_launch_regw(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                       int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream,
                       const uint64_t *sr_seed = nullptr);

// At most 192 reduced channels under one tap (pixels straight into registers, weights in LDS); HQ_E_BADSHAPE: not covered.
// sr_seed as for hq_launch_gemm.
int hq_try_launch_point(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                       int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream,
                       const uint64_t *sr_seed = nullptr);

// Fast path for 3x3 layers with 64 reduced channels whose weights fit in LDS; HQ_E_BADSHAPE means "not covered, use hq_launch_gemm".
// sr_seed as for hq_launch_gemm.
int hq_try_launch_band(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                       int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream,
                       const uint64_t *sr_seed = nullptr);

// Fast path for forward layers with 4 input channels (a network's first layer); HQ_E_BADSHAPE: not covered.
int hq_try_launch_direct(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                         const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                         int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream);

// 3x3 stride-1 layers of 128 or more channels on both sides, the reduced ones a multiple of 64, on images up to about 125 pixels wide (one row: 93);
// HQ_E_BADSHAPE: not covered.  sr_seed as for hq_launch_gemm.
int hq_try_launch_frame(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                        const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8, int32_t *out32,
                        hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed = nullptr);

// Layers whose reduced channels are a multiple of 128, from 8 lines of reduction and 65 tiles of 128 x 128 on (one tap: more);
// HQ_E_BADSHAPE: not covered.  sr_seed as for hq_launch_gemm.
int hq_try_launch_ring(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Bw,
                       const hq_qparams *bq, const int32_t *bsum, const hq_range *range, int8_t *out8,
                       int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream,
                       const uint64_t *sr_seed = nullptr);

// sr_seed as for hq_launch_gemm.
int hq_launch_depthwise(const hq_problem *p, int dgrad, const int8_t *A, const hq_qparams *aq, const int8_t *Wt,
                        const hq_qparams *bq, const int32_t *wsum, const hq_range *range, int8_t *out8,
                        int32_t *out32, hq_qparams *outq, hq_stats *st, hipStream_t stream, const uint64_t *sr_seed = nullptr);

size_t hq_wgrad_workspace_bytes(const hq_problem *p);

// ride: range updates to run in the call's last launch (NULL: none); see HqRideAlong.
struct HqRideAlong;
int hq_launch_wgrad(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                    const hq_qparams *gq, float *dW, int32_t *dW_acc, void *ws, hipStream_t stream,
                    const HqRideAlong *ride = nullptr);

// Weight gradients over few pixels, in one launch; HQ_E_BADSHAPE: not covered.
int hq_try_launch_wgrad_small(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                              const hq_qparams *gq, float *dW, int32_t *dW_acc, hipStream_t stream, const HqRideAlong *ride);

// 3x3 stride-1 layers with channel counts that are multiples of 64; HQ_E_BADSHAPE: not covered.  ws: hq_wgrad_band_bytes (0: not covered).
size_t hq_wgrad_band_bytes(const hq_problem *p);
int hq_try_launch_wgrad_band(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                             const hq_qparams *gq, float *dW, int32_t *dW_acc, void *ws, hipStream_t stream, const HqRideAlong *ride);

int hq_launch_depthwise_wgrad(const hq_problem *p, const int8_t *X, const hq_qparams *xq, const int8_t *dY,
                              const hq_qparams *gq, float *dW, int32_t *dW_acc, void *ws, hipStream_t stream,
                              const HqRideAlong *ride = nullptr);

// Weight side: re-laying and sums (one launch), Q_W (one or two launches).
int hq_launch_weight_prepare(const hq_problem *p, const int8_t *W, int8_t *Wd, int32_t *wsum, int32_t *wdsum, hipStream_t s);
int hq_launch_weight_quantize(const float *Wf, size_t n, int8_t *Wq, hq_qparams *wq, hipStream_t s);
