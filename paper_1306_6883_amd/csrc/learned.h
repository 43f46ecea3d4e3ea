// learned.h -- shapes and kernels of the learned initial guess (learned.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "internal.h"

namespace ccmg {

constexpr int kNetG = 128;     // grid of the network
constexpr int kNetC = 32;      // channels of the hidden layers
constexpr int kNetLayers = 6;  // dilations 1, 2, 4, 8, 16, 32
// parameter blocks (FP32 master copy, contiguous):
//   layer 0: [32 co][9 tap]            layers 1..4: [32 co][9 tap][32 ci]
//   layer 5: [9 tap][32 ci]
constexpr int kW0 = kNetC * 9;
constexpr int kWmid = kNetC * 9 * kNetC;
constexpr int kW5 = 9 * kNetC;
constexpr int kNetParams = kW0 + 4 * kWmid + kW5;  // 37440
inline int net_param_offset(int layer) { return layer == 0 ? 0 : kW0 + (layer - 1) * kWmid; }
inline int net_dilation(int layer) { return 1 << layer; }

template <bool PAIR>
__global__ void k_conv32(const __bf16 *in, const __bf16 *in_lo, const __bf16 *w, const __bf16 *w_lo, __bf16 *out,
                         __bf16 *out_lo, int dil, int seg);
__global__ void k_conv32_split(const __bf16 *in, const __bf16 *in_lo, const __bf16 *w, const __bf16 *w_lo, __bf16 *out,
                               __bf16 *out_lo, int nb, int dil);
// batches of at most this many images run k_conv32_split in the forward pass
constexpr int kConvSplitMaxBatch = 2;
// Rows per walk of k_conv32: as long as two workgroups per CU (512) have one,
// at most the rows of a class (a power of two, as both are).
inline int conv_seg(int nb, int dil) {
    int seg = 1;
    while (2 * seg <= kNetG / dil && nb * kNetG / (2 * seg) >= 512) seg *= 2;
    return seg;
}
template <int ALIGN>
__global__ void k_conv32_wgrad(const __bf16 *g, const __bf16 *in, float *part, int dil, int seg);
// Workgroups of k_conv32_wgrad (partial sums of a layer) for nb images, and the
// most that any batch up to `batch` needs.
inline int wgrad_blocks(int nb, int dil) { return nb * kNetG / conv_seg(nb, dil); }
inline int wgrad_blocks_max(int batch) {
    int most = 0;
    for (int nb = 1; nb <= batch; ++nb)
        for (int l = 1; l <= 4; ++l)
            if (wgrad_blocks(nb, net_dilation(l)) > most) most = wgrad_blocks(nb, net_dilation(l));
    return most;
}
constexpr int kSumGroups = 32;    // first-stage groups of the partial-sum reduction
constexpr int kLossBlocks = 256;  // workgroups (partial sums) of k_mse
__global__ void k_sum_partials(const float *part, int count, int len, float *out);
__global__ void k_to_bf16(const float *a, __bf16 *w16, __bf16 *w16lo, __bf16 *wt16, int count);
template <bool ADAM>
__global__ void k_finish(const float *groups, float *grad, const double *lpart, int pixels, float *loss, float *w,
                         float *m, float *v, __bf16 *w16, __bf16 *w16lo, __bf16 *wt16, float lr, float b1, float b2,
                         float eps, float c1, float c2);
__global__ void k_conv_in(const float *x, const float *w1, __bf16 *out, __bf16 *out_lo, int per, int dil);
template <int OUT>
__global__ void k_conv_out(const __bf16 *in, const __bf16 *in_lo, const float *w6, float *y);
// Batches of at most this many images run k_conv_out<1>: one workgroup a class
// leaves CUs idle there.  1, 2, 4, 8 and 16 images: 7.4, 7.7, 8.5, 9.4 and 14.8 us
// so, 8.1, 8.7, 9.0, 10.2 and 12.4 with <2>.
constexpr int kConvOutSplitMaxBatch = 8;
__global__ void k_conv_out_bwd(const float *dy, const float *w6, __bf16 *g, int per, int dil);
// Pixels per thread of k_conv_in and k_conv_out_bwd (workgroups of 64 x that
// many): as many as leave four workgroups per CU (1024), at most 16.
inline int pixels_per_thread(int nb) {
    int per = 1;
    while (per < 16 && nb * (kNetG * kNetG / 64) / (2 * per) >= 1024) per *= 2;
    return per;
}
template <bool LAST>
__global__ void k_wgrad_small(const __bf16 *act, const __bf16 *act_lo, const float *vec, float *part, int chunk,
                              int dil);
__global__ void k_mse(const float *y, const float *t, float *dy, double *part, int count);
__global__ void k_encode(const double *f, long pitch, int n, const double *sumsq, float *out);
constexpr int kRelaxThreads = 1024;
__global__ void k_coarse_relax(const float *y, const float *x, const double *sumsq, int nfine, double length,
                               int iters, double *out);
__global__ void k_decode_step(const double *c, int nc, double *fine, long out_pitch, int ghosted);

}  // namespace ccmg
