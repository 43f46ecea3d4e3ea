// cycle_end.h -- the end of a cycle (CycleEnd, internal.h) on one wavefront or on
// a workgroup of four, with the same sums in the same order: thread t of 256
// adds every 256th pair, the lanes of a wave meet in a butterfly, the four
// waves' totals are added in order (one wavefront plays the four in turn).
#pragma once
#include "internal.h"

namespace ccmg {

__device__ __forceinline__ double2 cycle_end_thread(const double *p, int count, int t) {
    double s0 = 0.0, s1 = 0.0;
    int i = t;
    for (; i + 3 * 256 < count; i += 4 * 256) {  // four pairs in flight, added in order
        double2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = *reinterpret_cast<const double2 *>(p + 2 * (i + k * 256));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            s0 += v[k].x;
            s1 += v[k].y;
        }
    }
    for (; i < count; i += 256) {
        s0 += p[2 * i];
        s1 += p[2 * i + 1];
    }
    return double2{s0, s1};
}
__device__ __forceinline__ double cycle_end_wave(double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
__device__ __forceinline__ void cycle_end_file(const CycleEnd &c, double s0, double s1) {
    const double rho = sqrt(s0) / sqrt(*c.f2);
    *c.rho_out = rho;
    if (c.host_rho) *c.host_rho = rho;  // read by the host after the cycle's event
    *c.phi_mean = c.singular ? s1 / ((double)c.n * (double)c.n) : 0.0;
    if (c.done && (rho <= c.rtol || !isfinite(rho))) *c.done = 1;
}
// one wavefront
__device__ __forceinline__ void cycle_end_one_wave(const CycleEnd &c) {
    if (c.done && *c.done) return;
    const int lane = threadIdx.x & 63;
    double w0[4], w1[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const double2 v = cycle_end_thread(c.partial, c.count, lane + 64 * w);
        w0[w] = v.x;
        w1[w] = v.y;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        w0[w] = cycle_end_wave(w0[w]);
        w1[w] = cycle_end_wave(w1[w]);
    }
    if (lane == 0) cycle_end_file(c, ((w0[0] + w0[1]) + w0[2]) + w0[3], ((w1[0] + w1[1]) + w1[2]) + w1[3]);
}

}  // namespace ccmg
