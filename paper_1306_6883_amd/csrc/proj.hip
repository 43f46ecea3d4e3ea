// proj.hip -- the cell-centred approximate projection (Sec. 3.5).
//
// A cell-centred velocity U* = (u, v) on the doubly periodic square is split
// as U^d + grad phi: Lap phi = D U*, then U = U* - G phi.  D and G are
// centred differences across two cells, Lap the solver's 5-point operator
// (D G != Lap: the projection is approximate).  Both passes are bound by
// memory: one thread per column of a short band of rows, whose loads are all
// issued before the first is used; neighbours wrap.  (Bands of 32 rows, row
// after row, left 128 workgroups at 1024^2: 15.5 us for the divergence and
// 18.3 for the gradient; now 7.1 and 9.1.)
#include <type_traits>

#include "internal.h"

namespace ccmg {

namespace {

constexpr int kPjThreads = 256;

template <int ROWS>
__global__ __launch_bounds__(kPjThreads) void k_divergence(const double *__restrict__ u, const double *__restrict__ v,
                                                           double *__restrict__ f, long pitch, int n, double i2h) {
    const int x = blockIdx.x * kPjThreads + threadIdx.x;
    if (x >= n) return;
    const int nm = n - 1;
    const int xw = x > 0 ? x - 1 : nm, xe = x < nm ? x + 1 : 0;
    const int y0 = blockIdx.y * ROWS;
    double ue[ROWS], uw[ROWS], vr[ROWS + 2];
#pragma unroll
    for (int r = 0; r < ROWS + 2; ++r) vr[r] = v[(long)(((y0 + r - 1) & nm) + 1) * pitch + 1 + x];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double *ur = u + (long)(((y0 + r) & nm) + 1) * pitch + 1;
        ue[r] = ur[xe];
        uw[r] = ur[xw];
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double dux = (ue[r] - uw[r]) * i2h;
        const double dvy = (vr[r + 2] - vr[r]) * i2h;
        if (y0 + r < n) f[(long)(y0 + r + 1) * pitch + 1 + x] = dux + dvy;
    }
}

template <int ROWS>
__global__ __launch_bounds__(kPjThreads) void k_subtract_gradient(const double *__restrict__ phi,
                                                                  double *__restrict__ u, double *__restrict__ v,
                                                                  long pitch, int n, double i2h) {
    const int x = blockIdx.x * kPjThreads + threadIdx.x;
    if (x >= n) return;
    const int nm = n - 1;
    const int xw = x > 0 ? x - 1 : nm, xe = x < nm ? x + 1 : 0;
    const int y0 = blockIdx.y * ROWS;
    double pe[ROWS], pw[ROWS], pr[ROWS + 2], uo[ROWS], vo[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS + 2; ++r) pr[r] = phi[(long)(((y0 + r - 1) & nm) + 1) * pitch + 1 + x];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const long row = (long)(((y0 + r) & nm) + 1) * pitch + 1;
        pe[r] = phi[row + xe];
        pw[r] = phi[row + xw];
        uo[r] = u[row + x];
        vo[r] = v[row + x];
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        if (y0 + r >= n) break;
        const long o = (long)(y0 + r + 1) * pitch + 1 + x;
        u[o] = uo[r] - (pe[r] - pw[r]) * i2h;
        v[o] = vo[r] - (pr[r + 2] - pr[r]) * i2h;
    }
}

// Rows per band: four up to 1024^2, where that gives each CU four workgroups;
// above it eight, which read two rows of halo for eight instead of for four.
template <typename F>
void with_rows(int n, F &&go) {
    if (n <= 1024) go(std::integral_constant<int, 4>{});
    else go(std::integral_constant<int, 8>{});
}
dim3 bands(int n, int rows) { return dim3((n + kPjThreads - 1) / kPjThreads, (n + rows - 1) / rows); }

}  // namespace

hipError_t launch_divergence(const double *u, const double *v, double *f, long pitch, int n, double h,
                             hipStream_t s) {
    with_rows(n, [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        hipLaunchKernelGGL(k_divergence<R>, bands(n, R), dim3(kPjThreads), 0, s, u, v, f, pitch, n, 1.0 / (2.0 * h));
    });
    return hipGetLastError();
}

hipError_t launch_subtract_gradient(const double *phi, double *u, double *v, long pitch, int n, double h,
                                    hipStream_t s) {
    with_rows(n, [&](auto rows) {
        constexpr int R = decltype(rows)::value;
        hipLaunchKernelGGL(k_subtract_gradient<R>, bands(n, R), dim3(kPjThreads), 0, s, phi, u, v, pitch, n,
                           1.0 / (2.0 * h));
    });
    return hipGetLastError();
}

}  // namespace ccmg
