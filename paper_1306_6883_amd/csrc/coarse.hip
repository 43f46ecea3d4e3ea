// coarse.hip -- the bottom of the V-cycle in one launch.
//
// Levels with at most kCoarseMax cells per side are too small to fill the
// GPU, so one workgroup runs the whole rest of the V-cycle for them: from the
// top level (n_top cells per side) down to the 2 x 2 grid and back up.  From
// 32 x 32 (any grid of 32^2 cells or more) that is one wavefront with every
// level in registers (tail_body); a finest grid of 16^2 cells or fewer runs in
// coarse_body, every level in LDS (phi and f, no ghost layer: side rules are
// applied where a neighbour is read).  The steps are those of the paper's V-cycle (Sec. 3.3):
// nu1 red-black Gauss-Seidel iterations, residual and four-cell restriction,
// recursion, centred-slope prolongation without the xy term, nu2 iterations;
// on the 2 x 2 grid nu_bottom relaxations, done in FP64 whatever T is.  Or an
// exact bottom on a 4 x 4 or 8 x 8 level: its inverse operator (computed once
// per plan by k_bottom_inverse) is applied in FP64.
#include <cstdlib>

#include "internal.h"

namespace ccmg {

namespace {

// Workgroup size NT of coarse_body (a template parameter).  With NT = 64 (one
// wavefront: a batch's small grids) no workgroup barrier is needed -- a wave's
// LDS operations complete in issue order, so ordering the compiler's code is
// enough between phases.  Largest level it holds; a larger tail is tail_body's.
constexpr int kCoarseThreads = 512;
constexpr int kBodyMax = kCoarseMax / 2;

template <int NT>
__device__ __forceinline__ void sync() {
    if constexpr (NT == 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// Side rules, held in scalar registers for the whole kernel.
struct Sides {
    bool px, py;          // periodic in x / y
    float sxl, sxh, syl, syh;  // ghost sign of a Dirichlet (-1) / Neumann (+1) side
};

// Neighbour values of cell (x, y) of an n x n level (n = 1 << lg) stored
// row-major in A.  Branch-free: every neighbour is one LDS read at a wrapped
// (periodic) or clamped (own cell) index, times the ghost sign (-1 Dirichlet,
// +1 Neumann) where the neighbour is a ghost; times 1 (exact) elsewhere.
template <typename T>
__device__ __forceinline__ void neighbours(const T *A, int lg, int x, int y, const Sides &sd, T self,
                                           T &e, T &w, T &nn, T &s) {
    (void)self;
    const int nm = (1 << lg) - 1;
    const bool xh = x == nm, xl = x == 0, yh = y == nm, yl = y == 0;
    const int xe = xh ? (sd.px ? 0 : x) : x + 1;
    const int xw = xl ? (sd.px ? nm : x) : x - 1;
    const int yn = yh ? (sd.py ? 0 : y) : y + 1;
    const int yS = yl ? (sd.py ? nm : y) : y - 1;
    const T ge = (xh && !sd.px) ? T(sd.sxh) : T(1);
    const T gw = (xl && !sd.px) ? T(sd.sxl) : T(1);
    const T gn = (yh && !sd.py) ? T(sd.syh) : T(1);
    const T gs = (yl && !sd.py) ? T(sd.syl) : T(1);
    const int row = y << lg;
    e = ge * A[row + xe];
    w = gw * A[row + xw];
    nn = gn * A[(yn << lg) + x];
    s = gs * A[(yS << lg) + x];
}

// Block-wide sum in a fixed order (per-thread strided sums, per-wave butterfly,
// then the wave totals in order).  All threads get the result.
template <int NT>
__device__ double block_sum(double v, double *red) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    if constexpr (NT == 64) {
        return v;
    } else {
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) red[wave] = v;
        __syncthreads();
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NT / 64; ++i) t += red[i];
        __syncthreads();
        return t;
    }
}

template <int NT, typename T>
__device__ void relax(T *P, const T *F, int lg, const Sides &sd, T cc, T invd, int iters) {
    const int n = 1 << lg, half = (n * n) >> 1, lgh = lg - 1;
    for (int it = 0; it < iters; ++it) {
        for (int colour = 0; colour < 2; ++colour) {
            for (int i = threadIdx.x; i < half; i += NT) {
                const int y = i >> lgh;
                const int x = 2 * (i - (y << lgh)) + ((y + colour) & 1);
                const T self = P[(y << lg) + x];
                T e, w, nn, s;
                neighbours(P, lg, x, y, sd, self, e, w, nn, s);
                P[(y << lg) + x] = (F[(y << lg) + x] + cc * (((e + w) + nn) + s)) * invd;
            }
            sync<NT>();
        }
    }
}

// Fc = four-cell average of r = F - A P (fine level of n = 1 << lg cells per side).
template <int NT, typename T>
__device__ void restrict_residual(const T *P, const T *F, T *Fc, int lg, const Sides &sd, T alpha, T beta,
                                  T ih2) {
    const int lgc = lg - 1, nc = 1 << lgc;
    for (int i = threadIdx.x; i < nc * nc; i += NT) {
        const int J = i >> lgc, I = i - (J << lgc);
        T r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int x = 2 * I + (q & 1), y = 2 * J + (q >> 1);
            const T p = P[(y << lg) + x];
            T e, w, nn, s;
            neighbours(P, lg, x, y, sd, p, e, w, nn, s);
            const T lap = ((((e - p) + (w - p)) + (nn - p)) + (s - p)) * ih2;
            r[q] = F[(y << lg) + x] - (alpha * p - beta * lap);
        }
        Fc[i] = T(0.25) * (((r[0] + r[1]) + r[2]) + r[3]);
    }
    sync<NT>();
}

template <int NT, typename T>
__device__ void remove_mean(T *A, int lg, double *red) {
    const int nn = 1 << (2 * lg);
    double s = 0.0;
    for (int i = threadIdx.x; i < nn; i += NT) s += (double)A[i];
    const T m = T(block_sum<NT>(s, red) / (double)nn);
    for (int i = threadIdx.x; i < nn; i += NT) A[i] -= m;
    sync<NT>();
}

// P (fine, n = 1 << lg per side) += prolongation of E (coarse, n/2 per side).
template <int NT, typename T>
__device__ void prolong_add(const T *E, T *P, int lg, const Sides &sd) {
    const int n = 1 << lg, lgc = lg - 1;
    for (int i = threadIdx.x; i < n * n; i += NT) {
        const int y = i >> lg, x = i - (y << lg);
        const int I = x >> 1, J = y >> 1;
        const T e = E[(J << lgc) + I];
        T ee, ew, en, es;
        neighbours(E, lgc, I, J, sd, e, ee, ew, en, es);
        const T mx = T(0.5) * (ee - ew), my = T(0.5) * (en - es);
        const T dx = (x & 1) ? T(0.25) : T(-0.25), dy = (y & 1) ? T(0.25) : T(-0.25);
        P[i] = P[i] + ((e + dx * mx) + dy * my);
    }
    sync<NT>();
}

}  // namespace

// Levels with at most 2^kWaveLg cells per side run on one wave (see coarse_body).
constexpr int kWaveLg = 3;

// One level on the way down: nu1 relaxations, residual restricted to the
// next level (its mean removed for singular problems), next level's
// correction zeroed.  NTW threads (the workgroup, or the first wave) take part.
template <int NTW, typename T>
__device__ void down_level(const CoarseArgs<T> &a, const Sides &sd, T *sP, T *sF, const int *off, int lg0, int l,
                           double *red) {
    const int lg = lg0 - l;
    relax<NTW>(sP + off[l], sF + off[l], lg, sd, T(a.cc[l]), T(a.invd[l]), a.nu1);
    restrict_residual<NTW>(sP + off[l], sF + off[l], sF + off[l + 1], lg, sd, T(a.alpha), T(a.beta),
                           T(a.ih2[l]));
    if (a.singular) remove_mean<NTW>(sF + off[l + 1], lg - 1, red);
    for (int i = threadIdx.x; i < (1 << (2 * (lg - 1))); i += NTW) sP[off[l + 1] + i] = T(0);
    sync<NTW>();
}

// One level on the way up: prolongation of the next level's correction, nu2
// relaxations.
template <int NTW, typename T>
__device__ void up_level(const CoarseArgs<T> &a, const Sides &sd, T *sP, const T *sF, const int *off, int lg0,
                         int l) {
    const int lg = lg0 - l;
    prolong_add<NTW>(sP + off[l + 1], sP + off[l], lg, sd);
    relax<NTW>(sP + off[l], sF + off[l], lg, sd, T(a.cc[l]), T(a.invd[l]), a.nu2);
}

// Bottom: 2 x 2 grid, relaxation only, in FP64 registers (f, p: the grid's
// right-hand side and iterate).  Cell q = 2y + x; its x-neighbour is q^1 and
// its y-neighbour q^2.  On a 2 x 2 grid the periodic image of that neighbour
// is the same cell, and a Dirichlet / Neumann ghost is -/+ the cell itself.
template <bool PX, bool PY>
__device__ __forceinline__ void relax2_sides(double c, double invd, int iters, double xl, double xh, double yl,
                                             double yh, const double (&f)[4], double (&p)[4]) {
    double p0 = p[0], p1 = p[1], p2 = p[2], p3 = p[3];
    // x-ghost of a cell at x = 0 is its west side (x-lo), at x = 1 its east side (x-hi)
    auto upd = [&](double self, double ex, double ey, double fq, bool x0, bool y0) {
        const double e = x0 ? ex : (PX ? ex : xh * self);
        const double w = x0 ? (PX ? ex : xl * self) : ex;
        const double nn = y0 ? ey : (PY ? ey : yh * self);
        const double s = y0 ? (PY ? ey : yl * self) : ey;
        return (fq + c * (((e + w) + nn) + s)) * invd;
    };
    // An iteration is a chain of ten dependent FP64 operations.  One that
    // changes nothing is a fixed point: the remaining ones would return
    // exactly these values.  That is looked at on every fourth only, off the chain.
    for (int it = 0; it < iters;) {
        bool same = false;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (it >= iters) break;
            const double q0 = upd(p0, p1, p2, f[0], true, true);    // red (0,0)
            const double q3 = upd(p3, p2, p1, f[3], false, false);  // red (1,1)
            const double q1 = upd(p1, q0, q3, f[1], false, true);   // black (1,0)
            const double q2 = upd(p2, q3, q0, f[2], true, false);   // black (0,1)
            if (u == 3) same = q0 == p0 && q1 == p1 && q2 == p2 && q3 == p3;
            p0 = q0, p1 = q1, p2 = q2, p3 = q3;
            ++it;
        }
        if (same) break;
    }
    p[0] = p0, p[1] = p1, p[2] = p2, p[3] = p3;
}
__device__ __forceinline__ void relax2(double c, double invd, int iters, bool px, bool py, double xl, double xh,
                                       double yl, double yh, const double (&f)[4], double (&p)[4]) {
    if (px) {
        if (py) relax2_sides<true, true>(c, invd, iters, xl, xh, yl, yh, f, p);
        else relax2_sides<true, false>(c, invd, iters, xl, xh, yl, yh, f, p);
    } else {
        if (py) relax2_sides<false, true>(c, invd, iters, xl, xh, yl, yh, f, p);
        else relax2_sides<false, false>(c, invd, iters, xl, xh, yl, yh, f, p);
    }
}
template <typename T>
__device__ void bottom(const CoarseArgs<T> &a, const Sides &sd, T *sP, const T *sF, const int *off, int L) {
    if (threadIdx.x != 0) return;
    const int l = L - 1;
    double p[4], f[4];
    for (int q = 0; q < 4; ++q) {
        p[q] = sP[off[l] + q];
        f[q] = sF[off[l] + q];
    }
    relax2(a.cc[l], a.invd[l], a.nu_bottom, sd.px, sd.py, sd.sxl, sd.sxh, sd.syl, sd.syh, f, p);
    for (int q = 0; q < 4; ++q) sP[off[l] + q] = T(p[q]);
}

// Exact bottom on level l (n = 1 << lg cells per side, m = n^2 unknowns), on
// the first wave: lane i computes P[i] = sum_j ainv[i][j] F[j] in FP64 in
// column order.  ainv is column-major in LDS, so a lane reads consecutive
// doubles and F[j] is one broadcast.
template <typename T>
__device__ void direct_bottom(const double *sInv, T *P, const T *F, int lg) {
    const int m = 1 << (2 * lg);
    const int i = threadIdx.x;
    if (i < m) {
        double s = 0.0;
        for (int j = 0; j < m; ++j) s += sInv[j * m + i] * (double)F[j];
        P[i] = T(s);
    }
}

template <int NT, typename T, bool DIRECT>
__device__ void coarse_body(const CoarseArgs<T> &a) {
    __shared__ T sP[kBodyMax * kBodyMax * 4 / 3 + 8];
    __shared__ T sF[kBodyMax * kBodyMax * 4 / 3 + 8];
    __shared__ double red[NT / 64];
    __shared__ double sInv[DIRECT ? kDirectMax * kDirectMax * kDirectMax * kDirectMax : 1];
    if (a.skip && *a.skip) return;  // uniform over the workgroup

    Sides sd;
    sd.px = a.bc[CCMG_XLO] == CCMG_BC_PERIODIC;
    sd.py = a.bc[CCMG_YLO] == CCMG_BC_PERIODIC;
    sd.sxl = a.bc[CCMG_XLO] == CCMG_BC_DIRICHLET ? -1.f : 1.f;
    sd.sxh = a.bc[CCMG_XHI] == CCMG_BC_DIRICHLET ? -1.f : 1.f;
    sd.syl = a.bc[CCMG_YLO] == CCMG_BC_DIRICHLET ? -1.f : 1.f;
    sd.syh = a.bc[CCMG_YHI] == CCMG_BC_DIRICHLET ? -1.f : 1.f;

    const int n0 = a.n_top;
    const int lg0 = 31 - __clz(n0);
    // levels n0, n0/2, ..., n_bottom (2 unless the bottom is exact)
    const int lgb = DIRECT ? 31 - __clz(a.n_bottom) : 1;
    const int L = lg0 - lgb + 1;
    if (DIRECT) {  // the inverse into LDS; its loads overlap the top level's
        const int mm = 1 << (4 * lgb);
        for (int i = threadIdx.x; i < mm; i += NT) sInv[i] = a.ainv[i];
    }
    int off[8];
    off[0] = 0;
    for (int l = 1; l < L; ++l) off[l] = off[l - 1] + (1 << (2 * (lg0 - l + 1)));

    // top level in
    const T shift = (a.load_phi && a.phi_shift) ? T(*a.phi_shift) : T(0);
    for (int i = threadIdx.x; i < n0 * n0; i += NT) {
        const int y = i >> lg0, x = i - (y << lg0);
        sF[i] = a.f[(long)(y + 1) * a.pf + 1 + x];
        sP[i] = a.load_phi ? a.phi_in[(long)(y + 1) * a.pin + 1 + x] - shift : T(0);
    }
    sync<NT>();
    if (a.sub_top_mean) remove_mean<NT>(sF, lg0, red);

    // Levels of at most 8 x 8 cells (and the bottom) run on the first wave
    // alone: 64 lanes cover such a level's colour in one pass, and a wave
    // needs no workgroup barrier between phases.  lw = first such level.
    int lw = 0;
    while (lw < L && lg0 - lw > kWaveLg) ++lw;
    // down, whole workgroup
    for (int l = 0; l < lw && l + 1 < L; ++l) down_level<NT>(a, sd, sP, sF, off, lg0, l, red);
    if (NT == 64 || threadIdx.x < 64) {
        for (int l = lw; l + 1 < L; ++l) down_level<64>(a, sd, sP, sF, off, lg0, l, red);
        if (DIRECT)
            direct_bottom(sInv, sP + off[L - 1], sF + off[L - 1], lgb);
        else
            bottom(a, sd, sP, sF, off, L);
        sync<64>();
        for (int l = L - 2; l >= lw; --l) up_level<64>(a, sd, sP, sF, off, lg0, l);
    }
    sync<NT>();
    // up, whole workgroup
    for (int l = (lw < L - 1 ? lw : L - 1) - 1; l >= 0; --l) up_level<NT>(a, sd, sP, sF, off, lg0, l);
    // top level out
    for (int i = threadIdx.x; i < n0 * n0; i += NT) {
        const int y = i >> lg0, x = i - (y << lg0);
        a.phi_out[(long)(y + 1) * a.pout + 1 + x] = sP[i];
    }
}

// ---- the tail of a 32 x 32 level on one wavefront ------------------------------
// The whole of the tail is a serial chain: some 40 colour sweeps and
// transfers, each waiting for the one before.  What bounds it is the latency
// of a step, so every level lives in the registers of one wave: no barrier
// between steps, no LDS addresses, neighbours by DPP moves along x (rows of 16
// lanes, whose rotation is the periodic wrap) and one ds_bpermute per sweep
// and direction between the four rows of lanes along y.
//
// Lane = 16 g + I, g = 0 .. 3, I = 0 .. 15:
//   32 x 32: columns 2I, 2I + 1 of rows 8g .. 8g + 7 (one red and one black cell a row)
//   16 x 16: column I of rows 4g .. 4g + 3, kept as two red and two black cells
//    8 x 8:  the cell of column I / 2, row 2g + I % 2
//    4 x 4:  the cell of column I / 4, row g (in all four lanes of a quad)
//    2 x 2:  all four cells in every lane
// so that restriction and prolongation move data within a quad of lanes only.
// The arithmetic of a cell is coarse_body's, operation for operation: the same
// bits (for singular problems, whose means are summed in another order, up to
// rounding).
// Per launch, some 2.5 us of it the launch itself, against coarse_body on 512
// threads: FP64 all-Dirichlet (50 bottom iterations) 22.1 -> 9.9 us, FP64
// Helmholtz (a few) 15.1 -> 7.2, FP32 periodic (means removed) 26.1 -> 11.2;
// a batch's 512 problems 30 -> 17.5 us.  (The columns of the tail as one
// 1024 x 1024 matrix, applied by all CUs, would be faster still, but its
// rounding differs: histories near the residual floor no longer follow the
// step-by-step arithmetic.)
namespace {

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// value of the lane D to the right / left in the row of 16 lanes (rotating)
template <int D, typename T>
__device__ __forceinline__ T from_right16(T v) { return dpp<0x120 + 16 - D>(v); }
template <int D, typename T>
__device__ __forceinline__ T from_left16(T v) { return dpp<0x120 + D>(v); }
// value of the other lane of a pair (quad_perm 1 0 3 2), of lane Q of the quad
template <typename T>
__device__ __forceinline__ T pair_swap(T v) { return dpp<0xB1>(v); }
template <int Q, typename T>
__device__ __forceinline__ T quad_lane(T v) { return dpp<Q * 0x55>(v); }
// value of lane addr / 4
__device__ __forceinline__ float lane_at(int addr, float v) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int(v)));
}
__device__ __forceinline__ double lane_at(int addr, double v) {
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float lane_const(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_const(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}
// Sum of v over the wave's lanes whose index within a row of 16 is a multiple
// of 16 / N (N distinct values a row): rotations within the rows, then the
// four rows in order.  Every lane gets the result.
template <int N>
__device__ __forceinline__ double wave_total(double v) {
    if constexpr (N >= 16) v += dpp<0x121>(v);
    if constexpr (N >= 8) v += dpp<0x122>(v);
    v += dpp<0x124>(v);
    v += dpp<0x128>(v);
    return ((lane_const(v, 0) + lane_const(v, 16)) + lane_const(v, 32)) + lane_const(v, 48);
}

// Side rules and this lane's place, for the whole kernel.
template <typename T>
struct TailSides {
    bool px, py;
    T sxl, sxh, syl, syh;
    int up, dn;            // ds_bpermute addresses of lanes + 16, - 16 (wrapping)
    bool odd;              // I odd
    int I, g;
    // ghost of a neighbour outside the domain, else the neighbour
    __device__ __forceinline__ T west(bool edge, T self, T w) const { return !px && edge ? sxl * self : w; }
    __device__ __forceinline__ T east(bool edge, T self, T e) const { return !px && edge ? sxh * self : e; }
    __device__ __forceinline__ T south(bool edge, T self, T s) const { return !py && edge ? syl * self : s; }
    __device__ __forceinline__ T north(bool edge, T self, T n) const { return !py && edge ? syh * self : n; }
};

template <typename T>
struct OpConst {
    T cc, invd, alpha, beta, ih2;
    __device__ __forceinline__ T relax(T f, T e, T w, T nn, T s) const {
        return (f + cc * (((e + w) + nn) + s)) * invd;
    }
    __device__ __forceinline__ T resid(T f, T p, T e, T w, T nn, T s) const {
        const T lap = ((((e - p) + (w - p)) + (nn - p)) + (s - p)) * ih2;
        return f - (alpha * p - beta * lap);
    }
};

// prolongated correction at the fine cell of quarter offsets dx, dy
template <typename T>
__device__ __forceinline__ T slopes(T e, T ee, T ew, T en, T es, T dx, T dy) {
    const T mx = T(0.5) * (ee - ew), my = T(0.5) * (en - es);
    return (e + dx * mx) + dy * my;
}

// ---- 32 x 32
template <typename T>
__device__ __forceinline__ void relax32(T (&P)[2][8], const T (&F)[2][8], const TailSides<T> &sd, const OpConst<T> &k,
                                        int iters) {
    const bool xl = sd.I == 0, xh = sd.I == 15;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int colour = 0; colour < 2; ++colour) {
            // row r updates column (r + colour) % 2
            const T below = lane_at(sd.dn, P[colour][7]), above = lane_at(sd.up, P[1 - colour][0]);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int c = (r + colour) & 1;
                const T self = P[c][r];
                T e = c ? from_right16<1>(P[0][r]) : P[1][r];
                T w = c ? P[0][r] : from_left16<1>(P[1][r]);
                if (c) e = sd.east(xh, self, e);
                else w = sd.west(xl, self, w);
                const T nn = r < 7 ? P[c][r < 7 ? r + 1 : 7] : sd.north(sd.g == 3, self, above);
                const T s = r > 0 ? P[c][r > 0 ? r - 1 : 0] : sd.south(sd.g == 0, self, below);
                P[c][r] = k.relax(F[c][r], e, w, nn, s);
            }
        }
    }
}

// ---- 16 x 16: R[j], B[j] are the lane's red and black cells of rows 2j, 2j + 1
template <int COLOUR, typename T>
__device__ __forceinline__ void sweep16(T (&A)[2], const T (&O)[2], const T (&F)[2], const TailSides<T> &sd,
                                        const OpConst<T> &k) {
    // a cell of this colour lies in row 2j + q, q = (I + COLOUR) % 2; its
    // vertical neighbours are O[j] and the O of the row pair below (q = 0) or
    // above (q = 1)
    const bool q = sd.odd != (COLOUR == 1);
    const T ext = lane_at(q ? sd.up : sd.dn, q ? O[0] : O[1]);
    const bool xl = sd.I == 0, xh = sd.I == 15;
    T n[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const T self = A[j];
        const T e = sd.east(xh, self, from_right16<1>(O[j])), w = sd.west(xl, self, from_left16<1>(O[j]));
        T nn = q ? (j == 0 ? O[1] : ext) : O[j];
        T s = q ? O[j] : (j == 0 ? ext : O[0]);
        if (j == 1) nn = sd.north(q && sd.g == 3, self, nn);
        if (j == 0) s = sd.south(!q && sd.g == 0, self, s);
        n[j] = k.relax(F[j], e, w, nn, s);
    }
    A[0] = n[0];
    A[1] = n[1];
}
template <typename T>
__device__ __forceinline__ void relax16(T (&R)[2], T (&B)[2], const T (&FR)[2], const T (&FB)[2], const TailSides<T> &sd,
                                        const OpConst<T> &k, int iters) {
    for (int it = 0; it < iters; ++it) {
        sweep16<0>(R, B, FR, sd, k);
        sweep16<1>(B, R, FB, sd, k);
    }
}
// rows in order <-> red and black cells
template <typename T>
__device__ __forceinline__ void rows_of(const T (&R)[2], const T (&B)[2], bool odd, T (&row)[4]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        row[2 * j] = odd ? B[j] : R[j];
        row[2 * j + 1] = odd ? R[j] : B[j];
    }
}
template <typename T>
__device__ __forceinline__ void colours_of(const T (&row)[4], bool odd, T (&R)[2], T (&B)[2]) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        R[j] = odd ? row[2 * j + 1] : row[2 * j];
        B[j] = odd ? row[2 * j] : row[2 * j + 1];
    }
}

// ---- 8 x 8: one cell per lane
template <typename T>
struct Nb {
    T e, w, n, s;
};
template <typename T>
__device__ __forceinline__ Nb<T> neighbours8(T p, const TailSides<T> &sd) {
    const T other = lane_at((((threadIdx.x & 63) + (sd.odd ? 15 : 49)) & 63) * 4, p);  // lane + 16 - 1 / lane - 16 + 1
    const T pair = pair_swap(p);
    Nb<T> v;
    v.e = sd.east(sd.I >= 14, p, from_right16<2>(p));
    v.w = sd.west(sd.I < 2, p, from_left16<2>(p));
    v.n = sd.north(sd.odd && sd.g == 3, p, sd.odd ? other : pair);
    v.s = sd.south(!sd.odd && sd.g == 0, p, sd.odd ? pair : other);
    return v;
}
template <typename T>
__device__ __forceinline__ Nb<T> neighbours4(T p, const TailSides<T> &sd) {
    Nb<T> v;
    v.e = sd.east(sd.I >= 12, p, from_right16<4>(p));
    v.w = sd.west(sd.I < 4, p, from_left16<4>(p));
    v.n = sd.north(sd.g == 3, p, lane_at(sd.up, p));
    v.s = sd.south(sd.g == 0, p, lane_at(sd.dn, p));
    return v;
}
// N = 8 or 4
template <int N, typename T>
__device__ __forceinline__ void relax1(T &p, T f, const TailSides<T> &sd, const OpConst<T> &k, int iters) {
    const int x = N == 8 ? sd.I >> 1 : sd.I >> 2, y = N == 8 ? 2 * sd.g + (sd.I & 1) : sd.g;
    const bool red = ((x + y) & 1) == 0;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int colour = 0; colour < 2; ++colour) {
            const Nb<T> v = N == 8 ? neighbours8(p, sd) : neighbours4(p, sd);
            const T q = k.relax(f, v.e, v.w, v.n, v.s);
            p = red == (colour == 0) ? q : p;
        }
    }
}

// Exact bottom on the 8 x 8 or 4 x 4 level held one cell per lane: cell i =
// sum_j ainv[j m + i] f_j in FP64, j in order (f_j is the value of lane_of(j)).
template <int N, typename T>
__device__ __forceinline__ T exact_bottom(const double *__restrict__ ainv, T f, const TailSides<T> &sd) {
    constexpr int M = N * N;
    const int i = N == 8 ? (2 * sd.g + (sd.I & 1)) * 8 + (sd.I >> 1) : (threadIdx.x & 63) >> 2;
    double s = 0.0;
#pragma unroll
    for (int j0 = 0; j0 < M; j0 += 16) {
        double a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = ainv[(j0 + j) * M + i];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int q = j0 + j, y = q >> 3, x = q & 7;
            const int l = N == 8 ? 16 * (y >> 1) + 2 * x + (y & 1) : 4 * q;
            s += a[j] * (double)lane_const(f, l);
        }
    }
    return T(s);
}

template <typename T>
__device__ __forceinline__ TailSides<T> tail_sides(const int *bc) {
    const int lane = threadIdx.x & 63;
    TailSides<T> sd;
    sd.px = bc[CCMG_XLO] == CCMG_BC_PERIODIC;
    sd.py = bc[CCMG_YLO] == CCMG_BC_PERIODIC;
    sd.sxl = bc[CCMG_XLO] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    sd.sxh = bc[CCMG_XHI] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    sd.syl = bc[CCMG_YLO] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    sd.syh = bc[CCMG_YHI] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    sd.I = lane & 15;
    sd.g = lane >> 4;
    sd.odd = lane & 1;
    sd.up = ((lane + 16) & 63) * 4;
    sd.dn = ((lane + 48) & 63) * 4;
    return sd;
}

// One V-cycle of the 32 x 32 level held in P5, F5 (by one wavefront).
template <typename T>
__device__ __forceinline__ void tail_core(const CoarseArgs<T> &a, const TailSides<T> &sd, T (&P5)[2][8], T (&F5)[2][8]) {
    auto consts = [&](int l) {
        return OpConst<T>{T(a.cc[l]), T(a.invd[l]), T(a.alpha), T(a.beta), T(a.ih2[l])};
    };
    if (a.sub_top_mean) {
        double t = 0.0;
#pragma unroll
        for (int r = 0; r < 8; ++r) t += (double)F5[0][r] + (double)F5[1][r];
        const T m = T(wave_total<16>(t) / 1024.0);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            F5[0][r] -= m;
            F5[1][r] -= m;
        }
    }
    const OpConst<T> k5 = consts(0), k4 = consts(1), k3 = consts(2), k2 = consts(3);
    const bool xl = sd.I == 0, xh = sd.I == 15;
    relax32(P5, F5, sd, k5, a.nu1);
    // residual and restriction 32 -> 16
    T frow[4];
    {
        T below[2], above[2], res[2][8];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            below[c] = lane_at(sd.dn, P5[c][7]);
            above[c] = lane_at(sd.up, P5[c][0]);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const T self = P5[c][r];
                const T e = c ? sd.east(xh, self, from_right16<1>(P5[0][r])) : P5[1][r];
                const T w = c ? P5[0][r] : sd.west(xl, self, from_left16<1>(P5[1][r]));
                const T nn = r < 7 ? P5[c][r < 7 ? r + 1 : 7] : sd.north(sd.g == 3, self, above[c]);
                const T s = r > 0 ? P5[c][r > 0 ? r - 1 : 0] : sd.south(sd.g == 0, self, below[c]);
                res[c][r] = k5.resid(F5[c][r], self, e, w, nn, s);
            }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            frow[j] = T(0.25) * (((res[0][2 * j] + res[1][2 * j]) + res[0][2 * j + 1]) + res[1][2 * j + 1]);
        if (a.singular) {
            const double t = (((double)frow[0] + (double)frow[1]) + (double)frow[2]) + (double)frow[3];
            const T m = T(wave_total<16>(t) / 256.0);
#pragma unroll
            for (int j = 0; j < 4; ++j) frow[j] -= m;
        }
    }
    // 16 x 16
    T R4[2] = {T(0), T(0)}, B4[2] = {T(0), T(0)}, FR4[2], FB4[2];
    colours_of(frow, sd.odd, FR4, FB4);
    relax16(R4, B4, FR4, FB4, sd, k4, a.nu1);
    T f3;
    {
        T p[4], res[4];
        rows_of(R4, B4, sd.odd, p);
        const T below = lane_at(sd.dn, p[3]), above = lane_at(sd.up, p[0]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const T e = sd.east(xh, p[r], from_right16<1>(p[r])), w = sd.west(xl, p[r], from_left16<1>(p[r]));
            const T nn = r < 3 ? p[r < 3 ? r + 1 : 3] : sd.north(sd.g == 3, p[r], above);
            const T s = r > 0 ? p[r > 0 ? r - 1 : 0] : sd.south(sd.g == 0, p[r], below);
            res[r] = k4.resid(frow[r], p[r], e, w, nn, s);
        }
        // the pair's four cells: rows 0, 1 in the even lane, 2, 3 in the odd one
        const T o0 = pair_swap(sd.odd ? res[0] : res[2]), o1 = pair_swap(sd.odd ? res[1] : res[3]);
        const T r00 = sd.odd ? o0 : res[0], r01 = sd.odd ? res[2] : o0;
        const T r10 = sd.odd ? o1 : res[1], r11 = sd.odd ? res[3] : o1;
        f3 = T(0.25) * (((r00 + r01) + r10) + r11);
        if (a.singular) f3 -= T(wave_total<16>((double)f3) / 64.0);
    }
    // 8 x 8
    T p3 = T(0);
    if (a.n_bottom == 8) {
        p3 = exact_bottom<8>(a.ainv, f3, sd);
    } else {
        relax1<8>(p3, f3, sd, k3, a.nu1);
        T f2;
        {
            const Nb<T> v = neighbours8(p3, sd);
            const T res = k3.resid(f3, p3, v.e, v.w, v.n, v.s);
            f2 = T(0.25) * (((quad_lane<0>(res) + quad_lane<2>(res)) + quad_lane<1>(res)) + quad_lane<3>(res));
            if (a.singular) f2 -= T(wave_total<4>((double)f2) / 16.0);
        }
        // 4 x 4
        T p2 = T(0);
        if (a.n_bottom == 4) {
            p2 = exact_bottom<4>(a.ainv, f2, sd);
        } else {
            relax1<4>(p2, f2, sd, k2, a.nu1);
            // residual and restriction 4 -> 2, the 2 x 2 grid in every lane
            T f1[4], p1[4];
            {
                const Nb<T> v = neighbours4(p2, sd);
                const T res = k2.resid(f2, p2, v.e, v.w, v.n, v.s);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int l = 32 * (q >> 1) + 8 * (q & 1);  // lane of the block's first cell
                    f1[q] = T(0.25) * (((lane_const(res, l) + lane_const(res, l + 4)) + lane_const(res, l + 16)) +
                                       lane_const(res, l + 20));
                }
                if (a.singular) {
                    const T m = T(((((double)f1[0] + (double)f1[1]) + (double)f1[2]) + (double)f1[3]) / 4.0);
#pragma unroll
                    for (int q = 0; q < 4; ++q) f1[q] -= m;
                }
            }
            {
                const double fd[4] = {(double)f1[0], (double)f1[1], (double)f1[2], (double)f1[3]};
                double pd[4] = {0.0, 0.0, 0.0, 0.0};
                relax2(a.cc[4], a.invd[4], a.nu_bottom, sd.px, sd.py, sd.sxl, sd.sxh, sd.syl, sd.syh, fd, pd);
#pragma unroll
                for (int q = 0; q < 4; ++q) p1[q] = T(pd[q]);
            }
            // prolongation 2 -> 4
            const int C = sd.I >> 2, X = C >> 1, Y = sd.g >> 1;
            const T own = Y ? (X ? p1[3] : p1[2]) : (X ? p1[1] : p1[0]);
            const T ox = Y ? (X ? p1[2] : p1[3]) : (X ? p1[0] : p1[1]);
            const T oy = Y ? (X ? p1[1] : p1[0]) : (X ? p1[3] : p1[2]);
            const T ee = X ? sd.east(true, own, ox) : ox, ew = X ? ox : sd.west(true, own, ox);
            const T en = Y ? sd.north(true, own, oy) : oy, es = Y ? oy : sd.south(true, own, oy);
            p2 = p2 + slopes(own, ee, ew, en, es, (C & 1) ? T(0.25) : T(-0.25), (sd.g & 1) ? T(0.25) : T(-0.25));
            relax1<4>(p2, f2, sd, k2, a.nu2);
        }
        // prolongation 4 -> 8: the coarse cell is the quad's
        {
            const Nb<T> v = neighbours4(p2, sd);
            p3 = p3 + slopes(p2, v.e, v.w, v.n, v.s, (sd.I & 2) ? T(0.25) : T(-0.25), sd.odd ? T(0.25) : T(-0.25));
        }
        relax1<8>(p3, f3, sd, k3, a.nu2);
    }
    // prolongation 8 -> 16: coarse rows 2g (even lane of the pair) and 2g + 1 (odd lane)
    {
        const T sw = pair_swap(p3);
        const T E[2] = {sd.odd ? sw : p3, sd.odd ? p3 : sw};
        const T below = lane_at(sd.dn, E[1]), above = lane_at(sd.up, E[0]);
        const T dx = sd.odd ? T(0.25) : T(-0.25);
        T p[4];
        rows_of(R4, B4, sd.odd, p);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const T ee = sd.east(sd.I >= 14, E[q], from_right16<2>(E[q])), ew = sd.west(sd.I < 2, E[q], from_left16<2>(E[q]));
            const T en = q == 0 ? E[1] : sd.north(sd.g == 3, E[1], above);
            const T es = q == 1 ? E[0] : sd.south(sd.g == 0, E[0], below);
            p[2 * q] = p[2 * q] + slopes(E[q], ee, ew, en, es, dx, T(-0.25));
            p[2 * q + 1] = p[2 * q + 1] + slopes(E[q], ee, ew, en, es, dx, T(0.25));
        }
        colours_of(p, sd.odd, R4, B4);
    }
    relax16(R4, B4, FR4, FB4, sd, k4, a.nu2);
    // prolongation 16 -> 32: the lane's own column and rows
    {
        T E[4];
        rows_of(R4, B4, sd.odd, E);
        const T below = lane_at(sd.dn, E[3]), above = lane_at(sd.up, E[0]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T ee = sd.east(xh, E[q], from_right16<1>(E[q])), ew = sd.west(xl, E[q], from_left16<1>(E[q]));
            const T en = q < 3 ? E[q < 3 ? q + 1 : 3] : sd.north(sd.g == 3, E[3], above);
            const T es = q > 0 ? E[q > 0 ? q - 1 : 0] : sd.south(sd.g == 0, E[0], below);
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    P5[c][2 * q + h] = P5[c][2 * q + h] + slopes(E[q], ee, ew, en, es, c ? T(0.25) : T(-0.25),
                                                                 h ? T(0.25) : T(-0.25));
        }
    }
    relax32(P5, F5, sd, k5, a.nu2);
}

template <typename T>
__device__ void tail_body(const CoarseArgs<T> &a) {
    const TailSides<T> sd = tail_sides<T>(a.bc);
    // every load before the skip flag is looked at
    T P5[2][8], F5[2][8];
    const int stop = a.skip ? *a.skip : 0;
    const double shift64 = (a.load_phi && a.phi_shift) ? *a.phi_shift : 0.0;
    {
        const T *f = a.f + (long)(8 * sd.g + 1) * a.pf + 1 + 2 * sd.I;
        const T *p = a.phi_in + (long)(8 * sd.g + 1) * a.pin + 1 + 2 * sd.I;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            F5[0][r] = f[(long)r * a.pf];
            F5[1][r] = f[(long)r * a.pf + 1];
        }
        if (a.load_phi) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                P5[0][r] = p[(long)r * a.pin];
                P5[1][r] = p[(long)r * a.pin + 1];
            }
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) P5[0][r] = P5[1][r] = T(0);
        }
    }
    if (stop) return;
    const T shift = T(shift64);
    if (a.load_phi) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            P5[0][r] -= shift;
            P5[1][r] -= shift;
        }
    }
    tail_core(a, sd, P5, F5);
    T *o = a.phi_out + (long)(8 * sd.g + 1) * a.pout + 1 + 2 * sd.I;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        o[(long)r * a.pout] = P5[0][r];
        o[(long)r * a.pout + 1] = P5[1][r];
    }
}

// Total of `count` partial sums in the row march's order (every 64th value per
// lane, loaded 16 at a time, then a butterfly).
__device__ __forceinline__ double tail_sum_partials(const double *p, int count) {
    const int lane = threadIdx.x & 63;
    double s = 0.0;
    for (int i = lane; i < count; i += 16 * 64) {
        double v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = i + 64 * k < count ? p[i + 64 * k] : 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (i + 64 * k < count) s += v[k];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    return s;
}

// ---- a 64 x 64 level on four wavefronts, around the tail -----------------------
// The level above the tail has 4096 cells: as launches of its own (two per
// cycle, 4.5 - 5.5 us each, half of it the launch) it cost as much as the
// tail.  Four wavefronts hold it in registers -- lane (I, G), G = 4 wave + g:
// columns 4I .. 4I + 3 of rows 4G .. 4G + 3 -- with x neighbours by DPP
// rotations as in the tail; a row group's first and last rows go through LDS
// (by colour, so one barrier per sweep), and the coarse right-hand side and
// correction too, for the first wavefront's tail.  The arithmetic of a cell is
// the row march's (products fused into sums within an expression only).
// FP64 Helmholtz: 11.2 us for 4.6 + 7.3 + 4.6 as three launches; periodic, with
// means, 13.8 for 5.5 + 8.9 + 5.5.
template <typename T>
struct L64 {
    static constexpr int CS = 34;                 // row stride of the coarse field in LDS
    T P[4][4], F[4][4];                           // [column][row]
    T (*E)[2][16][32];                            // [colour][first / last row][G][cells of the colour]
    T *C;                                         // [32][CS]
    int G;

    __device__ __forceinline__ void publish(int q) {  // the edge rows' cells of colour q
        const int k = 2 * (threadIdx.x & 15);
        E[q][0][G][k] = q ? P[1][0] : P[0][0];
        E[q][0][G][k + 1] = q ? P[3][0] : P[2][0];
        E[q][1][G][k] = q ? P[0][3] : P[1][3];
        E[q][1][G][k + 1] = q ? P[2][3] : P[3][3];
    }
    // neighbours of cell (c, r); s[], n[]: the rows below row 0 and above row 3
    __device__ __forceinline__ Nb<T> around(int c, int r, const T (&s)[4], const T (&n)[4], const TailSides<T> &sd) const {
        const T self = P[c][r];
        Nb<T> v;
        v.e = c < 3 ? P[c < 3 ? c + 1 : 3][r] : sd.east(sd.I == 15, self, from_right16<1>(P[0][r]));
        v.w = c > 0 ? P[c > 0 ? c - 1 : 0][r] : sd.west(sd.I == 0, self, from_left16<1>(P[3][r]));
        v.n = r < 3 ? P[c][r < 3 ? r + 1 : 3] : sd.north(G == 15, self, n[c]);
        v.s = r > 0 ? P[c][r > 0 ? r - 1 : 0] : sd.south(G == 0, self, s[c]);
        return v;
    }
    // one colour sweep; the other colour's edges are published
    template <int Q>
    __device__ __forceinline__ void sweep(const TailSides<T> &sd, const OpConst<T> &k) {
#pragma clang fp contract(on)
        const int at = 2 * sd.I;
        T s[4], n[4];
        s[Q] = E[1 - Q][1][(G + 15) & 15][at];
        s[Q + 2] = E[1 - Q][1][(G + 15) & 15][at + 1];
        n[1 - Q] = E[1 - Q][0][(G + 1) & 15][at];
        n[3 - Q] = E[1 - Q][0][(G + 1) & 15][at + 1];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = (r + Q) & 1; c < 4; c += 2) {
                const Nb<T> v = around(c, r, s, n, sd);
                P[c][r] = (F[c][r] + k.cc * (((v.e + v.w) + v.n) + v.s)) * k.invd;
            }
        publish(Q);
        __syncthreads();
    }
    // relaxations; zero: from a zero iterate, whose first red sweep reads no neighbour
    __device__ __forceinline__ void relax(const TailSides<T> &sd, const OpConst<T> &k, int iters, bool zero) {
        for (int it = 0; it < iters; ++it) {
            if (it == 0 && zero) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int c = r & 1; c < 4; c += 2) P[c][r] = F[c][r] * k.invd;
                publish(0);
                __syncthreads();
            } else {
                sweep<0>(sd, k);
            }
            sweep<1>(sd, k);
        }
    }
    // both colours' edges around the lane's cells
    __device__ __forceinline__ void edges(T (&s)[4], T (&n)[4], const TailSides<T> &sd) const {
        const int at = 2 * sd.I;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            s[c] = E[1 - (c & 1)][1][(G + 15) & 15][at + (c >> 1)];
            n[c] = E[c & 1][0][(G + 1) & 15][at + (c >> 1)];
        }
    }
    __device__ __forceinline__ T resid(int c, int r, const T (&s)[4], const T (&n)[4], const TailSides<T> &sd,
                                       const OpConst<T> &k) const {
#pragma clang fp contract(on)
        const Nb<T> v = around(c, r, s, n, sd);
        const T p = P[c][r];
        const T lap = ((((v.e - p) + (v.w - p)) + (v.n - p)) + (v.s - p)) * k.ih2;
        return F[c][r] - (k.alpha * p - k.beta * lap);
    }
    // the residual's four-cell averages into C
    __device__ __forceinline__ void restrict_to(const TailSides<T> &sd, const OpConst<T> &k) {
        T s[4], n[4];
        edges(s, n, sd);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const T r00 = resid(2 * a, 2 * b, s, n, sd, k), r01 = resid(2 * a + 1, 2 * b, s, n, sd, k);
                const T r10 = resid(2 * a, 2 * b + 1, s, n, sd, k), r11 = resid(2 * a + 1, 2 * b + 1, s, n, sd, k);
                C[(2 * G + b) * CS + 2 * sd.I + a] = T(0.25) * (((r00 + r01) + r10) + r11);
            }
    }
    // sums of r^2 and phi over the lane's cells
    __device__ __forceinline__ void norm(const TailSides<T> &sd, const OpConst<T> &k, double &r2, double &ph) const {
        T s[4], n[4];
        edges(s, n, sd);
        r2 = ph = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double q = (double)resid(c, r, s, n, sd, k);
                r2 += q * q;
                ph += (double)P[c][r];
            }
    }
    // P += prolongation of the coarse correction in C
    __device__ __forceinline__ void prolong(const TailSides<T> &sd) {
        T m[4][2], wv[2], ev[2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T *row = C + ((2 * G + q + 31) & 31) * CS + 2 * sd.I;
            m[q][0] = row[0];
            m[q][1] = row[1];
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            wv[b] = sd.west(sd.I == 0, m[1 + b][0], from_left16<1>(m[1 + b][1]));
            ev[b] = sd.east(sd.I == 15, m[1 + b][1], from_right16<1>(m[1 + b][0]));
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const T e = m[1 + b][a];
                const T ee = a ? ev[b] : m[1 + b][1], ew = a ? m[1 + b][0] : wv[b];
                const T en = b ? sd.north(G == 15, e, m[3][a]) : m[2][a];
                const T es = b ? m[1][a] : sd.south(G == 0, e, m[0][a]);
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        P[2 * a + x][2 * b + h] = P[2 * a + x][2 * b + h] +
                                                  slopes(e, ee, ew, en, es, x ? T(0.25) : T(-0.25),
                                                         h ? T(0.25) : T(-0.25));
            }
    }
    // one V-cycle (whole workgroup); the tail runs on the first wavefront
    __device__ __forceinline__ void cycle(const CoarseArgs<T> &a, const TailSides<T> &sd, const OpConst<T> &k, bool zero) {
        relax(sd, k, a.nu1, zero);
        restrict_to(sd, k);
        __syncthreads();
        if (threadIdx.x < 64) {
            T P5[2][8], F5[2][8];
            T *c = C + 8 * sd.g * CS + 2 * sd.I;
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    F5[x][r] = c[r * CS + x];
                    P5[x][r] = T(0);
                }
            tail_core(a, sd, P5, F5);
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int x = 0; x < 2; ++x) c[r * CS + x] = P5[x][r];
        }
        __syncthreads();
        prolong(sd);
        publish(1);  // the red sweep reads the black edges
        publish(0);
        __syncthreads();
        relax(sd, k, a.nu2, false);
    }
};

}  // namespace

template <typename T>
__global__ __launch_bounds__(64) void k_tail(const CoarseArgs<T> a) {
    tail_body<T>(a);
}

// A 64 x 64 level below the finest and its tail, from a zero iterate.
template <typename T>
__global__ __launch_bounds__(256) void k_tail64(const Tail64Args<T> a) {
    __shared__ T edge[2][2][16][32];
    __shared__ T coarse[32 * L64<T>::CS];
    const TailSides<T> sd = tail_sides<T>(a.c.bc);
    const OpConst<T> k{T(a.cc), T(a.invd), T(a.c.alpha), T(a.c.beta), T(a.ih2)};
    L64<T> lv;
    lv.E = edge;
    lv.C = coarse;
    lv.G = 4 * (threadIdx.x >> 6) + sd.g;
    const int stop = a.c.skip ? *a.c.skip : 0;
    const T *f = a.c.f + (long)(4 * lv.G + 1) * a.c.pf + 1 + 4 * sd.I;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            lv.F[c][r] = f[(long)r * a.c.pf + c];
            lv.P[c][r] = T(0);
        }
    if (a.fmean_part) {
        const T m = T(tail_sum_partials(a.fmean_part, a.fmean_count) / 4096.0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) lv.F[c][r] -= m;
    }
    if (stop) return;  // uniform
    if (a.c.nu1 == 0) {  // no sweep publishes the (zero) edges
        lv.publish(0);
        lv.publish(1);
        __syncthreads();
    }
    lv.cycle(a.c, sd, k, true);
    T *o = a.c.phi_out + (long)(4 * lv.G + 1) * a.c.pout + 1 + 4 * sd.I;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) o[(long)r * a.c.pout + c] = lv.P[c][r];
}

// ---- whole solves of 64 x 64 and 32 x 32 grids ---------------------------------
// A cycle of such a grid is a few microseconds of work behind three launches,
// an event and the host's stop test.  The levels already live in one
// workgroup's registers, so the whole solve does: V-cycles until the residual
// is within the tolerance (or not finite, or max_cycles have run), in one
// launch.  f's statistics come from its loads; a right-hand side that ends the
// solve (zero, not finite, or of nonzero mean on a singular problem) does so
// before the first cycle.  The arithmetic of a cell is the separate launches'.
// (64 x 64 Dirichlet, 12 cycles: 345 us in 38 launches, 173 in two, of which 155
// are this one.)
namespace {
// sum over the workgroup (fixed order), in every thread
template <int NT>
__device__ __forceinline__ double solo_sum(double v, double *red) {
    if constexpr (NT == 64) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        return v;
    } else {
        return block_sum<NT>(v, red);
    }
}
struct FStats {
    double s = 0.0, a = 0.0, q = 0.0, bad = 0.0;
    __device__ __forceinline__ void add(double v) {
        if (!isfinite(v)) {
            bad += 1.0;
        } else {
            s += v;
            a += fabs(v);
            q += v * v;
        }
    }
};
// The solve around a level held in registers.  start() readies a loaded guess
// for norm(); norm(r2, phi) gives this lane's sums, shift(m) subtracts m from
// the iterate, cycle(zero) runs a V-cycle.  Returns false when the iterate is
// not to be stored.
template <int NT, typename Start, typename Norm, typename Shift, typename Cycle>
__device__ bool solo_solve(const SoloArgs &a, double cells, FStats fs, double *red, Start &&start, Norm &&norm,
                           Shift &&shift, Cycle &&cycle) {
    double *info = a.out + CCMG_HISTORY;  // cycles, then f's statistics
    fs.s = solo_sum<NT>(fs.s, red);
    fs.a = solo_sum<NT>(fs.a, red);
    fs.q = solo_sum<NT>(fs.q, red);
    fs.bad = solo_sum<NT>(fs.bad, red);
    const bool first = threadIdx.x == 0;
    if (first) {
        info[0] = 0.0;
        info[1] = fs.s;
        info[2] = fs.a;
        info[3] = fs.q;
        info[4] = fs.bad;
    }
    if (fs.bad > 0.0 || !isfinite(fs.q) || fs.q == 0.0 || (a.singular && fabs(fs.s) > 1e-12 * fs.a)) return false;
    const double fnorm = sqrt(fs.q);
    auto residual = [&]() -> double {
        double r2, ph;
        norm(r2, ph);
        r2 = solo_sum<NT>(r2, red);
        ph = solo_sum<NT>(ph, red);
        if (a.singular) shift(ph / cells);
        return sqrt(r2) / fnorm;
    };
    double rho = 1.0;
    start();
    if (a.use_guess) rho = residual();
    if (first) a.out[0] = rho;
    if (!isfinite(rho)) return false;
    int k = 0;
    while (rho > a.rtol && k < a.max_cycles) {
        cycle(k == 0 && !a.use_guess);
        ++k;
        rho = residual();
        if (first) a.out[k] = rho;
        if (!isfinite(rho)) break;
    }
    if (first) info[0] = (double)k;
    return true;
}
}  // namespace

__global__ __launch_bounds__(256) void k_solve64(const SoloArgs a) {
    __shared__ double edge[2][2][16][32];
    __shared__ double coarse[32 * L64<double>::CS];
    __shared__ double red[4];
    const TailSides<double> sd = tail_sides<double>(a.c.bc);
    const OpConst<double> k{a.cc, a.invd, a.c.alpha, a.c.beta, a.ih2};
    L64<double> lv;
    lv.E = edge;
    lv.C = coarse;
    lv.G = 4 * (threadIdx.x >> 6) + sd.g;
    const double *f = a.f + (long)(4 * lv.G + 1) * a.pitch + 1 + 4 * sd.I;
    double *p = a.phi + (long)(4 * lv.G + 1) * a.pitch + 1 + 4 * sd.I;
    FStats fs;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            lv.F[c][r] = f[(long)r * a.pitch + c];
            lv.P[c][r] = a.use_guess ? p[(long)r * a.pitch + c] : 0.0;
        }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) fs.add(lv.F[c][r]);
    auto publish = [&]() {
        lv.publish(0);
        lv.publish(1);
        __syncthreads();
    };
    const bool store = solo_solve<256>(
        a, 4096.0, fs, red, publish, [&](double &r2, double &ph) { lv.norm(sd, k, r2, ph); },
        [&](double m) {  // (block sums have passed a barrier since the edges were read)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) lv.P[c][r] -= m;
            publish();
        },
        [&](bool zero) { lv.cycle(a.c, sd, k, zero); });
    if (!store) return;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) p[(long)r * a.pitch + c] = lv.P[c][r];
}

__global__ __launch_bounds__(64) void k_solve32(const SoloArgs a) {
    const TailSides<double> sd = tail_sides<double>(a.c.bc);
    const OpConst<double> k{a.cc, a.invd, a.c.alpha, a.c.beta, a.ih2};
    double P5[2][8], F5[2][8];
    const double *f = a.f + (long)(8 * sd.g + 1) * a.pitch + 1 + 2 * sd.I;
    double *p = a.phi + (long)(8 * sd.g + 1) * a.pitch + 1 + 2 * sd.I;
    FStats fs;
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            F5[c][r] = f[(long)r * a.pitch + c];
            P5[c][r] = a.use_guess ? p[(long)r * a.pitch + c] : 0.0;
        }
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) fs.add(F5[c][r]);
    const bool store = solo_solve<64>(
        a, 1024.0, fs, nullptr, [] {},
        [&](double &r2, double &ph) {
            double below[2], above[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                below[c] = lane_at(sd.dn, P5[c][7]);
                above[c] = lane_at(sd.up, P5[c][0]);
            }
            r2 = ph = 0.0;
#pragma unroll
            for (int r = 0; r < 8; ++r)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const double self = P5[c][r];
                    const double e = c ? sd.east(sd.I == 15, self, from_right16<1>(P5[0][r])) : P5[1][r];
                    const double w = c ? P5[0][r] : sd.west(sd.I == 0, self, from_left16<1>(P5[1][r]));
                    const double nn = r < 7 ? P5[c][r < 7 ? r + 1 : 7] : sd.north(sd.g == 3, self, above[c]);
                    const double s = r > 0 ? P5[c][r > 0 ? r - 1 : 0] : sd.south(sd.g == 0, self, below[c]);
                    const double q = k.resid(F5[c][r], self, e, w, nn, s);
                    r2 += q * q;
                    ph += self;
                }
        },
        [&](double m) {
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                P5[0][r] -= m;
                P5[1][r] -= m;
            }
        },
        [&](bool) { tail_core(a.c, sd, P5, F5); });
    if (!store) return;
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) p[(long)r * a.pitch + c] = P5[c][r];
}

hipError_t launch_solo(const SoloArgs &a0, int n, hipStream_t s) {
    SoloArgs a = a0;
    if ((n != 32 && n != 64) || a.c.n_top != kCoarseMax || a.max_cycles >= CCMG_HISTORY) return hipErrorInvalidValue;
    coarse_fill_consts(a.c);
    const bool direct = a.c.n_bottom >= 4;
    if (direct && (a.c.n_bottom > kDirectMax || (a.c.n_bottom & (a.c.n_bottom - 1)) || !a.c.ainv))
        return hipErrorInvalidValue;
    if (!direct) a.c.n_bottom = 0;
    if (n == 64) hipLaunchKernelGGL(k_solve64, dim3(1), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_solve32, dim3(1), dim3(64), 0, s, a);
    return hipGetLastError();
}

template <int NT, typename T, bool DIRECT>
__global__ __launch_bounds__(NT) void k_coarse(const CoarseArgs<T> a) {
    coarse_body<NT, T, DIRECT>(a);
}

// Batches: one wavefront per problem (relaxation bottom).
template <typename T>
__global__ __launch_bounds__(64) void k_coarse_list(const CoarseArgs<T> *__restrict__ list) {
    const CoarseArgs<T> &a = list[blockIdx.x];
    if (a.n_top == kCoarseMax) tail_body<T>(a);
    else coarse_body<64, T, false>(a);
}

// Inverse of a small level's operator by Gauss-Jordan elimination on [A | I]
// in LDS, one workgroup.  No pivoting: the operator is definite (symmetric,
// all eigenvalues of one sign; a singular one is made definite by c 1 1^T with
// c of the operator's sign), so every pivot is a nonzero Schur complement
// entry.  Four threads per row, each a quarter of the 2m columns.
constexpr int kInvThreads = 256;
__global__ __launch_bounds__(kInvThreads) void k_bottom_inverse(int lgb, int bc0, int bc1, int bc2, int bc3,
                                                                double alpha, double beta, double h, int singular,
                                                                double *__restrict__ out) {
    constexpr int kM = kDirectMax * kDirectMax;
    __shared__ double M[kM][2 * kM];
    const int nb = 1 << lgb, m = nb * nb, w = 2 * m;
    const int bc[4] = {bc0, bc1, bc2, bc3};
    const double c = beta / (h * h);
    for (int k = threadIdx.x; k < m; k += kInvThreads) {
        for (int q = 0; q < m; ++q) M[k][q] = singular ? c : 0.0;  // A (+ c 1 1^T) ...
        for (int q = m; q < w; ++q) M[k][q] = (q == k + m) ? 1.0 : 0.0;  // ... | I
        const int i = k % nb, j = k / nb;
        M[k][k] += alpha + 4.0 * c;
        const int ni[4] = {i - 1, i + 1, i, i}, nj[4] = {j, j, j - 1, j + 1};
        for (int s = 0; s < 4; ++s) {
            const bool inside = ni[s] >= 0 && ni[s] < nb && nj[s] >= 0 && nj[s] < nb;
            if (inside || bc[s] == CCMG_BC_PERIODIC)
                M[k][((nj[s] + nb) % nb) * nb + (ni[s] + nb) % nb] -= c;
            else  // ghost = -cell (Dirichlet) or +cell (Neumann)
                M[k][k] -= (bc[s] == CCMG_BC_DIRICHLET ? -c : c);
        }
    }
    const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
    const int q0 = part * (w / 4), q1 = q0 + w / 4;
    for (int col = 0; col < m; ++col) {
        __syncthreads();
        const double piv = M[col][col];
        const double g = (r < m && r != col) ? M[r][col] / piv : 0.0;
        __syncthreads();
        if (r < m && r != col)
            for (int q = q0; q < q1; ++q) M[r][q] -= g * M[col][q];
        __syncthreads();
        if (r == col)
            for (int q = q0; q < q1; ++q) M[col][q] /= piv;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < m * m; t += kInvThreads) {
        const int k = t % m, q = t / m;  // out[q * m + k] = inverse[k][q]
        out[t] = M[k][m + q];
    }
}

hipError_t launch_bottom_inverse(int nb, const int bc[4], double alpha, double beta, double h, int singular,
                                 double *out, hipStream_t s) {
    if (nb < 4 || nb > kDirectMax || (nb & (nb - 1)) || !out) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bottom_inverse, dim3(1), dim3(kInvThreads), 0, s, 31 - __builtin_clz(nb), bc[0], bc[1],
                       bc[2], bc[3], alpha, beta, h, singular, out);
    return hipGetLastError();
}

template <typename T>
void coarse_fill_consts(CoarseArgs<T> &a) {
    for (int l = 0; (a.n_top >> l) >= 2 && l < 8; ++l) {
        const double h = a.h_top * (double)(1 << l);
        const double c = a.beta / (h * h);
        a.cc[l] = c;
        a.invd[l] = 1.0 / (a.alpha + 4.0 * c);
        a.ih2[l] = 1.0 / (h * h);
    }
}

template <typename T>
hipError_t launch_coarse(const CoarseArgs<T> &a0, hipStream_t s) {
    if (a0.n_top < 2 || a0.n_top > kCoarseMax || (a0.n_top & (a0.n_top - 1))) return hipErrorInvalidValue;
    CoarseArgs<T> a = a0;
    coarse_fill_consts(a);
    const bool direct = a.n_bottom >= 4;
    if (direct && (a.n_bottom > kDirectMax || a.n_bottom > a.n_top || (a.n_bottom & (a.n_bottom - 1)) || !a.ainv))
        return hipErrorInvalidValue;
    if (a.n_top == kCoarseMax) {
        if (!direct) a.n_bottom = 0;
        hipLaunchKernelGGL(k_tail<T>, dim3(1), dim3(64), 0, s, a);
        return hipGetLastError();
    }
    constexpr int NT = kCoarseThreads;  // smaller finest levels
    if (direct) hipLaunchKernelGGL((k_coarse<NT, T, true>), dim3(1), dim3(NT), 0, s, a);
    else hipLaunchKernelGGL((k_coarse<NT, T, false>), dim3(1), dim3(NT), 0, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_tail64(const Tail64Args<T> &a0, hipStream_t s) {
    Tail64Args<T> a = a0;
    if (a.c.n_top != kCoarseMax || a.c.load_phi) return hipErrorInvalidValue;
    coarse_fill_consts(a.c);
    const bool direct = a.c.n_bottom >= 4;
    if (direct && (a.c.n_bottom > kDirectMax || (a.c.n_bottom & (a.c.n_bottom - 1)) || !a.c.ainv))
        return hipErrorInvalidValue;
    if (!direct) a.c.n_bottom = 0;
    hipLaunchKernelGGL(k_tail64<T>, dim3(1), dim3(256), 0, s, a);
    return hipGetLastError();
}
template hipError_t launch_tail64<double>(const Tail64Args<double> &, hipStream_t);
template hipError_t launch_tail64<float>(const Tail64Args<float> &, hipStream_t);

template <typename T>
hipError_t launch_coarse_list(const CoarseArgs<T> *list, int count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_coarse_list<T>, dim3(count), dim3(64), 0, s, list);
    return hipGetLastError();
}

template hipError_t launch_coarse<double>(const CoarseArgs<double> &, hipStream_t);
template hipError_t launch_coarse<float>(const CoarseArgs<float> &, hipStream_t);
template hipError_t launch_coarse_list<float>(const CoarseArgs<float> *, int, hipStream_t);
template hipError_t launch_coarse_list<double>(const CoarseArgs<double> *, int, hipStream_t);
template void coarse_fill_consts<float>(CoarseArgs<float> &);
template void coarse_fill_consts<double>(CoarseArgs<double> &);

}  // namespace ccmg
