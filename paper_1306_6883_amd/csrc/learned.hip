// learned.hip -- kernels of the learned initial guess.
//
// The network maps the right-hand side, averaged onto a G x G grid (G = 128),
// to the solution on that grid.  The map it has to learn is linear, so the
// network is linear: six 3x3 convolutions with circular padding and dilations
// 1, 2, 4, 8, 16, 32 (receptive field 127 cells: the whole periodic grid),
// channels 1 -> 32 -> 32 -> 32 -> 32 -> 32 -> 1, no biases.  Activations are
// pixel-major with the 32 channels contiguous ([b][y][x][c]) and carried
// between layers as a pair of BF16 planes (hi + lo, about 16 significant bits:
// a single BF16 activation puts a noise floor of about 1% on the output);
// weights are BF16 copies of FP32 master weights; gradients are single BF16.
//
// The 32 -> 32 layers are implicit GEMMs on the matrix cores
// (v_mfma_f32_32x32x16_bf16, FP32 accumulation): M = 32 pixels of one row,
// N = 32 output channels, K = 9 taps x 32 input channels.  The input gradient
// of such a layer is the same product with transposed, tap-flipped weights;
// the weight gradient is a product with K running over pixels.  The 1-channel
// first and last layers are small and run on the vector units.
//
// Operand layouts of v_mfma_f32_32x32x16_bf16 (wave64): lane l holds
//   A (32 x 16): row l % 32, k = 8 (l / 32) + i, i = 0..7;
//   B (16 x 32): column l % 32, k = 8 (l / 32) + i;
//   D (32 x 32, FP32): register j holds row 8 (j / 4) + 4 (l / 32) + j % 4,
//   column l % 32.
#include "learned.h"

#include <type_traits>

namespace ccmg {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

__device__ __forceinline__ int wrapg(int v) { return v & (kNetG - 1); }
// tap t = 3 ky + kx -> offset (ky - 1, kx - 1) * dilation
__device__ __forceinline__ int tap_dy(int t, int d) { return (t / 3 - 1) * d; }
__device__ __forceinline__ int tap_dx(int t, int d) { return (t % 3 - 1) * d; }

__device__ __forceinline__ bf16x8 load8(const __bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }

// Workgroups are dealt to the 8 XCDs round robin; when the grid divides by 8,
// give each XCD a contiguous run of workgroup indices instead, so that the
// rows one XCD's waves read for their (dilated) taps stay in its L2.
__device__ __forceinline__ int xcd_block() {
    const int nb = gridDim.x, b = blockIdx.x;
    return (nb & 7) == 0 ? (b & 7) * (nb >> 3) + (b >> 3) : b;
}

}  // namespace

// out[b][y][x][co] = sum_{tap, ci} w[co][tap][ci] * in[b][y + dy][x + dx][ci]
// An activation is carried as a pair of BF16 values (hi + lo, about 16
// significant bits) and so are the weights: a product takes three MFMAs (hi w,
// lo w, hi w_lo; lo x lo is below the FP32 sums' rounding).  Gradients are one
// BF16 value, one MFMA.  The FP32 sum runs over tap, then 16 channels, then
// those products, in that order in both kernels' wavefronts.

// Batches too small to give every CU a few rows (at most kConvSplitMaxBatch
// images): one 32-pixel tile of a row per workgroup of 192; wavefront s takes
// taps 3s .. 3s + 2 straight from memory and the first adds the other two's
// partial sums from LDS, (acc0 + acc1) + acc2.
__global__ __launch_bounds__(192, 3) void k_conv32_split(const __bf16 *__restrict__ in,
                                                         const __bf16 *__restrict__ in_lo,
                                                         const __bf16 *__restrict__ w,
                                                         const __bf16 *__restrict__ w_lo, __bf16 *__restrict__ out,
                                                         __bf16 *__restrict__ out_lo, int nb, int dil) {
    const int lane = threadIdx.x & 63;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tileno = xcd_block();
    const int tiles_per_row = kNetG / 32;
    if (tileno >= nb * kNetG * tiles_per_row) return;  // uniform over the workgroup
    const int b = tileno / (kNetG * tiles_per_row);
    const int rem = tileno - b * kNetG * tiles_per_row;
    const int y = rem / tiles_per_row;
    const int x0 = (rem - y * tiles_per_row) * 32;
    const int r = lane & 31, hk = lane >> 5;
    const size_t img = (size_t)b * kNetG * kNetG * kNetC;
    f32x16 acc = {};
    // every load before the first product: left to itself the compiler takes 48
    // registers and a few loads at a time (one image 6.1 us a layer, two 9.2;
    // so 5.7 and 8.4, with three waves per SIMD at two images either way)
    bf16x8 av[3][2], al[3][2], bv[3][2], bl[3][2];
#pragma unroll
    for (int tt = 0; tt < 3; ++tt) {
        const int t = 3 * wib + tt;
        const int ys = wrapg(y + tap_dy(t, dil));
        const int xs = wrapg(x0 + r + tap_dx(t, dil));
        const size_t px = img + ((size_t)ys * kNetG + xs) * kNetC;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int wo = (r * 9 + t) * kNetC + 16 * h + 8 * hk;
            bv[tt][h] = load8(w + wo);
            av[tt][h] = load8(in + px + 16 * h + 8 * hk);
            al[tt][h] = load8(in_lo + px + 16 * h + 8 * hk);
            bl[tt][h] = load8(w_lo + wo);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int tt = 0; tt < 3; ++tt)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[tt][h], bv[tt][h], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[tt][h], bv[tt][h], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[tt][h], bl[tt][h], acc, 0, 0, 0);
        }
    __shared__ float part[2][16][64];
    if (wib > 0)
#pragma unroll
        for (int j = 0; j < 16; ++j) part[wib - 1][j][lane] = acc[j];
    __syncthreads();
    if (wib > 0) return;
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] += part[s][j][lane];
    const size_t o = (((size_t)b * kNetG + y) * kNetG + x0) * kNetC;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const int row = 8 * (j / 4) + 4 * hk + (j % 4);  // pixel within the tile
        const __bf16 hi = (__bf16)acc[j];
        out[o + (size_t)row * kNetC + r] = hi;
        out_lo[o + (size_t)row * kNetC + r] = (__bf16)(acc[j] - (float)hi);
    }
}

// Larger batches.  Reading every tap of every 32-pixel tile through the L1, and
// the layer's 36 KB of weights again for each tile, is what bounds such a
// product (72 KB of L1 reads for 54 MFMAs), so here a wavefront keeps all the
// weights in registers (36 fragments, 144 registers) and a workgroup of four
// (one 32-pixel tile each) walks rows of the image that are `dil` apart: the
// three rows an output row needs lie in a ring of four in LDS, each read from
// memory once per walk, the next one on its way during this row's products.
// A row's 16-byte chunks are swizzled (chunk c of pixel x at place
// c ^ (x / 4) % 4), so that any 16 consecutive pixels' chunks lie in 16
// different bank groups.  The weights are the MFMA's first operand, so a lane
// ends with channels of one pixel and, after one swap between the wave's
// halves, writes them as 16-byte stores.
// PAIR: activations and weights are (hi, lo) pairs; else single BF16.
// Walks of `seg` rows: workgroup = (image, row class y % dil, segment).
// Measured, 64 images in pairs: 206 -> 64 us a layer (4.2 TB/s of the 268 MB it
// reads and writes, 0.9 PFLOP/s of MFMAs: busy a third of the launch, the LDS a
// seventh; half of the waves' time goes waiting to issue, an output row being 54
// dependent MFMAs on one accumulator, two waves to a SIMD); a training step of 32 images, whose
// eight launches averaged 67.5 us: 36 us forward, 16 us for a gradient.
namespace {
constexpr int kRowBytes = kNetG * kNetC * 2;  // one row of one plane: 8 KB
__device__ __forceinline__ unsigned pack2(__bf16 a, __bf16 b) {
    return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}
// registers j = 0 .. 15 of a tile as BF16: 16 bytes at channel 8 hk and 16 at
// channel 16 + 8 hk of this lane's pixel
__device__ __forceinline__ void store_pixel(__bf16 *px, int hk, const __bf16 (&v)[16]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const auto s0 = __builtin_amdgcn_permlane32_swap(pack2(v[8 * q], v[8 * q + 1]), pack2(v[8 * q + 4], v[8 * q + 5]),
                                                         false, false);
        const auto s1 = __builtin_amdgcn_permlane32_swap(pack2(v[8 * q + 2], v[8 * q + 3]),
                                                         pack2(v[8 * q + 6], v[8 * q + 7]), false, false);
        uint4 o;
        o.x = s0[0];
        o.y = s1[0];
        o.z = s0[1];
        o.w = s1[1];
        *reinterpret_cast<uint4 *>(px + 16 * q + 8 * hk) = o;
    }
}
}  // namespace

template <bool PAIR>
__global__ __launch_bounds__(256, 2) void k_conv32(const __bf16 *__restrict__ in, const __bf16 *__restrict__ in_lo,
                                                   const __bf16 *__restrict__ w, const __bf16 *__restrict__ w_lo,
                                                   __bf16 *__restrict__ out, __bf16 *__restrict__ out_lo, int dil,
                                                   int seg) {
    constexpr int PL = PAIR ? 2 : 1;  // planes
    __shared__ __attribute__((aligned(16))) unsigned char lds[4][PL][kRowBytes];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chain = kNetG / dil, segs = chain / seg;
    int q = xcd_block();
    const int i0 = (q % segs) * seg;
    q /= segs;
    const int y0 = q % dil, b = q / dil;
    const size_t img = (size_t)b * kNetG * kNetG * kNetC;
    const int r = lane & 31, hk = lane >> 5, x0 = 32 * wib;
    auto row_y = [&](int i) { return y0 + dil * ((i0 + i) & (chain - 1)); };  // row i of the walk (i >= -1)

    bf16x8 wf[9][2], wl[PAIR ? 9 : 1][2];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int wo = (r * 9 + t) * kNetC + 16 * h + 8 * hk;
            wf[t][h] = load8(w + wo);
            if constexpr (PAIR) wl[t][h] = load8(w_lo + wo);
        }
    // a row: 512 chunks of 16 bytes a plane, two per thread, to their swizzled places
    bf16x8 st[PL][2];
    auto fetch = [&](int i) {
        const size_t o = img + (size_t)row_y(i) * kNetG * kNetC;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            st[0][k] = load8(in + o + 8 * (tid + 256 * k));
            if constexpr (PAIR) st[1][k] = load8(in_lo + o + 8 * (tid + 256 * k));
        }
    };
    auto put = [&](int slot) {
#pragma unroll
        for (int p = 0; p < PL; ++p)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int c = tid + 256 * k, x = c >> 2;
                *reinterpret_cast<bf16x8 *>(&lds[slot][p][64 * x + 16 * ((c ^ (x >> 2)) & 3)]) = st[p][k];
            }
    };
#pragma unroll
    for (int i = -1; i < 2; ++i) {
        fetch(i);
        put(i + 1);
    }
    // byte places of this lane's chunk (channels 16 h + 8 hk ..) for the three column shifts
    int at[3][2];
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
        const int x = wrapg(x0 + r + (kx - 1) * dil);
#pragma unroll
        for (int h = 0; h < 2; ++h) at[kx][h] = 64 * x + 16 * ((2 * h + hk) ^ ((x >> 2) & 3));
    }
    __syncthreads();
    for (int i = 0; i < seg; ++i) {
        if (i + 1 < seg) fetch(i + 2);
        f32x16 acc = {};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const unsigned char *row = lds[(i + t / 3) & 3][0];  // walk row i - 1 + t / 3
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const unsigned char *p = row + at[t % 3][h];
                const bf16x8 av = *reinterpret_cast<const bf16x8 *>(p);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[t][h], av, acc, 0, 0, 0);
                if constexpr (PAIR) {
                    const bf16x8 al = *reinterpret_cast<const bf16x8 *>(p + kRowBytes);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[t][h], al, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl[t][h], av, acc, 0, 0, 0);
                }
            }
        }
        const size_t o = img + ((size_t)row_y(i) * kNetG + x0 + r) * kNetC;
        __bf16 hi[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) hi[j] = (__bf16)acc[j];
        store_pixel(out + o, hk, hi);
        if constexpr (PAIR) {
            __bf16 lo[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) lo[j] = (__bf16)(acc[j] - (float)hi[j]);
            store_pixel(out_lo + o, hk, lo);
        }
        // the slot of walk row i - 2, last read two rows ago
        if (i + 1 < seg) put((i + 3) & 3);
        __syncthreads();
    }
}

template __global__ void k_conv32<true>(const __bf16 *, const __bf16 *, const __bf16 *, const __bf16 *, __bf16 *,
                                        __bf16 *, int, int);
template __global__ void k_conv32<false>(const __bf16 *, const __bf16 *, const __bf16 *, const __bf16 *, __bf16 *,
                                         __bf16 *, int, int);

// Weight gradient of a 32 -> 32 layer:
//   dw[co][tap][ci] = sum_{b, y, x} g[b][y][x][co] * in[b][y + dy][x + dx][ci]
// K runs over pixels, the strided dimension of the pixel-major layout, so rows
// are transposed once as they enter LDS ([channel][pixel], pixel pairs packed
// into words) and serve all nine taps from there: a workgroup of four
// wavefronts walks rows `dil` apart as k_conv32 does, input rows in a ring of
// four with 16 wrapped columns on either side (the largest dilation here),
// gradient rows in a ring of two.  A wavefront takes 32 pixels of the row, two
// steps of 16, against the nine taps' shifted columns: 18 MFMAs into nine
// accumulators.  A channel's row of pixels is an odd number of 16-byte units
// long, so an operand's 16-byte reads lie in 16 different bank groups.  The
// four wavefronts' sums meet in LDS; per workgroup 9 x 32 x 32 partial sums.
// (The transposition used to be redone per tap, by two-byte LDS stores.
// Measured, 32 images: 77 -> 22 us a layer with dilation 8 or 16, 26 with 4 and
// 30 with 2, whose shifted reads are 8 and 4 bytes wide.)
// ALIGN: alignment of a shifted 16-byte read, min(16, 2 dil).
namespace {
constexpr int kPadX = 16;
constexpr int kInStride = kNetG + 2 * kPadX + 8;  // 336 bytes, 21 units
constexpr int kGStride = kNetG + 8;               // 272 bytes, 17 units
template <int ALIGN>
__device__ __forceinline__ bf16x8 lds8(const __bf16 *p) {
    bf16x8 v;
    if constexpr (ALIGN >= 16) {
        v = *reinterpret_cast<const bf16x8 *>(p);
    } else if constexpr (ALIGN == 8) {
        const uint2 *q = reinterpret_cast<const uint2 *>(p);
        const uint2 u0 = q[0], u1 = q[1];
        v = __builtin_bit_cast(bf16x8, uint4{u0.x, u0.y, u1.x, u1.y});
    } else {
        const unsigned *q = reinterpret_cast<const unsigned *>(p);
        v = __builtin_bit_cast(bf16x8, uint4{q[0], q[1], q[2], q[3]});
    }
    return v;
}
}  // namespace

template <int ALIGN>
__global__ __launch_bounds__(256, 2) void k_conv32_wgrad(const __bf16 *__restrict__ g, const __bf16 *__restrict__ in,
                                                         float *__restrict__ part, int dil, int seg) {
    constexpr int kInBytes = 4 * kNetC * kInStride * 2, kGBytes = 2 * kNetC * kGStride * 2;
    constexpr int kRed = 3 * 16 * 64;  // floats of one wavefront's three taps
    static_assert(4 * kRed * 4 <= kInBytes + kGBytes, "the final sums reuse the rows' space");
    __shared__ __attribute__((aligned(16))) unsigned char lds[kInBytes + kGBytes];
    __bf16 *tin = reinterpret_cast<__bf16 *>(lds);                // [4][32][kInStride]
    __bf16 *tg = reinterpret_cast<__bf16 *>(lds + kInBytes);      // [2][32][kGStride]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wib = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int chain = kNetG / dil, segs = chain / seg;
    const int blk = xcd_block();
    int q = blk;
    const int i0 = (q % segs) * seg;
    q /= segs;
    const int y0 = q % dil, b = q / dil;
    const size_t img = (size_t)b * kNetG * kNetG * kNetC;
    auto row_at = [&](int i) { return img + (size_t)(y0 + dil * ((i0 + i) & (chain - 1))) * kNetG * kNetC; };
    // loader roles: pixels 2 pp, 2 pp + 1, channels c8 .. c8 + 7
    const int pp = tid >> 2, c8 = 8 * (tid & 3);
    bf16x8 vi[2], vg[2];
    auto fetch = [&](const __bf16 *src, int i, bf16x8 (&v)[2]) {
        const __bf16 *p = src + row_at(i) + (size_t)(2 * pp) * kNetC + c8;
        v[0] = load8(p);
        v[1] = load8(p + kNetC);
    };
    auto put_in = [&](int slot) {
        unsigned *t = reinterpret_cast<unsigned *>(tin + slot * kNetC * kInStride);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const unsigned u = pack2(vi[0][k], vi[1][k]);
            unsigned *r = t + (c8 + k) * (kInStride / 2) + kPadX / 2 + pp;
            r[0] = u;
            if (pp < kPadX / 2) r[kNetG / 2] = u;                 // columns 128 .. 143
            if (pp >= (kNetG - kPadX) / 2) r[-(kNetG / 2)] = u;   // columns -16 .. -1
        }
    };
    auto put_g = [&](int slot) {
        unsigned *t = reinterpret_cast<unsigned *>(tg + slot * kNetC * kGStride);
#pragma unroll
        for (int k = 0; k < 8; ++k) t[(c8 + k) * (kGStride / 2) + pp] = pack2(vg[0][k], vg[1][k]);
    };
    for (int i = -1; i < 2; ++i) {
        fetch(in, i, vi);
        put_in(i + 1);
    }
    fetch(g, 0, vg);
    put_g(0);
    const int r = lane & 31, hk = lane >> 5;  // operand lane roles
    f32x16 acc[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) acc[t] = f32x16{};
    __syncthreads();
    for (int i = 0; i < seg; ++i) {
        if (i + 1 < seg) {
            fetch(in, i + 2, vi);
            fetch(g, i + 1, vg);
        }
        const __bf16 *gr = tg + ((i & 1) * kNetC + r) * kGStride + 32 * wib + 8 * hk;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const bf16x8 av = lds8<16>(gr + 16 * h);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const __bf16 *ir = tin + (((i + t / 3) & 3) * kNetC + r) * kInStride + kPadX + 32 * wib + 8 * hk +
                                   16 * h + (t % 3 - 1) * dil;
                const bf16x8 bv = t % 3 == 1 ? lds8<16>(ir) : lds8<ALIGN>(ir);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[t], 0, 0, 0);
            }
        }
        if (i + 1 < seg) {
            put_in((i + 3) & 3);  // the slot of walk row i - 2, last read two rows ago
            put_g((i + 1) & 1);   // the slot of gradient row i - 1
        }
        __syncthreads();
    }
    float *red = reinterpret_cast<float *>(lds);
    float *o = part + (size_t)blk * 9 * kNetC * kNetC;
#pragma unroll
    for (int t0 = 0; t0 < 9; t0 += 3) {
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) red[wib * kRed + (16 * t + j) * 64 + lane] = acc[t0 + t][j];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kRed / 256; ++k) {
            const int idx = tid + 256 * k;
            const int l = idx & 63, j = (idx >> 6) & 15, t = idx >> 10;
            const float s = ((red[idx] + red[kRed + idx]) + red[2 * kRed + idx]) + red[3 * kRed + idx];
            const int co = 8 * (j / 4) + 4 * (l >> 5) + (j % 4);
            o[((size_t)co * 9 + t0 + t) * kNetC + (l & 31)] = s;
        }
        __syncthreads();
    }
}
template __global__ void k_conv32_wgrad<4>(const __bf16 *, const __bf16 *, float *, int, int);
template __global__ void k_conv32_wgrad<8>(const __bf16 *, const __bf16 *, float *, int, int);
template __global__ void k_conv32_wgrad<16>(const __bf16 *, const __bf16 *, float *, int, int);

// Partial sums, first stage, in a fixed order: out[grp][i] = sum of partials
// k = grp, grp + kSumGroups, ... (grid: x over i, y over the groups, whose
// stride in `out` is that of the whole parameter vector).
__global__ __launch_bounds__(256) void k_sum_partials(const float *__restrict__ part, int count, int len,
                                                      float *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int grp = blockIdx.y;
    if (i >= len) return;
    float s = 0.f;
#pragma unroll 8
    for (int k = grp; k < count; k += kSumGroups) s += part[(size_t)k * len + i];
    out[(size_t)grp * kNetParams + i] = s;
}

namespace {
// Parameter i as the layers read it: a BF16 (hi, lo) pair, and for the 32 -> 32
// layers the transposed, tap-flipped copy wt[ci][tap][co] = w[co][8 - tap][ci]
// (the input gradient of a layer is the same convolution with those weights).
__device__ __forceinline__ void store_weight(int i, float a, __bf16 *w16, __bf16 *w16lo, __bf16 *wt16) {
    const __bf16 h = (__bf16)a;
    w16[i] = h;
    w16lo[i] = (__bf16)(a - (float)h);
    const int q = i - kW0;
    if (q >= 0 && q < 4 * kWmid) {
        const int l = q / kWmid, r = q - l * kWmid;
        const int co = r / (9 * kNetC), t = (r / kNetC) % 9, ci = r % kNetC;
        wt16[l * kWmid + (ci * 9 + (8 - t)) * kNetC + co] = h;
    }
}
}  // namespace

// Parameters set from outside.
__global__ void k_to_bf16(const float *__restrict__ a, __bf16 *__restrict__ w16, __bf16 *__restrict__ w16lo,
                          __bf16 *__restrict__ wt16, int count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) store_weight(i, a[i], w16, w16lo, wt16);
}

// End of a backward pass, every parameter at once: the groups' sums into the
// gradient; the loss (workgroup 0) from k_mse's partial sums; and, ADAM, the
// optimizer's step on the FP32 master weights with the copies the layers read.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_finish(const float *__restrict__ groups, float *__restrict__ grad,
                                                const double *__restrict__ lpart, int pixels,
                                                float *__restrict__ loss, float *__restrict__ w, float *__restrict__ m,
                                                float *__restrict__ v, __bf16 *__restrict__ w16,
                                                __bf16 *__restrict__ w16lo, __bf16 *__restrict__ wt16, float lr,
                                                float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < kNetParams) {
        float gi = 0.f;
#pragma unroll 16
        for (int k = 0; k < kSumGroups; ++k) gi += groups[(size_t)k * kNetParams + i];
        grad[i] = gi;
        if constexpr (ADAM) {
            const float mi = b1 * m[i] + (1.f - b1) * gi;
            const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
            m[i] = mi;
            v[i] = vi;
            const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
            w[i] = wi;
            store_weight(i, wi, w16, w16lo, wt16);
        }
    }
    if (blockIdx.x == 0) {
        static_assert(kLossBlocks == 256, "one partial sum per thread");
        __shared__ double red[4];
        double s = lpart[threadIdx.x];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
        __syncthreads();
        if (threadIdx.x == 0) *loss = (float)((((red[0] + red[1]) + red[2]) + red[3]) / pixels);
    }
}
template __global__ void k_finish<false>(const float *, float *, const double *, int, float *, float *, float *,
                                         float *, __bf16 *, __bf16 *, __bf16 *, float, float, float, float, float,
                                         float);
template __global__ void k_finish<true>(const float *, float *, const double *, int, float *, float *, float *, float *,
                                        __bf16 *, __bf16 *, __bf16 *, float, float, float, float, float, float);

// The 1-channel layers move 32 channels of BF16 per pixel for a few hundred
// operations: bound by memory once their accesses are whole cache lines.  Four
// neighbouring lanes share a pixel, eight channels (16 bytes) each, so that a
// wavefront's load or store covers 16 pixels without a gap; a thread keeps its
// channels' 72 weights in registers over `per` pixels (a workgroup: 64 x per).

// First layer (1 -> 32): FP32 input and weights, the output as a BF16 (hi, lo)
// pair.  (64 images: 55 -> 39 us.)
__global__ __launch_bounds__(256) void k_conv_in(const float *__restrict__ x, const float *__restrict__ w1,
                                                 __bf16 *__restrict__ out, __bf16 *__restrict__ out_lo, int per,
                                                 int dil) {
    const int c8 = 8 * (threadIdx.x & 3);
    float w[8][9];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int t = 0; t < 9; ++t) w[k][t] = w1[(c8 + k) * 9 + t];
    const int q0 = blockIdx.x * 64 * per + (threadIdx.x >> 2);
    for (int i = 0; i < per; ++i) {
        const int q = q0 + 64 * i;
        const int b = q / (kNetG * kNetG), rem = q - b * kNetG * kNetG, y = rem / kNetG, xx = rem % kNetG;
        float v[9];
#pragma unroll
        for (int t = 0; t < 9; ++t)
            v[t] = x[((size_t)b * kNetG + wrapg(y + tap_dy(t, dil))) * kNetG + wrapg(xx + tap_dx(t, dil))];
        bf16x8 h8, l8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < 9; ++t) s += w[k][t] * v[t];
            const __bf16 hi = (__bf16)s;
            h8[k] = hi;
            l8[k] = (__bf16)(s - (float)hi);
        }
        *reinterpret_cast<bf16x8 *>(out + (size_t)q * kNetC + c8) = h8;
        *reinterpret_cast<bf16x8 *>(out_lo + (size_t)q * kNetC + c8) = l8;
    }
}

// Last layer (32 -> 1): (hi + lo) activations, FP32 weights and output.  Rows
// 32 apart need only each other (four rows, circular), so a workgroup reads
// four of them once, as FP32 sums hi + lo in LDS, and makes their 512 outputs,
// OUT = 2 per thread, or half of them (OUT = 1, two workgroups to a class);
// the sum runs over tap, then channel.  A pixel's eight
// 16-byte chunks are swizzled (chunk c of pixel x at c ^ (x / 2) % 8: any 16
// consecutive pixels' chunks lie in 16 different bank groups).
// (64 images: 82 -> 37 us.)
template <int OUT>
__global__ __launch_bounds__(256, 2) void k_conv_out(const __bf16 *__restrict__ in, const __bf16 *__restrict__ in_lo,
                                                     const float *__restrict__ w6, float *__restrict__ y) {
    constexpr int D = 1 << (kNetLayers - 1);
    static_assert(kNetG / D == 4, "four rows a class");
    __shared__ __attribute__((aligned(16))) float act[4][kNetG * kNetC];
    const int tid = threadIdx.x;
    const int blk = xcd_block();
    const int half = OUT == 1 ? blk & 1 : 0, cls = OUT == 1 ? blk >> 1 : blk;
    const int b = cls / D, y0 = cls % D;
    auto place = [](int x, int c) { return x * kNetC + 4 * ((c ^ (x >> 1)) & 7); };
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const size_t o = ((size_t)b * kNetG + y0 + D * row) * kNetG * kNetC;
        bf16x8 h[2], l[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            h[k] = load8(in + o + 8 * (tid + 256 * k));
            l[k] = load8(in_lo + o + 8 * (tid + 256 * k));
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int q = tid + 256 * k, x = q >> 2, c = 2 * (q & 3);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                float4 v;
                v.x = (float)h[k][4 * e + 0] + (float)l[k][4 * e + 0];
                v.y = (float)h[k][4 * e + 1] + (float)l[k][4 * e + 1];
                v.z = (float)h[k][4 * e + 2] + (float)l[k][4 * e + 2];
                v.w = (float)h[k][4 * e + 3] + (float)l[k][4 * e + 3];
                *reinterpret_cast<float4 *>(&act[row][place(x, c + e)]) = v;
            }
        }
    }
    __syncthreads();
    const int x = tid & (kNetG - 1), r0 = (tid >> 7) + 2 * half;  // row r0 of the class (and r0 + 2)
    float s[OUT] = {};
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        const int xs = wrapg(x + tap_dx(t, D));
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int at = place(xs, c);
#pragma unroll
            for (int k = 0; k < OUT; ++k) {
                const float4 v = *reinterpret_cast<const float4 *>(&act[(r0 + 2 * k + t / 3 + 3) & 3][at]);
                const float *wt = w6 + t * kNetC + 4 * c;
                s[k] += wt[0] * v.x;
                s[k] += wt[1] * v.y;
                s[k] += wt[2] * v.z;
                s[k] += wt[3] * v.w;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < OUT; ++k) y[((size_t)b * kNetG + y0 + D * (r0 + 2 * k)) * kNetG + x] = s[k];
}
template __global__ void k_conv_out<1>(const __bf16 *, const __bf16 *, const float *, float *);
template __global__ void k_conv_out<2>(const __bf16 *, const __bf16 *, const float *, float *);

// Input gradient of the last layer: g[b][p][ci] = sum_tap w6[tap][ci] * dy[b][p - off(tap)].
// (32 images: 19 -> 16 us.)
__global__ __launch_bounds__(256) void k_conv_out_bwd(const float *__restrict__ dy, const float *__restrict__ w6,
                                                      __bf16 *__restrict__ g, int per, int dil) {
    const int c8 = 8 * (threadIdx.x & 3);
    float w[9][8];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int k = 0; k < 8; ++k) w[t][k] = (float)(__bf16)w6[t * kNetC + c8 + k];
    const int q0 = blockIdx.x * 64 * per + (threadIdx.x >> 2);
    for (int i = 0; i < per; ++i) {
        const int q = q0 + 64 * i;
        const int b = q / (kNetG * kNetG), rem = q - b * kNetG * kNetG, yy = rem / kNetG, xx = rem % kNetG;
        float d[9];
#pragma unroll
        for (int t = 0; t < 9; ++t)
            d[t] = (float)(__bf16)dy[((size_t)b * kNetG + wrapg(yy - tap_dy(t, dil))) * kNetG + wrapg(xx - tap_dx(t, dil))];
        bf16x8 g8;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float s = 0.f;
#pragma unroll
            for (int t = 0; t < 9; ++t) s += w[t][k] * d[t];
            g8[k] = (__bf16)s;
        }
        *reinterpret_cast<bf16x8 *>(g + (size_t)q * kNetC + c8) = g8;
    }
}

// Weight gradients of the 1-channel layers, per-block partials:
//   LAST = false (first layer): part[blk][co][tap] = sum_p g[p][co] * x[p + off(tap)]
//   LAST = true  (last layer):  part[blk][tap][ci] = sum_p in[p][ci] * dy[p - off(tap)]
// (in = act + act_lo, the activation pair; dy rounded to BF16).  Each pixel's
// activations are read once, against the nine scalars around it; lanes as in
// the layers above.  A thread's 8 x 9 sums meet by rotations within the rows
// of 16 lanes, then the workgroup's 16 rows in LDS.
// (32 images, per layer: 52 -> 16 us.)
template <bool LAST>
__global__ __launch_bounds__(256) void k_wgrad_small(const __bf16 *__restrict__ act, const __bf16 *__restrict__ act_lo,
                                                     const float *__restrict__ vec, float *__restrict__ part,
                                                     int chunk, int dil) {
    __shared__ float red[16][4][73];
    const int c = threadIdx.x & 3, row16 = threadIdx.x >> 4;
    const int p0 = blockIdx.x * chunk + (threadIdx.x >> 2);
    float acc[8][9];
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int t = 0; t < 9; ++t) acc[k][t] = 0.f;
    for (int i = 0; i < chunk; i += 64) {
        const int q = p0 + i;
        const int b = q / (kNetG * kNetG), rem = q - b * kNetG * kNetG, yy = rem / kNetG, xx = rem % kNetG;
        const bf16x8 h8 = load8(act + (size_t)q * kNetC + 8 * c);
        float v[9], u[8];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int ys = wrapg(LAST ? yy - tap_dy(t, dil) : yy + tap_dy(t, dil));
            const int xs = wrapg(LAST ? xx - tap_dx(t, dil) : xx + tap_dx(t, dil));
            v[t] = vec[((size_t)b * kNetG + ys) * kNetG + xs];
            if constexpr (LAST) v[t] = (float)(__bf16)v[t];
        }
        if constexpr (LAST) {
            const bf16x8 l8 = load8(act_lo + (size_t)q * kNetC + 8 * c);
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = (float)h8[k] + (float)l8[k];
        } else {
#pragma unroll
            for (int k = 0; k < 8; ++k) u[k] = (float)h8[k];
        }
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[k][t] += u[k] * v[t];
    }
    // lanes 4, 8, 12 further on in the row hold the same channels
    auto rot = [](float a, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a), decltype(ctrl)::value, 0xf, 0xf, true));
    };
#pragma unroll
    for (int k = 0; k < 8; ++k)
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            float a = acc[k][t];
            a += rot(a, std::integral_constant<int, 0x124>{});
            a += rot(a, std::integral_constant<int, 0x128>{});
            if ((threadIdx.x & 15) < 4) red[row16][c][9 * k + t] = a;
        }
    __syncthreads();
    for (int i = threadIdx.x; i < 9 * kNetC; i += 256) {
        const int ch = i / 9, t = i - 9 * ch;
        float s = 0.f;
        for (int k = 0; k < 16; ++k) s += red[k][ch >> 3][9 * (ch & 7) + t];
        part[(size_t)blockIdx.x * 9 * kNetC + (LAST ? t * kNetC + ch : ch * 9 + t)] = s;
    }
}
template __global__ void k_wgrad_small<false>(const __bf16 *, const __bf16 *, const float *, float *, int, int);
template __global__ void k_wgrad_small<true>(const __bf16 *, const __bf16 *, const float *, float *, int, int);

// Mean squared error: dy = 2 (y - t) / count, and per-block partial sums of (y - t)^2.
__global__ __launch_bounds__(256) void k_mse(const float *__restrict__ y, const float *__restrict__ t,
                                             float *__restrict__ dy, double *__restrict__ part, int count) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < count; i += gridDim.x * 256) {
        const float e = y[i] - t[i];
        dy[i] = 2.f * e / (float)count;
        s += (double)e * (double)e;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Scale of a right-hand side: its RMS over the valid cells, sqrt(sum f^2 / n^2);
// 1 when no statistics are given.
__device__ __forceinline__ double rms_scale(const double *sumsq, int n) {
    if (!sumsq) return 1.0;
    const double s = sqrt(*sumsq / ((double)n * (double)n));
    return s > 0.0 ? s : 1.0;
}

// Encoder: out[y][x] = mean of the r x r block of f (FP64, ghosted, pitch) / scale,
// with r = n / G (a mean of four-cell means is this block mean).  A workgroup
// covers 64 blocks of one block row; its four waves take every fourth fine
// row, each lane summing its block's r columns (a wave reads 64 r contiguous
// values per row), and the four row sums meet in LDS.
__global__ __launch_bounds__(256) void k_encode(const double *__restrict__ f, long pitch, int n,
                                                const double *__restrict__ sumsq, float *__restrict__ out) {
    __shared__ double red[4][64];
    const int xi = threadIdx.x & 63, ph = threadIdx.x >> 6;
    const int x = blockIdx.x * 64 + xi, y = blockIdx.y;
    const int r = n / kNetG;
    double s = 0.0;
    for (int j = ph; j < r; j += 4) {
        const double *row = f + (long)(y * r + j + 1) * pitch + 1 + (long)x * r;
        for (int i = 0; i < r; ++i) s += row[i];
    }
    red[ph][xi] = s;
    __syncthreads();
    if (ph == 0) {
        const double t = (red[0][xi] + red[1][xi]) + (red[2][xi] + red[3][xi]);
        out[y * kNetG + x] = (float)(t / ((double)r * r) / rms_scale(sumsq, n));
    }
}

// Decoder, first step: the network output on the G x G grid in physical units
// (times the RMS of f when given, and the square of the domain side), then
// `iters` red-black Gauss-Seidel iterations of the periodic Poisson problem
// Lap u = f on that grid against the encoded right-hand side (x times the
// RMS), red ((row + column) even) first, which remove the grid-scale noise of
// the network output.  FP32 (it is only a guess).  One workgroup of 1024
// threads, each keeping a 4 x 4 block in registers and exchanging only block
// edges through LDS.  Output: G x G FP64 (no ghosts).
// LDS layout of the G x G grid: one pad word after every 4 columns and rows of
// kRelaxRow words, so that the 64 lanes of a wave (32 blocks across, 2 block
// rows down) reading or writing one edge cell each hit 64 different banks
// (a plain 128-word row put them on far fewer).
constexpr int kRelaxB = 4;
constexpr int kRelaxRow = 168;
__device__ __forceinline__ int relax_at(int r, int c) { return r * kRelaxRow + c + (c >> 2); }

__global__ __launch_bounds__(kRelaxThreads) void k_coarse_relax(const float *__restrict__ y,
                                                                const float *__restrict__ x,
                                                                const double *__restrict__ sumsq, int nfine,
                                                                double length, int iters,
                                                                double *__restrict__ out) {
    constexpr int B = kRelaxB, NB = kNetG / B, m = kNetG - 1;  // 32 x 32 blocks of 4 x 4 cells
    static_assert(NB * NB <= kRelaxThreads, "one block per thread");
    __shared__ float u[kNetG * kRelaxRow];
    const int t = threadIdx.x;
    const double rms = rms_scale(sumsq, nfine);
    const float su = (float)(rms * length * length);
    const float h2 = (float)(length * length / ((double)kNetG * kNetG));
    for (int q = t; q < kNetG * kNetG; q += kRelaxThreads) u[relax_at(q / kNetG, q % kNetG)] = y[q] * su;
    __syncthreads();
    if (t < NB * NB) {
        const int R0 = B * (t / NB), C0 = B * (t % NB);  // block origin (even: block parity = global parity)
        float v[B][B], hf[B][B];
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) {
                v[i][j] = u[relax_at(R0 + i, C0 + j)];
                hf[i][j] = -h2 * (float)(x[(R0 + i) * kNetG + C0 + j] * rms);
            }
        const int up = (R0 - 1) & m, dn = (R0 + B) & m, lf = (C0 - 1) & m, rt = (C0 + B) & m;
        for (int it = 0; it < iters; ++it) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                // updates of colour c: neighbours inside the block from registers,
                // outside from the edges the neighbouring blocks published
#pragma unroll
                for (int i = 0; i < B; ++i)
#pragma unroll
                    for (int j = 0; j < B; ++j) {
                        if (((i + j) & 1) != c) continue;
                        const float w = j > 0 ? v[i][j - 1] : u[relax_at(R0 + i, lf)];
                        const float e = j < B - 1 ? v[i][j + 1] : u[relax_at(R0 + i, rt)];
                        const float nn = i > 0 ? v[i - 1][j] : u[relax_at(up, C0 + j)];
                        const float ss = i < B - 1 ? v[i + 1][j] : u[relax_at(dn, C0 + j)];
                        v[i][j] = 0.25f * (hf[i][j] + ((e + w) + (ss + nn)));  // u = (sum - h^2 f) / 4
                    }
                // publish the updated edge cells
#pragma unroll
                for (int i = 0; i < B; ++i)
#pragma unroll
                    for (int j = 0; j < B; ++j) {
                        if (((i + j) & 1) != c) continue;
                        if (i == 0 || i == B - 1 || j == 0 || j == B - 1) u[relax_at(R0 + i, C0 + j)] = v[i][j];
                    }
                __syncthreads();
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i)
#pragma unroll
            for (int j = 0; j < B; ++j) u[relax_at(R0 + i, C0 + j)] = v[i][j];
    } else {
        for (int it = 0; it < 2 * iters; ++it) __syncthreads();  // keep the barrier count of the relaxing threads
    }
    __syncthreads();
    for (int q = t; q < kNetG * kNetG; q += kRelaxThreads) out[q] = (double)u[relax_at(q / kNetG, q % kNetG)];
}

// Decoder step: one multigrid prolongation (centred slopes, no xy term,
// periodic) from an nc x nc FP64 grid (no ghosts) to 2nc x 2nc, written plain
// (out_pitch = 2nc) or into the valid cells of a ghosted field.
__global__ void k_decode_step(const double *__restrict__ c, int nc, double *__restrict__ fine, long out_pitch,
                              int ghosted) {
    const int n = 2 * nc;
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n * n) return;
    const int y = q / n, x = q % n, I = x >> 1, J = y >> 1, m = nc - 1;
    auto at = [&](int jj, int ii) -> double { return c[(jj & m) * nc + (ii & m)]; };
    const double e = at(J, I);
    const double mx = 0.5 * (at(J, I + 1) - at(J, I - 1)), my = 0.5 * (at(J + 1, I) - at(J - 1, I));
    const double dx = (x & 1) ? 0.25 : -0.25, dy = (y & 1) ? 0.25 : -0.25;
    const double v = (e + dx * mx) + dy * my;
    if (ghosted) fine[(long)(y + 1) * out_pitch + x + 1] = v;
    else fine[q] = v;
}


}  // namespace ccmg
