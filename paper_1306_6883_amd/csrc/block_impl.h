// block_impl.h -- short bands of a level held in registers whole.
// (Included by the block_*.hip files, each of which instantiates a subset.)
//
// The row march (march_impl.h) walks a band a row at a time: right for the
// large levels, whose launches are bound by memory, but a level of 64^2 to
// 1024^2 cells has little to do per launch, and there the walk itself is the
// time: some twenty steps, each a chain of five or more dependent stages
// behind the loads of three rows ahead.  Here one wavefront takes the same
// 128 columns (two adjacent cells per lane) of a band of R = 8 or 16 rows and
// loads the band with its halo rows at once -- one round trip to memory --
// then runs each colour sweep over all rows (independent of each other, so
// the chain of a launch is its stages, not its rows times its stages), the
// region shrinking by one row a side per sweep.
// Per launch, FP64: a level's two launches 7.1 - 8.4 -> 4.3 - 5.7 us (64^2 to
// 512^2; some 2.5 us are the launch), the fused finest launch of 64^2 21.7 ->
// 9.8, of 256^2 18.3 -> 10.1 us; a V-cycle of 2048^2 with all its coarse levels
// so 150 -> 128 us.
//
// The arithmetic of a cell is the row march's, operation for operation, and
// what a tile writes does not depend on the tiling: the same bits.  Side rules:
// on a Dirichlet or Neumann x side by selects in the tiles that touch it, as
// there; on a y side the rows y = 0 and y = n - 1 sit at fixed places of a
// band or of its halo (R divides n), so only those need a select.
#pragma once
#include "cycle_end.h"
#include "march_impl.h"

#pragma clang fp contract(on)

namespace ccmg {

// Compile-time shape: rows and columns that the stages of a launch use up.
template <int NU, bool LOADPHI, bool PROLONG, int POST, int R>
struct BlockCfg {
    static constexpr bool FUSED = POST == POST_FUSED;
    static constexpr bool RES = POST != POST_NONE;
    static constexpr int LAST = 2 * NU + (RES ? 1 : 0);
    // from zero the first red sweep reads no neighbour
    static constexpr bool ZERO1 = !LOADPHI && !PROLONG && NU > 0;
    static constexpr int H = LAST - (ZERO1 ? 1 : 0);  // halo rows a side
    static constexpr int NR = R + 2 * H;
    // the same columns as the row march, so that its per-tile sums are the same
    static constexpr int HX = march_halo_x(NU, PROLONG, RES);
    static constexpr int OUTW = 128 - 2 * HX;
    // coarse rows J0 - 1 .. of the prolongation (J0: that of the first row)
    static constexpr int JF = -((H + 1) / 2);  // floor(-H / 2)
    static constexpr int NC = PROLONG ? (((R + H - 1) >> 1) - JF + 3) : 1;
};

// Sums of a tile: the restricted residual, the norm pair (sum r^2, sum phi),
// and f's statistics.
struct BlockSums {
    double v[7];
    enum { RC = 0, R2 = 1, PHI = 2, F = 3 };
};

// stop: the skip flag's value, loaded by the caller; looked at (and the tile
// left) once the tile's own loads are on their way.
template <typename T, int NU, bool LOADPHI, bool PROLONG, int POST, int R, bool XB>
__device__ __forceinline__ void block_tile(const MarchArgs<T> &a, const int strip, const int y0, const int stop,
                                           BlockSums &sums) {
    using C = BlockCfg<NU, LOADPHI, PROLONG, POST, R>;
    constexpr int NR = C::NR, H = C::H, NC = C::NC;
    const int lane = threadIdx.x & 63;
    const int n = a.n, nm = n - 1, nc = n >> 1;
    const bool px = a.bc[CCMG_XLO] == CCMG_BC_PERIODIC, py = a.bc[CCMG_YLO] == CCMG_BC_PERIODIC;
    const int xo0 = strip * C::OUTW, x0 = xo0 - C::HX + 2 * lane;
    const bool inx = px || (x0 >= 0 && x0 < n);
    const int xl = px ? (x0 & nm) : (inx ? x0 : 0);  // out-of-domain lanes read column 0
    const bool wedge = !px && x0 == 0, eedge = !px && x0 + 1 == nm;
    const bool outl = x0 >= xo0 && x0 < xo0 + C::OUTW && x0 >= 0 && x0 < n;
    // the domain's first / last row is the band's, or the next band's (whose
    // rows reach into this band's halo where that is taller than R)
    const bool ylo = !py && y0 == 0, yhi = !py && y0 + R == n;
    const bool ylo1 = !py && y0 == R, yhi1 = !py && y0 + 2 * R == n;
    // row slot k is the domain's first / last row (false for all but two slots each)
    auto first_row = [&](auto kc) -> bool {
        constexpr int k = decltype(kc)::value;
        if constexpr (k == H) return ylo;
        else if constexpr (k == H - R) return ylo1;
        else return false;
    };
    auto last_row = [&](auto kc) -> bool {
        constexpr int k = decltype(kc)::value;
        if constexpr (k == H + R - 1) return yhi;
        else if constexpr (k == H + 2 * R - 1) return yhi1;
        else return false;
    };

    // 1. every load of the tile, then the skip flag and the mean shifts
    T P0[NR], P1[NR], F0[NR], F1[NR], Cw[NC];
    const double psub64 = (LOADPHI && a.phi_shift) ? *a.phi_shift : 0.0;
    const int lo = 1 + xl;
    static_for<0, NR>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        int y = y0 - H + k;
        y = py ? (y & nm) : min(max(y, 0), nm);
        if constexpr (NU > 0 || C::RES) {
            // a row outside every sweep's region has no right-hand side to read
            if constexpr (C::ZERO1 || (k > 0 && k < NR - 1)) {
                const T *fr = a.f + row_off(y + 1, a.pf);
                F0[k] = fr[lo];
                F1[k] = fr[lo + 1];
            } else {
                F0[k] = F1[k] = T(0);
            }
        }
        if constexpr (LOADPHI) {
            const T *pr = a.phi_in + row_off(y + 1, a.pin);
            P0[k] = pr[lo];
            P1[k] = pr[lo + 1];
        } else {
            P0[k] = P1[k] = T(0);
        }
    });
    const int I = x0 >> 1;
    if constexpr (PROLONG) {
        const int Il = px ? (I & (nc - 1)) : min(max(I, 0), nc - 1);
        static_for<0, NC>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            int J = (y0 >> 1) + C::JF - 1 + q;
            J = py ? (J & (nc - 1)) : min(max(J, 0), nc - 1);
            Cw[q] = (a.ec + row_off(J + 1, a.pc))[1 + Il];
        });
    }
    T fsub = T(0);
    if (a.fmean_part) {
        const int cnt = a.fmean_count_ptr ? *a.fmean_count_ptr : a.fmean_count;
        fsub = T(sum_partials(a.fmean_part, cnt) / ((double)n * (double)n));
    }
    if (stop) return;
    const T psub = T(psub64);
    const T sxl = a.bc[CCMG_XLO] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    const T sxh = a.bc[CCMG_XHI] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    const T syl = a.bc[CCMG_YLO] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    const T syh = a.bc[CCMG_YHI] == CCMG_BC_DIRICHLET ? T(-1) : T(1);
    const T cc = a.cc, invd = a.invd;
    if (a.fmean_part) {
        static_for<0, NR>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if constexpr (NU > 0 || C::RES) {
                F0[k] -= fsub;
                F1[k] -= fsub;
            }
        });
    }
    if constexpr (LOADPHI) {
        if (a.phi_shift) {
            static_for<0, NR>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                P0[k] -= psub;
                P1[k] -= psub;
            });
        }
    }

    // 2. prolongation of the coarse correction
    if constexpr (PROLONG) {
        const bool cwedge = !px && I == 0, ceedge = !px && I == nc - 1;
        static_for<0, NC - 2>([&](auto qc) {  // coarse row q + 1: fine rows 2 (JF + q), + 1 of the band
            constexpr int q = decltype(qc)::value;
            constexpr int ke = 2 * (C::JF + q) + H;  // row slot of the even fine row
            const T c0 = Cw[q + 1];
            T cm = Cw[q], cp = Cw[q + 2];
            // the coarse row is the domain's first / last where the fine row is
            if (first_row(std::integral_constant<int, ke>{})) cm = syl * c0;
            if (last_row(std::integral_constant<int, ke + 1>{})) cp = syh * c0;
            T ew = from_left(c0), ee = from_right(c0);
            if constexpr (XB) {
                if (cwedge) ew = sxl * c0;
                if (ceedge) ee = sxh * c0;
            }
            const T mx = T(0.5) * (ee - ew);
            const T my = T(0.5) * (cp - cm);
            static_for<0, 2>([&](auto hc) {
                constexpr int h = decltype(hc)::value, k = ke + h;
                if constexpr (k >= 0 && k < NR) {
                    const T dy = h ? T(0.25) : T(-0.25);
                    P0[k] = P0[k] + ((c0 + T(-0.25) * mx) + dy * my);
                    P1[k] = P1[k] + ((c0 + T(0.25) * mx) + dy * my);
                }
            });
        });
    }

    // 3. colour sweeps: sweep s (odd red, even black) on the rows it can still do
    auto sweep = [&](auto sc) {
        constexpr int s = decltype(sc)::value;
        constexpr int m = s - (C::ZERO1 ? 1 : 0);  // rows used up a side
        static_for<m, NR - m>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            constexpr int par = (k - H) & 1;  // parity of the row (y0 is even)
            constexpr int col = (s & 1) ? par : 1 - par;
            if constexpr (C::ZERO1 && s == 1) {  // every neighbour is zero
                if constexpr (col == 0) P0[k] = F0[k] * invd;
                else P1[k] = F1[k] * invd;
            } else if constexpr (col == 0) {
                const T self = P0[k];
                const T e = P1[k];
                T w = from_left(P1[k]);
                if constexpr (XB) {
                    if (wedge) w = sxl * self;
                }
                T nn = P0[k + 1], ss = P0[k - 1];
                if (last_row(kc)) nn = syh * self;
                if (first_row(kc)) ss = syl * self;
                P0[k] = (F0[k] + cc * (((e + w) + nn) + ss)) * invd;
            } else {
                const T self = P1[k];
                const T w = P0[k];
                T e = from_right(P0[k]);
                if constexpr (XB) {
                    if (eedge) e = sxh * self;
                }
                T nn = P1[k + 1], ss = P1[k - 1];
                if (last_row(kc)) nn = syh * self;
                if (first_row(kc)) ss = syl * self;
                P1[k] = (F1[k] + cc * (((e + w) + nn) + ss)) * invd;
            }
        });
    };
    // residual of output row slot k
    auto resid = [&](auto kc, T &r0, T &r1) {
        constexpr int k = decltype(kc)::value;
        const T p0 = P0[k], p1 = P1[k];
        T w0 = from_left(P1[k]);
        T e1 = from_right(P0[k]);
        if constexpr (XB) {
            if (wedge) w0 = sxl * p0;
            if (eedge) e1 = sxh * p1;
        }
        T n0 = P0[k + 1], n1 = P1[k + 1], s0 = P0[k - 1], s1 = P1[k - 1];
        if constexpr (k == H + R - 1) {
            if (yhi) {
                n0 = syh * p0;
                n1 = syh * p1;
            }
        }
        if constexpr (k == H) {
            if (ylo) {
                s0 = syl * p0;
                s1 = syl * p1;
            }
        }
        const T ih2 = a.ih2;
        const T lap0 = ((((p1 - p0) + (w0 - p0)) + (n0 - p0)) + (s0 - p0)) * ih2;
        const T lap1 = ((((e1 - p1) + (p0 - p1)) + (n1 - p1)) + (s1 - p1)) * ih2;
        r0 = F0[k] - (a.alpha * p0 - a.beta * lap0);
        r1 = F1[k] - (a.alpha * p1 - a.beta * lap1);
    };
    auto store = [&](T *dst, long pitch) {
        static_for<H, H + R>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (outl) {
                T *o = dst + row_off(y0 + k - H + 1, pitch);
                o[1 + x0] = P0[k];
                o[2 + x0] = P1[k];
            }
        });
    };
    // residual norm sums of the output rows
    auto norm = [&](double &s2, double &s1) {
        double q2 = 0.0, q1 = 0.0;
        static_for<H, H + R>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            T r0, r1;
            resid(kc, r0, r1);
            if (outl) {
                q2 += (double)r0 * (double)r0 + (double)r1 * (double)r1;
                q1 += (double)P0[k] + (double)P1[k];
            }
        });
        s2 = wave_sum(q2);
        s1 = wave_sum(q1);
    };

    // a solve's first launch: the residual norm of the guess as loaded, and f's statistics
    if constexpr (LOADPHI && !PROLONG && POST == POST_RESTRICT) {
        if (a.in_norm_part) norm(sums.v[BlockSums::R2], sums.v[BlockSums::PHI]);
    }
    if constexpr (!PROLONG && POST == POST_RESTRICT) {
        if (a.fstat_part) {
            double fs = 0.0, fa = 0.0, f2 = 0.0, fbad = 0.0;
            auto add = [&](double v) {
                if (!isfinite(v)) {
                    fbad += 1.0;
                } else {
                    fs += v;
                    fa += fabs(v);
                    f2 += v * v;
                }
            };
            if (outl) {
                static_for<H, H + R>([&](auto kc) {
                    add((double)F0[decltype(kc)::value]);
                    add((double)F1[decltype(kc)::value]);
                });
            }
            sums.v[BlockSums::F + 0] = wave_sum(fs);
            sums.v[BlockSums::F + 1] = wave_sum(fa);
            sums.v[BlockSums::F + 2] = wave_sum(f2);
            sums.v[BlockSums::F + 3] = wave_sum(fbad);
        }
    }

    if constexpr (C::FUSED) {
        static_for<1, 5>(sweep);
        if (a.partial_norm) {
            norm(sums.v[BlockSums::R2], sums.v[BlockSums::PHI]);
        }
        if (a.phi_mid) store(a.phi_mid, a.pmid);
        static_for<5, 2 * NU + 1>(sweep);
    } else {
        static_for<1, 2 * NU + 1>(sweep);
    }
    if (a.phi_out) store(a.phi_out, a.pout);
    if constexpr (POST == POST_NORM) norm(sums.v[BlockSums::R2], sums.v[BlockSums::PHI]);
    // 4. residual -> four-cell averages, and their sum
    if constexpr (POST == POST_RESTRICT || C::FUSED) {
        double acc = 0.0;
        static_for<0, R / 2>([&](auto jc) {
            constexpr int k = H + 2 * decltype(jc)::value;
            T r00, r01, r10, r11;
            resid(std::integral_constant<int, k>{}, r00, r01);
            resid(std::integral_constant<int, k + 1>{}, r10, r11);
            const T v = T(0.25) * (((r00 + r01) + r10) + r11);
            if (outl) {
                (a.aux + row_off(((y0 + k - H) >> 1) + 1, a.paux))[1 + (x0 >> 1)] = v;
                acc += (double)v;
            }
        });
        sums.v[BlockSums::RC] = wave_sum(acc);
    }
}

// A tile's sums are added up within the workgroup (wpb waves): every wave of
// the next level's launches adds all partial sums of the restricted residual
// on singular problems, a round trip to memory per 1024 of them.
// OCC: waves per SIMD to leave registers for.
template <typename T, int NU, bool LOADPHI, bool PROLONG, int POST, int R, int OCC>
__global__ __launch_bounds__(256, OCC) void k_block(const MarchArgs<T> a) {
    using C = BlockCfg<NU, LOADPHI, PROLONG, POST, R>;
    __shared__ double part[4][7];
    if constexpr (!LOADPHI && !PROLONG && POST == POST_RESTRICT) {
        // the last workgroup: the end of the cycle before, which nothing else in
        // this launch reads (a launch of its own took 4 us of every cycle)
        if (a.end.partial && blockIdx.x == gridDim.x - 1) {
            if (threadIdx.x < 64) cycle_end_one_wave(a.end);
            return;
        }
    }
    const int wpb = blockDim.x >> 6;
    const int wib = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // XCD-aware order, as in k_march: each XCD gets a contiguous run of tiles
    const int grp = (blockIdx.x & 7) * a.groups_per_xcd + (blockIdx.x >> 3);
    const int tile = grp * wpb + wib;
    const int stop = a.skip ? *a.skip : 0;
    BlockSums s{};
    if (tile < a.ntiles) {
        const int band = tile / a.strips, strip = tile - band * a.strips;
        const int X0 = strip * C::OUTW - C::HX;
        const bool xb = a.bc[CCMG_XLO] != CCMG_BC_PERIODIC && (X0 <= 0 || X0 + 128 >= a.n - 1);
        if (xb) block_tile<T, NU, LOADPHI, PROLONG, POST, R, true>(a, strip, band * R, stop, s);
        else block_tile<T, NU, LOADPHI, PROLONG, POST, R, false>(a, strip, band * R, stop, s);
    }
    if (stop) return;  // uniform
    if constexpr (C::RES) {
        if (wpb > 1) {
            if ((threadIdx.x & 63) == 0)
#pragma unroll
                for (int q = 0; q < 7; ++q) part[wib][q] = s.v[q];
            __syncthreads();
            if (threadIdx.x == 0)
                for (int w = 1; w < wpb; ++w)
#pragma unroll
                    for (int q = 0; q < 7; ++q) s.v[q] += part[w][q];
        }
        if (threadIdx.x == 0 && grp * wpb < a.ntiles) {
            const double r2 = s.v[BlockSums::R2], phi = s.v[BlockSums::PHI];
            auto pair = [&](double *p) {
                if (!p) return;
                p[2 * grp] = r2;
                p[2 * grp + 1] = phi;
            };
            if constexpr (POST == POST_NORM) {
                pair(a.partial);
            } else {
                a.partial[grp] = s.v[BlockSums::RC];
                if constexpr (C::FUSED) {
                    pair(a.partial_norm);
                } else if constexpr (!PROLONG) {
                    if constexpr (LOADPHI) pair(a.in_norm_part);
                    if (a.fstat_part)
#pragma unroll
                        for (int q = 0; q < 4; ++q) a.fstat_part[4 * grp + q] = s.v[BlockSums::F + q];
                }
            }
        }
    }
}

template <typename T, int NU, bool LOADPHI, bool PROLONG, int POST, int R, int OCC = 1>
static hipError_t go_block(const MarchArgs<T> &a0, int wpb, hipStream_t s, int *nt) {
    MarchArgs<T> a = a0;
    a.outw = BlockCfg<NU, LOADPHI, PROLONG, POST, R>::OUTW;
    a.ty = R;
    a.strips = (a.n + a.outw - 1) / a.outw;
    a.chunks = a.n / R;
    a.ntiles = a.strips * a.chunks;
    a.ety = R;
    a.echunks = 0;
    const int groups = (a.ntiles + wpb - 1) / wpb;
    if (nt) *nt = groups;
    a.groups_per_xcd = (groups + 7) / 8;
    const int extra = !LOADPHI && !PROLONG && POST == POST_RESTRICT && a.end.partial ? 1 : 0;
    hipLaunchKernelGGL((k_block<T, NU, LOADPHI, PROLONG, POST, R, OCC>), dim3(8 * a.groups_per_xcd + extra),
                       dim3(64 * wpb), 0, s, a);
    return hipGetLastError();
}

// The V(2,2) launches of a level in bands of R rows; hipErrorNotSupported for
// any other (the caller then runs the row march).
template <typename T, int R>
hipError_t dispatch_block(const MarchArgs<T> &a, int nu, bool load_phi, bool prolong, int post, int wpb,
                          hipStream_t s, int *nt) {
    if (a.count_out || !block_runs(a.n, nu, load_phi, prolong, post, MarchShape{R, 1}, sizeof(T) == 8))
        return hipErrorNotSupported;
    // (16 rows and the 18 halo rows of the fused launch do not fit the registers in FP64)
    if constexpr (R == 8 || sizeof(T) == 4) {
        if (post == POST_FUSED && nu == 4 && load_phi && prolong) {
            // FP64 needs 267 registers, one wave per SIMD.  From 1024^2 a launch
            // has more waves than SIMDs (1280 there): two per SIMD, at twenty
            // registers' spills, then take 67.8 - 71.1 us per cycle against
            // 72.6 - 73.2; at 512^2 (640 waves) 51.9 against 50.4.
            if constexpr (R == 8 && sizeof(T) == 8) {
                if (a.n >= 1024) return go_block<T, 4, true, true, POST_FUSED, R, 2>(a, wpb, s, nt);
            }
            return go_block<T, 4, true, true, POST_FUSED, R>(a, wpb, s, nt);
        }
    }
    if (nu != 2) return hipErrorNotSupported;
    if (!load_phi && !prolong && post == POST_RESTRICT) return go_block<T, 2, false, false, POST_RESTRICT, R>(a, wpb, s, nt);
    if (load_phi && !prolong && post == POST_RESTRICT) return go_block<T, 2, true, false, POST_RESTRICT, R>(a, wpb, s, nt);
    if (load_phi && prolong && post == POST_NONE) return go_block<T, 2, true, true, POST_NONE, R>(a, wpb, s, nt);
    if (load_phi && prolong && post == POST_NORM) return go_block<T, 2, true, true, POST_NORM, R>(a, wpb, s, nt);
    return hipErrorNotSupported;
}

}  // namespace ccmg
