// march.hip -- host entry of the row-march kernels: picks the variant with the
// requested number of fused red-black iterations (see march_impl.h).
#include <type_traits>

#include "internal.h"

namespace ccmg {

template <typename T>
hipError_t launch_march(const MarchArgs<T> &a, int nu, bool load_phi, bool prolong, int post,
                        MarchShape shape, hipStream_t s, int *nt) {
    if (shape.ty == 0) shape = MarchShape{8, 1};
    // Bands of 8 and 16 rows are held in registers whole where that variant
    // exists, for every level: measured per launch against the row march in
    // bands of 8 to 128 rows (and against 32 x 32 LDS blocks) it was faster on
    // all levels of 64^2 to 2048^2 cells, by 3 us to a factor of two.
    if ((shape.ty == 8 || shape.ty == 16) && shape.wpb >= 1 && shape.wpb <= 4) {
        const hipError_t e = shape.ty == 8 ? dispatch_block<T, 8>(a, nu, load_phi, prolong, post, shape.wpb, s, nt)
                                           : dispatch_block<T, 16>(a, nu, load_phi, prolong, post, shape.wpb, s, nt);
        if (e != hipErrorNotSupported) return e;
    }
    if (post == POST_FUSED) {
        if (nu == 4 && load_phi && prolong && shape.ty >= 2 && !(shape.ty & 1) && shape.wpb >= 1 && shape.wpb <= 4)
            return dispatch_fused(a, shape, s, nt);
        return hipErrorInvalidValue;
    }
    if (post == POST_CNPRE) {
        if constexpr (std::is_same<T, double>::value) {
            if (nu == 2 && load_phi && !prolong && shape.ty >= 2 && !(shape.ty & 1) && shape.wpb >= 1 &&
                shape.wpb <= 4)
                return dispatch_cnpre(a, shape, s, nt);
        }
        return hipErrorInvalidValue;
    }
    if (post == POST_FUSED0) {
        if constexpr (std::is_same<T, double>::value) {
            if (nu == 6 && !load_phi && prolong && shape.ty >= 2 && !(shape.ty & 1) && shape.wpb >= 1 &&
                shape.wpb <= 4)
                return dispatch_fused0(a, shape, s, nt);
        }
        return hipErrorInvalidValue;
    }
    if (post == POST_VISIT) {
        if (nu == 4 && !load_phi && prolong && shape.ty >= 2 && !(shape.ty & 1) && shape.wpb >= 1 && shape.wpb <= 4)
            return dispatch_visit(a, shape, s, nt);
        return hipErrorInvalidValue;
    }
    if (shape.ty < 2 || (shape.ty & 1) || shape.wpb < 1 || shape.wpb > 4) return hipErrorInvalidValue;
    switch (nu) {
        case 0: return dispatch_nu<T, 0>(a, load_phi, prolong, post, shape, s, nt);
        case 1: return dispatch_nu<T, 1>(a, load_phi, prolong, post, shape, s, nt);
        case 2: return dispatch_nu<T, 2>(a, load_phi, prolong, post, shape, s, nt);
    }
    return hipErrorInvalidValue;
}

template hipError_t launch_march<double>(const MarchArgs<double> &, int, bool, bool, int, MarchShape,
                                         hipStream_t, int *);
template hipError_t launch_march<float>(const MarchArgs<float> &, int, bool, bool, int, MarchShape,
                                        hipStream_t, int *);

}  // namespace ccmg
