// Bands of 8 rows held in registers whole (block_impl.h), double.
#include "block_impl.h"

namespace ccmg {
template hipError_t dispatch_block<double, 8>(const MarchArgs<double> &, int, bool, bool, int, int, hipStream_t,
                                           int *);
}  // namespace ccmg
