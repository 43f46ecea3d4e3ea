// Bands of 8 rows held in registers whole (block_impl.h), float.
#include "block_impl.h"

namespace ccmg {
template hipError_t dispatch_block<float, 8>(const MarchArgs<float> &, int, bool, bool, int, int, hipStream_t,
                                           int *);
}  // namespace ccmg
