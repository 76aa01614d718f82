// Instantiations of the fold kernel for a workgroup per tile: int32 elements, partial sums written on the way.
// See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

OnceKernel once_i32_mid(int n, bool all, bool half, bool many, bool sum) {
    return sum ? pick_once<unsigned, true, true>(n, all, half, many) : pick_once<unsigned, false, true>(n, all, half, many);
}

}  // namespace blink
