// Instantiations of the fold kernel for a workgroup per tile: fp32 elements, partial sums written on the way.
// See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

OnceKernel once_f32_mid(int n, bool all, bool half, bool many, bool sum) {
    return sum ? pick_once<float, true, true>(n, all, half, many) : pick_once<float, false, true>(n, all, half, many);
}

}  // namespace blink
