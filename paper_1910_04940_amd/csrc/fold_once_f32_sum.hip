// Instantiations of the fold kernel for a workgroup per tile: sums of fp32 elements.  See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

OnceKernel once_f32_sum(int n, bool all, bool half, bool many) { return pick_once<float, true, false>(n, all, half, many); }

}  // namespace blink
