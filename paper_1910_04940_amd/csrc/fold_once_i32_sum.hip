// Instantiations of the fold kernel for a workgroup per tile: sums of int32 elements.  See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

OnceKernel once_i32_sum(int n, bool half, bool many) { return pick_once<unsigned, true>(n, half, many); }

}  // namespace blink
