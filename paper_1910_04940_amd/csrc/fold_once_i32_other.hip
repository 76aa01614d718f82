// Instantiations of the fold kernel for a workgroup per tile: products, minima and maxima of int32 elements.  See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

OnceKernel once_i32_other(int n, bool all, bool half, bool many) { return pick_once<unsigned, false, false>(n, all, half, many); }

}  // namespace blink
