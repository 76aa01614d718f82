// Instantiations of the fold kernel: products, minima and maxima of int32 elements.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_other(int n, bool all, FoldTile tile) { return pick_fold<unsigned, false>(n, all, tile); }

}  // namespace blink
