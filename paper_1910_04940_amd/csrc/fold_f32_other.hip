// Instantiations of the fold kernel: products, minima and maxima of fp32 elements.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_other(int n, bool all, FoldTile tile) { return pick_fold<float, false>(n, all, tile); }

}  // namespace blink
