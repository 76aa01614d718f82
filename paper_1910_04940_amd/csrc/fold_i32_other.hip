// Instantiations of the fold kernel: products, minima and maxima of int32 elements.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_other(int n, bool all, bool half) {
    if (!all) return pick_fold_one<unsigned, false>(n);
    return half ? pick_fold_half<unsigned, false>(n) : pick_fold_all<unsigned, false, kFoldKeep>(n);
}

}  // namespace blink
