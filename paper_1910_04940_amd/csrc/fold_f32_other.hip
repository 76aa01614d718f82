// Instantiations of the fold kernel: products, minima and maxima of fp32 elements.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_other(int n, bool all, bool half) {
    if (!all) return pick_fold_one<float, false>(n);
    return half ? pick_fold_half<float, false>(n) : pick_fold_all<float, false, kFoldKeep>(n);
}

}  // namespace blink
