// Instantiations of the fold kernel: fp32 elements, partial sums written on the way.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_mid(int n, bool all, bool sum, bool half) {
    if (!all) return sum ? pick_fold_one<float, true, true>(n) : pick_fold_one<float, false, true>(n);
    if (half) return sum ? pick_fold_half<float, true, true>(n) : pick_fold_half<float, false, true>(n);
    return sum ? pick_fold_all<float, true, kFoldKeep, true>(n) : pick_fold_all<float, false, kFoldKeep, true>(n);
}

}  // namespace blink
