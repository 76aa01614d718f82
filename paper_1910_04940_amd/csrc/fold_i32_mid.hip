// Instantiations of the fold kernel: int32 elements, partial sums written on the way.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_mid(int n, bool all, bool sum, bool half) {
    if (!all) return sum ? pick_fold_one<unsigned, true, true>(n) : pick_fold_one<unsigned, false, true>(n);
    if (half) return sum ? pick_fold_half<unsigned, true, true>(n) : pick_fold_half<unsigned, false, true>(n);
    return sum ? pick_fold_all<unsigned, true, kFoldKeep, true>(n) : pick_fold_all<unsigned, false, kFoldKeep, true>(n);
}

}  // namespace blink
