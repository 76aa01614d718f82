// Instantiations of the fold kernel: sums of int32 elements.  See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_sum(int n, bool all, bool stream, bool half) {
    if (!all) return pick_fold_one<unsigned, true>(n);
    if (half) return pick_fold_half<unsigned, true>(n);
    return stream ? pick_fold_all<unsigned, true, kFoldStream>(n) : pick_fold_all<unsigned, true, kFoldKeep>(n);
}

}  // namespace blink
