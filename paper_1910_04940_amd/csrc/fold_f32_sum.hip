// Instantiations of the fold kernel: sums of fp32 elements.  See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_sum(int n, bool all, bool stream, bool half) {
    if (!all) return pick_fold_one<float, true>(n);
    if (half) return pick_fold_half<float, true>(n);
    return stream ? pick_fold_all<float, true, kFoldStream>(n) : pick_fold_all<float, true, kFoldKeep>(n);
}

}  // namespace blink
