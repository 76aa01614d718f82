// Instantiations of the fold kernel: fp32 elements, partial sums written on the way.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_mid(int n, bool all, FoldTile tile, bool sum) {
    return sum ? pick_fold<float, true, true>(n, all, tile) : pick_fold<float, false, true>(n, all, tile);
}

}  // namespace blink
