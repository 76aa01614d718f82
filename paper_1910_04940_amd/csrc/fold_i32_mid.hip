// Instantiations of the fold kernel: int32 elements, partial sums written on the way.
// See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_mid(int n, bool all, FoldTile tile, bool sum) {
    return sum ? pick_fold<unsigned, true, true>(n, all, tile) : pick_fold<unsigned, false, true>(n, all, tile);
}

}  // namespace blink
