// Instantiations of the fold kernel: sums of int32 elements.  See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_i32_sum(int n, bool all, FoldTile tile, bool stream) {
    return stream && all && tile == FoldTile::kDrawn ? pick_fold_drawn<unsigned, true, kFoldStream>(n) : pick_fold<unsigned, true>(n, all, tile);
}

}  // namespace blink
