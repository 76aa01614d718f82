// Instantiations of the fold kernel: sums of fp32 elements.  See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_f32_sum(int n, bool all, FoldTile tile, bool stream) {
    return stream && all && tile == FoldTile::kDrawn ? pick_fold_drawn<float, true, kFoldStream>(n) : pick_fold<float, true>(n, all, tile);
}

}  // namespace blink
