// Instantiations of the fold kernel: one rank read and copied to others.  See fold.hpp.
#include "fold.hpp"
#include "state.hpp"

namespace blink {

static_assert(kInlineLevels == kInlineFlows, "the launcher and the handle agree on what a launch carries");

FoldFn fold_copy(int policy) {
    return policy == kFoldSpread   ? blink_fold<unsigned, 1, false, true, kFoldSpread, false, false>
           : policy == kFoldStream ? blink_fold<unsigned, 1, false, true, kFoldStream, false, false>
                                   : blink_fold<unsigned, 1, false, true, kFoldKeep, false, false>;
}

}  // namespace blink
