// Instantiations of the fold kernel: one rank read and copied to others.  See fold.hpp.
#include "fold.hpp"

namespace blink {

FoldFn fold_copy(int policy) {
    return policy == kFoldSpread   ? blink_fold<unsigned, 1, false, true, kFoldSpread, false, false>
           : policy == kFoldStream ? blink_fold<unsigned, 1, false, true, kFoldStream, false, false>
                                   : blink_fold<unsigned, 1, false, true, kFoldKeep, false, false>;
}

}  // namespace blink
