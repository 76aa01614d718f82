// Instantiations of the fold kernel: one rank read and copied to others.  See fold.hpp.
#include "fold.hpp"

namespace blink {

namespace {
template <int POLICY, int U>
constexpr FoldFn kCopy = blink_fold<unsigned, 1, false, true, POLICY, U, false>;
}

FoldFn fold_copy(int policy, int columns) {
    if (policy == kFoldSpread) {
        switch (columns) {
            case 2: return kCopy<kFoldSpread, 2>;
            case 3: return kCopy<kFoldSpread, 3>;
            case 4: return kCopy<kFoldSpread, 4>;
            case 8: return kCopy<kFoldSpread, 8>;
            default: return nullptr;
        }
    }
    switch (columns) {   // to one rank
        case 4: return policy == kFoldKeep ? kCopy<kFoldKeep, 4> : nullptr;   // (what fits the cache is kept)
        case 16: return policy == kFoldStream ? kCopy<kFoldStream, 16> : kCopy<kFoldKeep, 16>;
        default: return nullptr;
    }
}

}  // namespace blink
