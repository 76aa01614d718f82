// Instantiations of the fold kernel for a workgroup per tile: one rank read and copied to others.  See fold_once.hpp.
#include "fold_once.hpp"

namespace blink {

namespace {
template <int K, int M, int F>
OnceKernel kernel() {
    return {reinterpret_cast<const void*>(blink_once_copy<K, M, F, once_copy_columns(M)>), fill_once_copy<K, F>, K,
            sizeof(void*) * K + 4 * (F + 1 + F * K / 8)};
}
template <int F>
OnceKernel pick(int k, int m) {
    if (k <= 8) {
        switch (m) {
#define BLINK_CASE(M) case M: return kernel<8, M, F>();
            BLINK_CASE(1) BLINK_CASE(2) BLINK_CASE(3) BLINK_CASE(4) BLINK_CASE(5) BLINK_CASE(6) BLINK_CASE(7)
#undef BLINK_CASE
            default: return {};
        }
    }
    switch (m) {
#define BLINK_CASE(M) case M: return kernel<16, M, F>();
        BLINK_CASE(1) BLINK_CASE(2) BLINK_CASE(3) BLINK_CASE(4) BLINK_CASE(5) BLINK_CASE(6) BLINK_CASE(7) BLINK_CASE(8)
        BLINK_CASE(9) BLINK_CASE(10) BLINK_CASE(11) BLINK_CASE(12) BLINK_CASE(13) BLINK_CASE(14) BLINK_CASE(15)
#undef BLINK_CASE
        default: return {};
    }
}
}  // namespace

OnceKernel once_copy(int k, int m, bool many) { return many ? pick<kOnceMostFlows>(k, m) : pick<kOnceFewFlows>(k, m); }

}  // namespace blink
