// Instantiation of the kernel for stages that wait for one another: int32 elements.  See
// kernel.hpp.
#include "kernel.hpp"

namespace blink {

KernelFn kernel_i32() { return blink_consume<unsigned>; }

}  // namespace blink
