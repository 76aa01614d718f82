// Instantiation of the kernel for stages that wait for one another: int32 elements,
// 16 columns per lane.  See kernel.hpp.
#include "kernel.hpp"

namespace blink {

KernelFn kernel_i32_many() { return blink_consume<unsigned, kColumnsMany>; }

}  // namespace blink
