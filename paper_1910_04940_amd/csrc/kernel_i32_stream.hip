// Instantiation of the kernel for stages that wait for one another: int32 elements,
// 32 columns per lane.  See kernel.hpp.
#include "kernel.hpp"

namespace blink {

KernelFn kernel_i32_stream() { return blink_consume<unsigned, kColumnsStream>; }

}  // namespace blink
