// Instantiation of the kernel for stages that wait for one another: fp32 elements,
// 32 columns per lane.  See kernel.hpp.
#include "kernel.hpp"

namespace blink {

KernelFn kernel_f32_stream() { return blink_consume<float, kColumnsStream>; }

}  // namespace blink
