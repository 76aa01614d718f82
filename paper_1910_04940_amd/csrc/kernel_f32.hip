// Instantiation of the kernel for stages that wait for one another: fp32 elements.  See
// kernel.hpp.
#include "kernel.hpp"

namespace blink {

KernelFn kernel_f32() { return blink_consume<float>; }

}  // namespace blink
