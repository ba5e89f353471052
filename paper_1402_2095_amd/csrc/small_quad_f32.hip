// FP32 instantiations of the small-system kernel with M in registers.
#include "small_quad.hpp"

namespace fth {
template <>
int launch_small_quad<float>(const StepArgs<float>& a, const SmallTraj<float>& tj, int K, void* stream) {
    return launch_small_quad_impl<float>(a, tj, K, stream);
}
}  // namespace fth
