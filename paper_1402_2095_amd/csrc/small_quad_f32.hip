// FP32 instantiations of the small-system kernel with M in registers.
#include "small_quad.hpp"

namespace fth {
template <>
int launch_small_quad<float>(const StepArgs<float>& a, const SmallTraj<float>& tj, int64_t n0, int K, void* stream) {
    return launch_small_quad_impl<float>(a, tj, n0, K, stream);
}
}  // namespace fth
