// FP64 instantiations of the small-system kernel with M in registers.
#include "small_quad.hpp"

namespace fth {
template <>
int launch_small_quad<double>(const StepArgs<double>& a, const SmallTraj<double>& tj, int64_t n0, int K, void* stream) {
    return launch_small_quad_impl<double>(a, tj, n0, K, stream);
}
}  // namespace fth
