// FP32 instantiations of the few-replica dense step.
#include "dense_gemv.hpp"

namespace fth {
template <>
int launch_dense_gemv<float>(const StepArgs<float>& a, const float* M, int64_t ld, int k, void* stream) {
    return launch_dense_gemv_impl<float>(a, M, ld, k, stream);
}
template <>
int launch_gemv_force<float>(const float* M, int64_t ld, int64_t N, int R, const float* q, float* part, void* stream) {
    return launch_gemv_force_impl<float>(M, ld, N, R, q, part, stream);
}
}  // namespace fth
