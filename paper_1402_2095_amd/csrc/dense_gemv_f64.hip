// FP64 instantiations of the few-replica dense step.
#include "dense_gemv.hpp"

namespace fth {
template <>
int launch_dense_gemv<double>(const StepArgs<double>& a, const double* M, int64_t ld, int k, void* stream) {
    return launch_dense_gemv_impl<double>(a, M, ld, k, stream);
}
template <>
int launch_gemv_force<double>(const double* M, int64_t ld, int64_t N, int R, const double* q, double* part, void* stream) {
    return launch_gemv_force_impl<double>(M, ld, N, R, q, part, stream);
}
}  // namespace fth
