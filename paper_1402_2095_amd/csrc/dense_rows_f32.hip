// FP32 (split-BF16x3) instantiations of the one-launch dense step.
#include "dense_rows.hpp"

namespace fth {
template <>
int launch_dense_rows<float>(const StepArgs<float>& a, const DenseRowsArgs& g, int ct, int k, void* stream) {
    return launch_dense_rows_impl<float>(a, g, ct, k, stream);
}
}  // namespace fth
