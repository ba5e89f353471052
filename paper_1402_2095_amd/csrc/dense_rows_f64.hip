// FP64 instantiations of the one-launch dense step.
#include "dense_rows.hpp"

namespace fth {
template <>
int launch_dense_rows<double>(const StepArgs<double>& a, const DenseRowsArgs& g, int ct, int k, void* stream) {
    return launch_dense_rows_impl<double>(a, g, ct, k, stream);
}
}  // namespace fth
