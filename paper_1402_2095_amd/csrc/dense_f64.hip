// FP64 dense force GEMM (plain FP64 form) and the FP64 dense epilogue.
#include "dense.hpp"

namespace fth {

namespace {
template <int RT>
void launch_f64(const DenseGemmArgs& g, int64_t grid, hipStream_t s) {
    if (g.krem == 0)
        hipLaunchKernelGGL((dev::gemm_f64_kernel<RT, true>), dim3(unsigned(grid)), dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL((dev::gemm_f64_kernel<RT, false>), dim3(unsigned(grid)), dim3(256), 0, s, g);
}
}  // namespace

int launch_gemm_f64(const DenseGemmArgs& g0, void* stream) {
    DenseGemmArgs g = g0;
    if (g.rows_pad % 64 != 0 || g.n > g.rows_pad || g.ksplit < 1 || (g.n + 15) / 16 < g.ksplit) return -3;
    g.kq = int32_t((g.n + 15) / 16 / g.ksplit);
    g.krem = int32_t((g.n + 15) / 16 % g.ksplit);
    g.kslice = int64_t(g.kq) * 16;
    const int64_t grid = ((g.n + 63) / 64) * g.ksplit;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    switch (g.R) {
        case 16: launch_f64<1>(g, grid, s); break;
        case 32: launch_f64<2>(g, grid, s); break;
        case 64: launch_f64<4>(g, grid, s); break;
        case 128: launch_f64<8>(g, grid, s); break;
        default: return -2;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <>
int launch_dense_epilogue<double>(const StepArgs<double>& a, const StepLaunch& L, int k, void* stream) {
    return launch_dense_epilogue_impl<double>(a, L, k, stream);
}

}  // namespace fth
