// Split-BF16x3 dense force GEMM, the bf16 split kernels and the FP32 dense
// epilogue instantiations.
#include "dense.hpp"

namespace fth {
namespace dev {

// `given` rows of M (row-major, n columns, rounded to FP32) -> bf16 hi/lo parts of
// `rows` rows in the GEMM's tiled layout (mt: the first one's row block), zero past
// the given rows and column n; one 16-byte output unit (8 consecutive k of one row,
// one part) per iteration.
template <typename Src>
__global__ void split_bf16_tiled_kernel(const Src* __restrict__ m, int64_t given, int64_t n, u32x4* __restrict__ mt,
                                        int64_t rows, int64_t P) {
    const int64_t total = rows * P / 4;  // rows x P elements x 2 parts x 2 bytes / 16 bytes
    const int64_t KB = P / 64;
    for (int64_t o = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; o < total; o += int64_t(gridDim.x) * blockDim.x) {
        const int l = int(o & 63), u = int((o >> 6) & 7), w = int((o >> 9) & 3);
        const int64_t tile = o >> 11;
        const int64_t row = (tile / KB) * 128 + 32 * w + 16 * (u >> 2) + (l & 15);
        const int64_t k = (tile % KB) * 64 + 16 * (l >> 4) + 8 * (u & 1);
        const bool lo = ((u >> 1) & 1) != 0;
        uint32_t word[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t two = 0;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int64_t kk = k + 2 * t + e;
                const float x = row < given && kk < n ? float(m[row * n + kk]) : 0.0f;
                const uint16_t h = bf16_bits(x);
                const uint16_t part = lo ? bf16_bits(x - bf16_value(h)) : h;
                two |= uint32_t(part) << (16 * e);
            }
            word[t] = two;
        }
        mt[o] = u32x4{word[0], word[1], word[2], word[3]};
    }
}

// `given` rows of M (row-major, n columns) -> [rows][ld] in the state precision, zero
// past the given rows and column n.
template <typename Src, typename Real>
__global__ void pad_dense_kernel(const Src* __restrict__ m, int64_t given, int64_t n, Real* __restrict__ out,
                                 int64_t rows, int64_t ld) {
    const int64_t total = rows * ld;
    for (int64_t o = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; o < total; o += int64_t(gridDim.x) * blockDim.x) {
        const int64_t i = o / ld, j = o % ld;
        out[o] = i < given && j < n ? Real(m[i * n + j]) : Real(0);
    }
}

__global__ void qt_from_q_kernel(const float* __restrict__ q, uint16_t* __restrict__ qt, int64_t N, int32_t R) {
    const int64_t total = N * R;
    for (int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; t < total; t += int64_t(gridDim.x) * blockDim.x)
        put_qt(qt, t / R, t % R, R, q[t]);
}

}  // namespace dev

int launch_gemm_bf16x3(const DenseGemmArgs& g0, void* stream) {
    DenseGemmArgs g = g0;
    if (g.rows_pad % 128 != 0 || g.n > g.rows_pad || g.ksplit < 1 || (g.n + 63) / 64 < g.ksplit) return -3;
    g.kq = int32_t((g.n + 63) / 64 / g.ksplit);
    g.krem = int32_t((g.n + 63) / 64 % g.ksplit);
    const int64_t grid = ((g.n + 127) / 128) * g.ksplit;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    switch (g.R) {
        case 16: hipLaunchKernelGGL(dev::gemm_bf16x3_kernel<1>, dim3(unsigned(grid)), dim3(256), 0, s, g); break;
        case 32: hipLaunchKernelGGL(dev::gemm_bf16x3_kernel<2>, dim3(unsigned(grid)), dim3(256), 0, s, g); break;
        case 64: hipLaunchKernelGGL(dev::gemm_bf16x3_kernel<4>, dim3(unsigned(grid)), dim3(256), 0, s, g); break;
        case 128: hipLaunchKernelGGL(dev::gemm_bf16x3_kernel<8>, dim3(unsigned(grid)), dim3(256), 0, s, g); break;
        default: return -2;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_split_bf16_tiled(const void* m, bool m_f64, int64_t given, int64_t n, void* mt, int64_t rows, int64_t P,
                            void* stream) {
    if (P % 128 != 0 || rows % 128 != 0 || given < 0 || given > rows || rows > P || n < 1 || n > P) return -3;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    dev::u32x4* out = static_cast<dev::u32x4*>(mt);
    if (m_f64)
        hipLaunchKernelGGL(dev::split_bf16_tiled_kernel<double>, dim3(4096), dim3(256), 0, s,
                           static_cast<const double*>(m), given, n, out, rows, P);
    else
        hipLaunchKernelGGL(dev::split_bf16_tiled_kernel<float>, dim3(4096), dim3(256), 0, s, static_cast<const float*>(m),
                           given, n, out, rows, P);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

namespace {
template <typename Src, typename Real>
void pad_dense(const void* m, int64_t given, int64_t n, void* out, int64_t rows, int64_t ld, hipStream_t s) {
    hipLaunchKernelGGL((dev::pad_dense_kernel<Src, Real>), dim3(4096), dim3(256), 0, s, static_cast<const Src*>(m), given,
                       n, static_cast<Real*>(out), rows, ld);
}
}  // namespace

int launch_pad_dense(const void* m, bool m_f64, int64_t given, int64_t n, void* out, bool out_f64, int64_t rows,
                     int64_t ld, void* stream) {
    if (given < 0 || rows < given || ld < n || n < 1) return -3;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (m_f64 && out_f64)
        pad_dense<double, double>(m, given, n, out, rows, ld, s);
    else if (m_f64)
        pad_dense<double, float>(m, given, n, out, rows, ld, s);
    else if (out_f64)
        pad_dense<float, double>(m, given, n, out, rows, ld, s);
    else
        pad_dense<float, float>(m, given, n, out, rows, ld, s);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_qt_from_q(const float* q, uint16_t* qt, int64_t N, int64_t rows_pad, int32_t R, void* stream) {
    (void)rows_pad;
    hipLaunchKernelGGL(dev::qt_from_q_kernel, dim3(2048), dim3(256), 0, static_cast<hipStream_t>(stream), q, qt, N, R);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <>
int launch_dense_epilogue<float>(const StepArgs<float>& a, const StepLaunch& L, int k, void* stream) {
    return launch_dense_epilogue_impl<float>(a, L, k, stream);
}

}  // namespace fth
