// Readout: means and block standard errors of every estimate, formed on the
// device from the FP64 accumulators and written straight into pinned host
// memory, one chunk of estimates per launch (the host copies a chunk out while
// the next one is formed).
//
// Bound by the host link and by the host's copy into the caller's arrays: two
// doubles leave the device per estimate instead of three, from pinned memory,
// and the host divides and takes no roots.  Measured (copies of the accumulators and a host loop before):
// 1001024 estimates 6760 -> 580 us, 263168 estimates 1790 -> 175 us, 127 estimates 45 -> 20 us a read.
#include <hip/hip_runtime.h>

#include "fth_internal.h"

namespace fth {
namespace dev {

// The arithmetic is the one of the block averages, in FP64 without contraction:
// est = (s1 + blk) / samples; var = (sum of squared block means - (sum)^2 / nb) / (nb - 1).
__global__ __launch_bounds__(256) void read_estimates_kernel(const double* __restrict__ acc, int64_t no, int64_t k0,
                                                             int64_t count, ReadScale rs, double* __restrict__ est,
                                                             double* __restrict__ se) {
    const int64_t x = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (x >= count) return;
    const int64_t k = k0 + x;
    const double s1 = acc[no + k];
    est[x] = rs.samples > 0.0 ? (s1 + acc[k]) / rs.samples : __builtin_nan("");
    double e = __builtin_inf();
    if (rs.blocks >= 2.0) {
        const double s2 = acc[2 * no + k];
        const double sb = s1 * rs.per_block, sbb = s2 * rs.per_block * rs.per_block;
        const double var = (sbb - sb * sb / rs.blocks) / (rs.blocks - 1.0);
        e = sqrt((var < 0.0 ? 0.0 : var) / rs.blocks);
    }
    se[x] = e;
}

}  // namespace dev

int launch_read_estimates(const double* acc, int64_t no, int64_t k0, int64_t count, const ReadScale& rs, double* est,
                          double* se, void* stream) {
    if (count <= 0) return 0;
    hipLaunchKernelGGL(dev::read_estimates_kernel, dim3(unsigned((count + 255) / 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), acc, no, k0, count, rs, est, se);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace fth
