// Dense step for few replicas (R in {1, 2, 4, 8}), one launch per step: the force
// F = -M q_n as R matrix-vector products and the row update of the same rows.
// With so few right-hand sides the work is one pass over M per step, bound by
// memory; the matrix cores' 16-column tiles would compute mostly zero columns, so
// the products use plain FMAs in the state precision.
//
// Layouts: M row-major Real [N][ld], ld = N rounded up to 4 with zero columns;
// q_n [ld][R] (the context's q buffers, zero rows past N).  Workgroup b owns rows
// ROWS b + (0 .. ROWS-1), and its four waves share the columns: lane l of wave w
// takes columns 256 w + 4 l .. + 3 of every 1024, loads 4 entries of each row (the
// next pass's while the current one's FMAs run) and keeps one partial sum per
// (row, replica).  The lanes' partials are added by halving exchanges, then the
// four waves' in wave order, so the result does not depend on scheduling.  A
// workgroup per 8 rows (a wave per 8 rows before) gives four times the waves:
// 6001 rows are 751 workgroups instead of 188, which left a quarter of the 256 CUs
// idle.
//
// Since a workgroup ends with the complete sums of its rows, it applies the row
// update itself.  The normals of the rows are drawn while the first pass's loads
// are in flight, one Philox block per lane across all four waves, and kept in LDS.
// Non-temporal loads of M measured slower wherever M fits the last-level cache
// (9000 rows, R = 1, FP64: 128 against 107 us).  A step, with the force and the row
// update as two launches before:
//   6001 rows  R = 1 FP32 28.8 -> 23.0 us, R = 8 FP32 66.7 -> 32.3, R = 1 FP64 74.8 -> 43.8
//   16384 rows R = 1 FP32 183.5 -> 181.7, R = 8 FP32 214.7 -> 183.3, R = 4 FP64 488 -> 382
// (1074 MB in 182 us is 5.9 TB/s; 144 MB in 23 us, from the last-level cache, 6.3).
#pragma once

#include "dense.hpp"

namespace fth {
namespace dev {

// Sum of each of the C values over the 64 lanes, C a power of two: the first
// exchanges halve the number of values a lane holds (lane distance 32, 16, ...),
// the remaining ones are a butterfly on the one value left.  Lane l ends with the
// sum of value gemv_value<C>(l).
template <typename Real, int C, int OFF>
__device__ __forceinline__ Real lanes_sum(Real (&v)[C], int lane) {
    if constexpr (OFF == 0) {
        return v[0];
    } else if constexpr (C == 1) {
        Real one[1] = {v[0] + __shfl_xor(v[0], OFF, 64)};
        return lanes_sum<Real, 1, OFF / 2>(one, lane);
    } else {
        Real half[C / 2];
        const bool up = (lane & OFF) != 0;
#pragma unroll
        for (int x = 0; x < C / 2; ++x) {
            const Real keep = up ? v[x + C / 2] : v[x];
            const Real give = up ? v[x] : v[x + C / 2];
            half[x] = keep + __shfl_xor(give, OFF, 64);
        }
        return lanes_sum<Real, C / 2, OFF / 2>(half, lane);
    }
}
// the value whose sum lane l holds: the bits of l from 32 down, most significant first
template <int C>
__device__ __forceinline__ int gemv_value(int lane) {
    int x = 0;
#pragma unroll
    for (int b = 32, s = C / 2; s >= 1; b >>= 1, s >>= 1) x |= (lane & b) ? s : 0;
    return x;
}

// Partial sums of the workgroup's rows: red[w][row * R + r] over wave w's columns.
// `between` runs once, after the first pass's loads are issued.  Every thread of
// the workgroup calls it; rows past N - 1 repeat row N - 1 (their sums are unused).
template <typename Real, int R, typename F>
__device__ __forceinline__ void gemv_partials(const Real* __restrict__ M, int64_t ld, int64_t N,
                                              const Real* __restrict__ q, int64_t row0,
                                              Real (&red)[4][gemv_rows(sizeof(Real) == 8, R) * R], F&& between) {
    constexpr int ROWS = gemv_rows(sizeof(Real) == 8, R), VW = 4;
    constexpr int PASS = 256 * VW;  // columns per pass of the workgroup
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const Real* mrow[ROWS];
#pragma unroll
    for (int rr = 0; rr < ROWS; ++rr) mrow[rr] = M + min(row0 + rr, N - 1) * ld;
    Real acc[ROWS * R];
#pragma unroll
    for (int x = 0; x < ROWS * R; ++x) acc[x] = Real(0);
    struct Pass {
        Vec<Real, 4> m[ROWS];
        Vec<Real, 4> q[R];
    };
    auto load = [&](Pass& p, int j) {
#pragma unroll
        for (int rr = 0; rr < ROWS; ++rr) p.m[rr] = load_vec<Real, 4>(mrow[rr] + j);
#pragma unroll
        for (int u = 0; u < R; ++u) p.q[u] = load_vec<Real, 4>(q + int64_t(j) * R + 4 * u);  // rows j .. j+3
    };
    auto use = [&](const Pass& p) {
#pragma unroll
        for (int rr = 0; rr < ROWS; ++rr)
#pragma unroll
            for (int c = 0; c < VW; ++c)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int e = c * R + r;  // element (j + c, r) of the lane's 4 R values
                    acc[rr * R + r] = fmaR(p.m[rr].v[c], p.q[e >> 2].v[e & 3], acc[rr * R + r]);
                }
    };
    const int n = int(ld);
    int j = (w * 64 + lane) * VW;
    // two passes in flight while their registers allow it (not at 8 replicas)
    if constexpr (R < 8) {
        Pass A, B;
        if (j < n) load(A, j);
        between();
        while (j < n) {
            if (j + PASS < n) load(B, j + PASS);
            use(A);
            j += PASS;
            if (j >= n) break;
            if (j + PASS < n) load(A, j + PASS);
            use(B);
            j += PASS;
        }
    } else {
        between();
        for (; j < n; j += PASS) {
            Pass A;
            load(A, j);
            use(A);
        }
    }
    constexpr int C = ROWS * R < 64 ? ROWS * R : 64;  // at most one value per lane is left of a group
    constexpr int SPAN = 64 / C;                       // lanes that hold the same sum
#pragma unroll
    for (int x = 0; x < ROWS * R; x += C) {
        Real v[C];
#pragma unroll
        for (int y = 0; y < C; ++y) v[y] = acc[x + y];
        const Real sum = lanes_sum<Real, C, 32>(v, lane);
        if ((lane & (SPAN - 1)) == 0) red[w][x + gemv_value<C>(lane)] = sum;
    }
}

template <typename Real, int NS, int R>
__global__ __launch_bounds__(256) void dense_gemv_kernel(const StepArgs<Real> a, const Real* __restrict__ M,
                                                         const int64_t ld, const int k) {
    constexpr int ROWS = gemv_rows(sizeof(Real) == 8, R), RPT = R < 4 ? R : 4, TPR = R / RPT;
    __shared__ Real red[4][ROWS * R];
    __shared__ alignas(32) Real xs[NS + 1][ROWS * R];
    __shared__ double trl[ROWS * 3];
    const StepInfo si = step_info<Real, RPT>(a, k);
    const Real* __restrict__ qr = (si.n & 1) ? a.q1 : a.q0;
    Real* __restrict__ qw = (si.n & 1) ? a.q0 : a.q1;
    const int64_t b = blockIdx.x;
    if (b >= a.row_tiles) {  // selected pairs
        const int64_t pk = (b - a.row_tiles) * (int(blockDim.x) / TPR) + si.slot;
        if (pk < a.npairs) pair_update<Real, RPT>(a, si, qr, pk);
        return;
    }
    // odd steps take the row blocks in reverse: the last rows of M that a step read are
    // still in the 256 MB last-level cache when the next one starts with them
    const int64_t row0 = ((si.n & 1) ? a.row_tiles - 1 - b : b) * ROWS;
    gemv_partials<Real, R>(M, ld, a.N, qr, row0, red, [&]() {
        // one Philox block (4 replicas of one component of one row) per lane, dealt to the waves in turn
        constexpr int BLOCKS = (NS + 1) * ROWS * TPR;
        for (int t = int(threadIdx.x & 63) * 4 + int(threadIdx.x >> 6); t < BLOCKS; t += 256) {
            const int c = t / (ROWS * TPR), x = t % (ROWS * TPR);  // x: (row, group of replicas)
            Vec<Real, RPT> z;
            normals<Real, RPT>(a.key0, a.key1, a.stream, uint32_t(row0 + x / TPR), uint32_t(si.n), uint32_t(c),
                               uint32_t((x % TPR) * RPT), z.v);
            store_vec<Real, RPT>(&xs[c][x * RPT], z);
        }
    });
    const int64_t i = row0 + si.slot;
    const bool mine = si.slot < ROWS && i < a.N;
    RowState<Real, NS, RPT> st;
    if (mine) st = load_row<Real, NS, RPT, false>(a, si, qr, i);
    __syncthreads();
    if (mine) {
        Real acc[RPT], xi[NS + 1][RPT];
        const int x0 = si.slot * R + si.r0;
#pragma unroll
        for (int m = 0; m < RPT; ++m) acc[m] = ((red[0][x0 + m] + red[1][x0 + m]) + red[2][x0 + m]) + red[3][x0 + m];
#pragma unroll
        for (int c = 0; c <= NS; ++c)
#pragma unroll
            for (int m = 0; m < RPT; ++m) xi[c][m] = xs[c][x0 + m];
        (void)finish_row<Real, NS, RPT, false>(a, si, i, st, acc, xi, qw,
                                               a.tpart != nullptr ? trl + si.slot * 3 : nullptr);
    }
    if (a.tpart != nullptr) {
        __syncthreads();
        wave0_sum_rows(trl, min(int64_t(ROWS), a.N - row0), a.tpart + (int64_t(k) * a.tpart_w + b) * 3);
    }
}

// The force alone: part[i][r] = (M q)_ir.
template <typename Real, int R>
__global__ __launch_bounds__(256) void gemv_force_kernel(const Real* __restrict__ M, const int64_t ld, const int64_t N,
                                                         const Real* __restrict__ q, Real* __restrict__ part) {
    constexpr int ROWS = gemv_rows(sizeof(Real) == 8, R);
    __shared__ Real red[4][ROWS * R];
    const int64_t row0 = int64_t(blockIdx.x) * ROWS;
    gemv_partials<Real, R>(M, ld, N, q, row0, red, []() {});
    __syncthreads();
    const int x = threadIdx.x;
    if (x < ROWS * R && row0 + x / R < N)
        part[row0 * R + x] = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
}

template <typename Real, int NS>
const void* pick_gemv_r(int R) {
    switch (R) {
        case 1: return reinterpret_cast<const void*>(&dense_gemv_kernel<Real, NS, 1>);
        case 2: return reinterpret_cast<const void*>(&dense_gemv_kernel<Real, NS, 2>);
        case 4: return reinterpret_cast<const void*>(&dense_gemv_kernel<Real, NS, 4>);
        case 8: return reinterpret_cast<const void*>(&dense_gemv_kernel<Real, NS, 8>);
        default: return nullptr;
    }
}

template <typename Real>
const void* pick_gemv(int ns, int R) {
    switch (ns) {
        case 0: return pick_gemv_r<Real, 0>(R);
        case 1: return pick_gemv_r<Real, 1>(R);
        case 2: return pick_gemv_r<Real, 2>(R);
        case 3: return pick_gemv_r<Real, 3>(R);
        case 4: return pick_gemv_r<Real, 4>(R);
        case 5: return pick_gemv_r<Real, 5>(R);
        case 6: return pick_gemv_r<Real, 6>(R);
        case 7: return pick_gemv_r<Real, 7>(R);
        case 8: return pick_gemv_r<Real, 8>(R);
        case 9: return pick_gemv_r<Real, 9>(R);
        case 10: return pick_gemv_r<Real, 10>(R);
        default: return nullptr;
    }
}

}  // namespace dev

template <typename Real>
int launch_dense_gemv_impl(const StepArgs<Real>& a, const Real* M, int64_t ld, int k, void* stream) {
    if (ld % 4 != 0 || ld < a.N || ld > 0x3FFFFFFF) return -4;
    const void* fn = dev::pick_gemv<Real>(a.ns, a.R);
    if (fn == nullptr) return -2;
    StepArgs<Real> aa = a;
    const int rows = gemv_rows(sizeof(Real) == 8, a.R);
    aa.row_tiles = (a.N + rows - 1) / rows;
    const int rpt = a.R < 4 ? a.R : 4;
    if ((a.R / rpt) != (1 << a.lg_tpr)) return -4;
    const int64_t per = 256 / (a.R / rpt);
    const int64_t grid = aa.row_tiles + (a.npairs + per - 1) / per;
    if (grid > 0x7FFFFFFF) return -3;
    void* args[] = {&aa, &M, &ld, &k};
    hipError_t e = hipLaunchKernel(fn, dim3(unsigned(grid)), dim3(256), args, 0, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? 0 : -1;
}

template <typename Real>
int launch_gemv_force_impl(const Real* M, int64_t ld, int64_t N, int R, const Real* q, Real* part, void* stream) {
    if (ld % 4 != 0 || ld < N || ld > 0x3FFFFFFF) return -4;
    const int rows = gemv_rows(sizeof(Real) == 8, R);
    const dim3 grid(unsigned((N + rows - 1) / rows)), block(256);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    switch (R) {
        case 1: hipLaunchKernelGGL((dev::gemv_force_kernel<Real, 1>), grid, block, 0, s, M, ld, N, q, part); break;
        case 2: hipLaunchKernelGGL((dev::gemv_force_kernel<Real, 2>), grid, block, 0, s, M, ld, N, q, part); break;
        case 4: hipLaunchKernelGGL((dev::gemv_force_kernel<Real, 4>), grid, block, 0, s, M, ld, N, q, part); break;
        case 8: hipLaunchKernelGGL((dev::gemv_force_kernel<Real, 8>), grid, block, 0, s, M, ld, N, q, part); break;
        default: return -2;
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace fth
