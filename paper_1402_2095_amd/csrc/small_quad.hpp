// Step loop for small dense systems of up to 128 rows, M in registers.
//
// A step of such a system is a chain of short latencies, so the work of a row is
// spread until the chain is short and everything that need not be in it is taken
// out:
//   - four lanes of a wave share a row; each holds a quarter of the row of M in
//     registers for the whole launch and sums its quarter, and a quad exchange (DPP)
//     leaves all four with the sum; the row's state (q, p, s) is in their registers;
//   - a workgroup takes one replica (they are independent), so R replicas run on R
//     CUs.  With four replicas a workgroup, which use every Philox word, the LDS reads
//     and the products of a step took longer than the words saved: 100 rows, ns = 4,
//     FP32 1.27 us a step, 2 replicas 0.93, 1 replica 0.81;
//   - the normals do not depend on the state: every four steps lane c of a row draws
//     those of step 4 m + c, and the row's lanes read them back from LDS;
//   - the steps write q_n (and p_n, and M q_n for traces, where kept) to a
//     trajectory buffer and nothing waits for it; the estimates are formed from
//     it afterwards, all steps of an estimate in parallel (small_fold_kernel);
//   - one barrier per step, for LDS only: the global stores stay in flight.
// The one-workgroup form (small_dense.hpp) keeps larger systems.  Measured, per
// step, against that form: 64 rows, 1 replica, FP64, white noise 2.2 -> 0.45 us; 100
// rows, 16 replicas, ns = 4 FP32 5.1 -> 0.81 us.
#pragma once

#include <hip/hip_runtime.h>

#include "small_dense.hpp"

namespace fth {
namespace dev {

// Value of the lane at distance X (1 or 2) within the quad.
template <int X>
__device__ __forceinline__ uint32_t quad_xor_u32(uint32_t v) {
    constexpr int ctrl = X == 1 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), ctrl, 0xF, 0xF, true));
}
template <int X>
__device__ __forceinline__ float quad_xor(float v) {
    return __uint_as_float(quad_xor_u32<X>(__float_as_uint(v)));
}
template <int X>
__device__ __forceinline__ double quad_xor(double v) {
    const uint64_t b = uint64_t(__double_as_longlong(v));
    const uint64_t lo = quad_xor_u32<X>(uint32_t(b)), hi = quad_xor_u32<X>(uint32_t(b >> 32));
    return __longlong_as_double(int64_t((hi << 32) | lo));
}

template <typename Real>
__device__ __forceinline__ Real quad_total(Real v) {
    const Real a = v + quad_xor<1>(v);
    return a + quad_xor<2>(a);
}

// Workgroup barrier that orders LDS accesses only: what the waves exchange between
// barriers is in LDS, and stores to the trajectory buffer stay in flight.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// CPL: columns of M per lane (4 CPL >= N).
template <typename Real, int NS, int CPL>
__global__ __launch_bounds__(512) void small_dense_kernel_quad(const StepArgs<Real> a, const SmallTraj<Real> tj,
                                                               const int64_t n0, const int K) {
    extern __shared__ double smem_d[];
    constexpr int D = NS + 1;
    constexpr int NP = 4 * CPL;                    // columns, padded with zeros
    constexpr int VL = 16 / int(sizeof(Real));     // columns of one 16-byte read
    static_assert(CPL % VL == 0, "a lane's columns are whole reads");
    const int N = int(a.N), R = a.R;
    const int tid = int(threadIdx.x), nthr = int(blockDim.x);
    const int c = tid & 3, i = tid >> 2;
    const int r0 = int(blockIdx.x);  // the workgroup's replica
    const int rows = nthr >> 2;
    const bool active = i < N;
    const bool owner = active && c == 0;  // one lane per row stores
    // LDS: q [2][NP] | normals [4 steps][D][rows] | T, S [2][D][D]
    Real* qb = reinterpret_cast<Real*>(smem_d);
    Real* xs = qb + 2 * NP;
    Real* tsl = xs + 4 * D * rows;
    const Real* qg = (n0 & 1) ? a.q1 : a.q0;
    for (int x = tid; x < 2 * NP; x += nthr) qb[x] = Real(0);
    for (int x = tid; x < 2 * D * D; x += nthr) tsl[x] = a.TS[x];
    __syncthreads();
    for (int x = tid; x < N; x += nthr) qb[(n0 & 1) * NP + x] = qg[int64_t(x) * R + r0];

    // column u of the lane: reads of the quad's lanes are consecutive 16-byte pieces
    Real m[CPL];
#pragma unroll
    for (int u = 0; u < CPL; ++u) {
        const int j = ((u / VL) * 4 + c) * VL + u % VL;
        m[u] = active && j < N ? a.mdense[int64_t(j) * N + i] : Real(0);
    }
    RowState<Real, NS, 1> st;
    const int64_t cs = ps_stride(R, a.ps_lg);
    st.q.v[0] = st.p.v[0] = Real(0);
#pragma unroll
    for (int k = 0; k < NS; ++k) st.s[k].v[0] = Real(0);
    if (active) {
        st.q.v[0] = qg[int64_t(i) * R + r0];
        const Real* psrow = ps_row(ps_at_step(a, n0), i, D, R, a.ps_lg) + r0;
        st.p.v[0] = psrow[0];
#pragma unroll
        for (int k = 0; k < NS; ++k) st.s[k].v[0] = psrow[(k + 1) * cs];
    }
    __syncthreads();
    // T and S in registers while they are small, else read from LDS in every step
    constexpr bool TREG = NS <= 4;
    Real ts[TREG ? 2 * D * D : 1];
    if constexpr (TREG) {
#pragma unroll
        for (int x = 0; x < 2 * D * D; ++x) ts[x] = tsl[x];
    }
    const Real* T = TREG ? ts : tsl;
    const Real* S = T + D * D;
    bool ok = true;

    for (int k = 0; k < K; ++k) {
        const int64_t n = n0 + k;
        const Real* qr = qb + (n & 1) * NP;
        Real* qw = qb + ((n + 1) & 1) * NP;
        if (k == 0 || (n & 3) == 0) {  // the normals of steps (n & ~3) .. + 3, step + c by lane c
#pragma unroll
            for (int g = 0; g < D; ++g) {
                normals<Real, 1>(a.key0, a.key1, a.stream, uint32_t(i), uint32_t(n & ~int64_t(3)) + uint32_t(c),
                                 uint32_t(g), uint32_t(r0), xs + (c * D + g) * rows + i);
            }
            __builtin_amdgcn_wave_barrier();  // read back by the same wave only
        }
        if (owner) {
            const int64_t x = (int64_t(k) * N + i) * R + r0;
            tj.q[x] = st.q.v[0];
            if (tj.p != nullptr) tj.p[x] = st.p.v[0];
        }
        // this lane's columns, in four independent chains
        Real part[4] = {Real(0), Real(0), Real(0), Real(0)};
#pragma unroll
        for (int u = 0; u < CPL; u += VL) {
            const Vec<Real, VL> v = load_vec<Real, VL>(qr + ((u / VL) * 4 + c) * VL);
#pragma unroll
            for (int e = 0; e < VL; ++e) part[(u + e) % 4] = fmaR(m[u + e], v.v[e], part[(u + e) % 4]);
        }
        const Real acc[1] = {quad_total<Real>((part[0] + part[1]) + (part[2] + part[3]))};
        if (tj.f != nullptr && owner) tj.f[(int64_t(k) * N + i) * R + r0] = acc[0];
        Real xi[NS + 1][1];
#pragma unroll
        for (int g = 0; g < D; ++g) xi[g][0] = xs[(int(n & 3) * D + g) * rows + i];
        RowState<Real, NS, 1> nx;
        const bool fin = ou_update<Real, NS, 1>(T, S, a.h, a.hh, st, acc, xi, nx);
        ok = ok && (fin || !active);
        st = nx;
        if (owner) qw[i] = st.q.v[0];
        lds_barrier();
    }
    const int64_t nend = n0 + K;
    if (owner) {
        Real* qo = (nend & 1) ? a.q1 : a.q0;
        qo[int64_t(i) * R + r0] = st.q.v[0];
        Real* psrow = ps_row(ps_at_step(a, nend), i, D, R, a.ps_lg) + r0;
        psrow[0] = st.p.v[0];
#pragma unroll
        for (int k = 0; k < NS; ++k) psrow[(k + 1) * cs] = st.s[k].v[0];
    }
    if (!ok) a.flag[0] = 1;
    // (nothing of these launches reads the counter: the first step is an argument)
    if (blockIdx.x == 0 && tid == 0) const_cast<int64_t*>(a.step_base)[0] = nend;
}

// The estimates of K steps from the trajectory: workgroup x takes estimate x of the q-q
// (y = 0) or p-p (y = 1) kind, forms the replica sums of all steps in parallel and adds
// them to the block sum in step order.
template <typename Real>
__global__ __launch_bounds__(kSmallQuadSteps) void small_fold_kernel(const StepArgs<Real> a, const SmallTraj<Real> tj,
                                                                     const int64_t n0, const int K) {
    __shared__ double xs[kSmallQuadSteps];
    const int64_t e = blockIdx.x, np = a.npairs;
    const bool mom = blockIdx.y != 0;
    const Real* src = mom ? tj.p : tj.q;
    int64_t ia, ib, at;
    double *blk, *s1, *s2;
    if (e < np) {
        ia = a.pairs[2 * e];
        ib = a.pairs[2 * e + 1];
        at = e;
        blk = mom ? a.pp_blk : a.pblk;
        s1 = mom ? a.pp_s1 : a.ps1;
        s2 = mom ? a.pp_s2 : a.ps2;
    } else {
        ia = ib = at = e - np;
        blk = mom ? a.dp_blk : a.dblk;
        s1 = mom ? a.dp_s1 : a.ds1;
        s2 = mom ? a.dp_s2 : a.ds2;
    }
    double b = blk[at], v1 = s1[at], v2 = s2[at];
    const int t = int(threadIdx.x);
    if (t < K) {
        const Real* row = src + int64_t(t) * a.N * a.R;
        xs[t] = pair_dot(row + ia * a.R, row + ib * a.R, int64_t(a.R));
    }
    __syncthreads();
    if (t != 0) return;
    // runs of steps up to the end of the open block
    int j = int(min(max(a.burn_in - n0, int64_t(0)), int64_t(K)));
    int64_t left = a.block_len - (n0 > a.burn_in ? (n0 - a.burn_in) % a.block_len : 0);
    while (j < K) {
        const int end = int(min(int64_t(K), j + left));
        left -= end - j;
#pragma unroll 8
        for (; j < end; ++j) b = b + xs[j];
        if (left == 0) {
            v1 = v1 + b;
            v2 = v2 + b * b;
            b = 0.0;
            left = a.block_len;
        }
    }
    blk[at] = b;
    s1[at] = v1;
    s2[at] = v2;
}

// Trace sums of step k (workgroup k) from the trajectory, in a fixed order.
template <typename Real>
__global__ __launch_bounds__(256) void small_trace_kernel(const StepArgs<Real> a, const SmallTraj<Real> tj) {
    __shared__ double red[16 * 3];
    const int64_t k = blockIdx.x, total = a.N * a.R;
    double v[3] = {0.0, 0.0, 0.0};
    for (int64_t x = threadIdx.x; x < total; x += blockDim.x) {
        const double q = double(tj.q[k * total + x]), f = double(tj.f[k * total + x]), p = double(tj.p[k * total + x]);
        v[0] += q * q;
        v[1] += q * f;
        v[2] += p * p;
    }
    workgroup_sum3(v, red);
    if (threadIdx.x == 0)
        for (int c = 0; c < 3; ++c) a.tpart[k * a.tpart_w * 3 + c] = v[c];
}

template <typename Real, int NS>
const void* pick_quad_n(int N) {
    return N <= 64 ? reinterpret_cast<const void*>(&small_dense_kernel_quad<Real, NS, 16>)
                   : reinterpret_cast<const void*>(&small_dense_kernel_quad<Real, NS, 32>);
}

template <typename Real>
const void* pick_quad(int ns, int N) {
    switch (ns) {
        case 0: return pick_quad_n<Real, 0>(N);
        case 1: return pick_quad_n<Real, 1>(N);
        case 2: return pick_quad_n<Real, 2>(N);
        case 3: return pick_quad_n<Real, 3>(N);
        case 4: return pick_quad_n<Real, 4>(N);
        case 5: return pick_quad_n<Real, 5>(N);
        case 6: return pick_quad_n<Real, 6>(N);
        case 7: return pick_quad_n<Real, 7>(N);
        case 8: return pick_quad_n<Real, 8>(N);
        case 9: return pick_quad_n<Real, 9>(N);
        case 10: return pick_quad_n<Real, 10>(N);
        default: return nullptr;
    }
}

}  // namespace dev

template <typename Real>
int launch_small_quad_impl(const StepArgs<Real>& a, const SmallTraj<Real>& tj, int64_t n0, int K, void* stream) {
    if (a.N > kSmallQuadRows || a.N < 1 || K < 1 || K > kSmallQuadSteps) return -3;
    const int block = int((a.N * 4 + 63) / 64 * 64);
    const size_t lds = small_quad_lds(a.N, a.ns, sizeof(Real) == 8);
    const void* fn = dev::pick_quad<Real>(a.ns, int(a.N));
    if (fn == nullptr) return -2;
    const hipStream_t s = static_cast<hipStream_t>(stream);
    StepArgs<Real> aa = a;
    SmallTraj<Real> tt = tj;
    int kk = K;
    void* args[] = {&aa, &tt, &n0, &kk};
    if (hipLaunchKernel(fn, dim3(unsigned(a.R)), dim3(unsigned(block)), args, lds, s) != hipSuccess) return -1;
    const int64_t ne = a.npairs + (a.dblk != nullptr ? a.N : 0);
    if (ne > 0) {
        if (ne > 0x7FFFFFFF) return -3;
        hipLaunchKernelGGL(dev::small_fold_kernel<Real>, dim3(unsigned(ne), a.pp_blk != nullptr ? 2 : 1), dim3(kSmallQuadSteps),
                           0, s, a, tj, n0, K);
    }
    if (a.tpart != nullptr)
        hipLaunchKernelGGL(dev::small_trace_kernel<Real>, dim3(unsigned(K)), dim3(256), 0, s, a, tj);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace fth
