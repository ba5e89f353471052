// Dense step in one launch: a workgroup forms the force of 16 rows over the whole
// of K on the matrix cores and applies the row update to them.
//
// The split-K GEMM with its epilogue (dense.hpp) writes and reads partial sums and
// pays two launches a step, which at a few thousand rows is most of the step, and
// its 128-row blocks leave CUs idle there.  Here the eight waves of a workgroup take
// the k-steps in turn, read A fragments of their 16 rows (which the row block's other
// column groups read too) and the q fragments of 16 CT columns straight into
// registers, one k-step ahead, and their partial sums meet in LDS in wave order.  The
// normals of the rows are drawn between the first loads and their use and wait in LDS.
// What it costs is q: every workgroup reads all N rows of its columns from L2, N / 16
// times N R values a step, so the GEMM form stays for large N R (see
// dense_rows_cols).  M stays in the caches from step to step at these sizes, so its
// loads are plain ones: non-temporal ones took 12.7 us a step for 10.1 (2100 rows,
// R = 64), FP64 14.3 for 12.1 (1500 rows, R = 32), the same up to 1000 rows.
//
// Column groups: with CT < R / 16 a row block is cut into R / (16 CT) workgroups,
// which puts small systems on more CUs.  A row's replicas are then spread over
// workgroups, so the diagonal estimates are taken like the selected pairs, by
// further workgroups of the launch that read q_n (and p_n).
//
// Hazards: q, (p, s) and the bf16 split of q are all double-buffered by step
// parity; no workgroup writes what another one of the launch reads.
#pragma once

#include "dense.hpp"

namespace fth {
namespace dev {

constexpr int kRowsWaves = 8;
constexpr int kRowsThreads = 64 * kRowsWaves;

// Everything after the partial sums: reduction over the waves, row update, and for
// the split form the bf16 split of q_{n+1} (written 16 bytes at a time).
template <typename Real, int NS, int CT>
__device__ __forceinline__ void rows_finish(const StepArgs<Real>& a, int64_t n, int k, int64_t row0, int col0,
                                            const Real* red, const Real* xs, double* trl, Real* qst, uint16_t* qt,
                                            int64_t tile) {
    constexpr int W = 16 * CT, TPR = 4 * CT;
    const int tid = int(threadIdx.x);
    const Real* __restrict__ qr = (n & 1) ? a.q1 : a.q0;
    Real* __restrict__ qw = (n & 1) ? a.q0 : a.q1;
    StepInfo si;
    si.n = n;
    si.acc_on = false;  // no accumulators here
    si.close = false;
    si.tpr = TPR;
    si.rq = tid & (TPR - 1);
    si.r0 = col0 + si.rq * 4;
    si.slot = tid / TPR;
    const int64_t i = row0 + si.slot;
    const bool mine = si.slot < 16;
    const bool live = mine && i < a.N;
    RowState<Real, NS, 4> st;
    if (live) st = load_row<Real, NS, 4, false>(a, si, qr, i);
    __syncthreads();
    if (mine) {
        Vec<Real, 4> qn;
#pragma unroll
        for (int m = 0; m < 4; ++m) qn.v[m] = Real(0);
        if (live) {
            const int x0 = si.slot * W + si.rq * 4;
            Real acc[4], xi[NS + 1][4];
#pragma unroll
            for (int m = 0; m < 4; ++m) acc[m] = Real(0);
#pragma unroll
            for (int w = 0; w < kRowsWaves; ++w) {
                const Vec<Real, 4> v = load_vec<Real, 4>(red + w * 16 * W + x0);
#pragma unroll
                for (int m = 0; m < 4; ++m) acc[m] = acc[m] + v.v[m];
            }
#pragma unroll
            for (int c = 0; c <= NS; ++c) {
                const Vec<Real, 4> v = load_vec<Real, 4>(xs + c * 16 * W + x0);
#pragma unroll
                for (int m = 0; m < 4; ++m) xi[c][m] = v.v[m];
            }
            qn = finish_row<Real, NS, 4, false>(a, si, i, st, acc, xi, qw, a.tpart != nullptr ? trl + si.slot * 3 : nullptr);
        }
        if (qt != nullptr) store_vec<Real, 4>(qst + si.slot * (W + 4) + si.rq * 4, qn);
    }
    if (a.tpart != nullptr || qt != nullptr) __syncthreads();
    if (a.tpart != nullptr)
        wave0_sum_rows(trl, min(int64_t(16), a.N - row0), a.tpart + (int64_t(k) * a.tpart_w + tile) * 3);
    if (qt != nullptr && tid < 4 * W) {
        // unit (8 rows, column, part): qt[k/8][col][hi|lo][k%8]
        const int part = tid & 1, col = (tid >> 1) % W, kb = (tid >> 1) / W;
        uint32_t word[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t two = 0;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float x = float(qst[(kb * 8 + 2 * t + e) * (W + 4) + col]);
                const uint16_t h = bf16_bits(x);
                two |= uint32_t(part ? bf16_bits(x - bf16_value(h)) : h) << (16 * e);
            }
            word[t] = two;
        }
        reinterpret_cast<u32x4*>(qt)[(((row0 >> 3) + kb) * a.R + col0 + col) * 2 + part] =
            u32x4{word[0], word[1], word[2], word[3]};
    }
}

// The normals of the block's 16 rows and 16 CT columns into xs[c][row][col], one
// Philox block per lane and turn.
template <typename Real, int NS, int CT>
__device__ __forceinline__ void rows_noise(const StepArgs<Real>& a, int64_t n, int64_t row0, int col0, Real* xs) {
    constexpr int W = 16 * CT, BLOCKS = (NS + 1) * 16 * 4 * CT;
    for (int t = int(threadIdx.x); t < BLOCKS; t += kRowsThreads) {
        const int c = t / (4 * W), x = t % (4 * W);  // x: (row, group of 4 columns)
        Vec<Real, 4> z;
        normals<Real, 4>(a.key0, a.key1, a.stream, uint32_t(row0 + x / (4 * CT)), uint32_t(n), uint32_t(c),
                         uint32_t(col0 + (x % (4 * CT)) * 4), z.v);
        store_vec<Real, 4>(xs + c * 16 * W + x * 4, z);
    }
}

// Selected pairs and, after them, the diagonal, by the workgroups past the row tiles.
template <typename Real>
__device__ __forceinline__ void rows_estimates(const StepArgs<Real>& a, int k, int64_t block) {
    const StepInfo si = step_info<Real, 4>(a, k);
    const Real* qr = (si.n & 1) ? a.q1 : a.q0;
    const int64_t e = block * (kRowsThreads >> a.lg_tpr) + si.slot;
    if (e < a.npairs) {
        pair_update<Real, 4>(a, si, qr, e);
        return;
    }
    const int64_t i = e - a.npairs;
    if (a.dblk == nullptr || i >= a.N) return;
    const Vec<Real, 4> q = load_vec<Real, 4>(qr + i * a.R + si.r0);
    const double x = dot_row<Real, 4>(q, q, si.tpr);
    if (si.rq == 0 && si.acc_on) acc_update(a.dblk, a.ds1, a.ds2, i, x, si.close);
    if (a.dp_blk != nullptr) {
        const Vec<Real, 4> p = load_vec<Real, 4>(ps_row(ps_at_step(a, si.n), i, a.D(), a.R, a.ps_lg) + si.r0);
        const double y = dot_row<Real, 4>(p, p, si.tpr);
        if (si.rq == 0 && si.acc_on) acc_update(a.dp_blk, a.dp_s1, a.dp_s2, i, y, si.close);
    }
}

// Row block and column group of workgroup b: the column groups of a row block go to
// the same XCD (workgroups are dealt round-robin over the 8), so its rows of M are
// read into one L2.
// (cgroups is a power of two.)
__device__ __forceinline__ bool rows_tile(uint32_t b, int cgroups, int64_t N, int64_t& rg, int& cg) {
    cg = int(b >> 3) & (cgroups - 1);
    rg = int64_t(b >> (3 + __builtin_ctz(uint32_t(cgroups)))) * 8 + (b & 7);
    return rg * 16 < N;
}

template <int NS, int CT>
__global__ __launch_bounds__(kRowsThreads) void dense_rows_bf16x3_kernel(const StepArgs<float> aa,
                                                                         const DenseRowsArgs g, const int k) {
    constexpr int W = 16 * CT;
    extern __shared__ double rows_smem[];
    if (int64_t(blockIdx.x) >= g.tiles) {
        rows_estimates<float>(aa, k, int64_t(blockIdx.x) - g.tiles);
        return;
    }
    int64_t rg;
    int cg;
    if (!rows_tile(blockIdx.x, g.cgroups, aa.N, rg, cg)) return;  // whole workgroup
    StepArgs<float> a = aa;
    a.dblk = a.dp_blk = nullptr;
    const int R = a.R, col0 = cg * W;
    const int64_t row0 = rg * 16, n = a.step_base[0] + k;
    double* trl = rows_smem;                          // [16][3]
    float* red = reinterpret_cast<float*>(trl + 48);  // [waves][16][W]
    float* xs = red + kRowsWaves * 16 * W;            // [NS + 1][16][W]
    float* qst = xs + (NS + 1) * 16 * W;              // [16][W + 4]
    const uint16_t* qt_in = (n & 1) ? g.qt1 : g.qt0;
    uint16_t* qt_out = (n & 1) ? g.qt0 : g.qt1;
    const int l = int(threadIdx.x) & 63, lr = l & 15, lg = l >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int64_t KB = g.rows_pad >> 6;
    // the four 1 KB slots (hi and lo, two substeps) of the 16 rows in k-step kb
    const u32x4* mt = static_cast<const u32x4*>(g.m) + (rg >> 3) * KB * 2048 + ((rg >> 1) & 3) * 512 + (rg & 1) * 256 + l;
    const u32x4* qs = reinterpret_cast<const u32x4*>(qt_in) + (int64_t(2 * lg) * R + col0 + lr) * 2;

    f32x4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    struct Frag {
        u32x4 m[4];          // hi t0, hi t1, lo t0, lo t1
        u32x4 q[2][CT][2];   // [substep][column tile][hi|lo]
    };
    auto load = [&](Frag& f, int kb) {
        const u32x4* ms = mt + int64_t(kb) * 2048;
#pragma unroll
        for (int u = 0; u < 4; ++u) f.m[u] = ms[u * 64];
        const u32x4* q = qs + int64_t(kb) * 16 * R;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                f.q[t][c][0] = q[(t * R + 16 * c) * 2];
                f.q[t][c][1] = q[(t * R + 16 * c) * 2 + 1];
            }
    };
    auto use = [&](const Frag& f) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const bf16x8 hi = __builtin_bit_cast(bf16x8, f.m[t]), lo = __builtin_bit_cast(bf16x8, f.m[2 + t]);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, __builtin_bit_cast(bf16x8, f.q[t][c][0]), acc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, __builtin_bit_cast(bf16x8, f.q[t][c][1]), acc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, __builtin_bit_cast(bf16x8, f.q[t][c][0]), acc[c], 0, 0, 0);
        }
    };
    Frag A, B;
    int kb = wave;
    if (kb < g.ksteps) load(A, kb);
    rows_noise<float, NS, CT>(a, n, row0, col0, xs);
    while (kb < g.ksteps) {
        if (kb + kRowsWaves < g.ksteps) load(B, kb + kRowsWaves);
        use(A);
        kb += kRowsWaves;
        if (kb >= g.ksteps) break;
        if (kb + kRowsWaves < g.ksteps) load(A, kb + kRowsWaves);
        use(B);
        kb += kRowsWaves;
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[(wave * 16 + 4 * lg + e) * W + 16 * c + lr] = acc[c][e];
    rows_finish<float, NS, CT>(a, n, k, row0, col0, red, xs, trl, qst, qt_out, rg * g.cgroups + cg);
}

template <int NS, int CT>
__global__ __launch_bounds__(kRowsThreads) void dense_rows_f64_kernel(const StepArgs<double> aa, const DenseRowsArgs g,
                                                                      const int k) {
    constexpr int W = 16 * CT;
    extern __shared__ double rows_smem[];
    if (int64_t(blockIdx.x) >= g.tiles) {
        rows_estimates<double>(aa, k, int64_t(blockIdx.x) - g.tiles);
        return;
    }
    int64_t rg;
    int cg;
    if (!rows_tile(blockIdx.x, g.cgroups, aa.N, rg, cg)) return;  // whole workgroup
    StepArgs<double> a = aa;
    a.dblk = a.dp_blk = nullptr;
    const int R = a.R, col0 = cg * W;
    const int64_t row0 = rg * 16, n = a.step_base[0] + k, P = g.rows_pad;
    double* trl = rows_smem;
    double* red = trl + 48;
    double* xs = red + kRowsWaves * 16 * W;
    const double* q = (n & 1) ? a.q1 : a.q0;
    const int l = int(threadIdx.x) & 63, lr = l & 15, lg = l >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    // within a k-step of 16, lane group lg handles k = 4 lg + t at substep t
    const double* arow = static_cast<const double*>(g.m) + (row0 + lr) * P + 4 * lg;
    const double* qcol = q + int64_t(4 * lg) * R + col0 + lr;

    f64x4 acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f64x4{0.0, 0.0, 0.0, 0.0};
    struct Frag {
        f64x2 m[2];
        double q[4][CT];
    };
    auto load = [&](Frag& f, int kb) {
        f.m[0] = *reinterpret_cast<const f64x2*>(arow + int64_t(kb) * 16);
        f.m[1] = *reinterpret_cast<const f64x2*>(arow + int64_t(kb) * 16 + 2);
        const double* qk = qcol + int64_t(kb) * 16 * R;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c) f.q[t][c] = qk[t * R + 16 * c];
    };
    auto use = [&](const Frag& f) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int c = 0; c < CT; ++c)
                acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(f.m[t >> 1][t & 1], f.q[t][c], acc[c], 0, 0, 0);
    };
    Frag A, B;
    int kb = wave;
    if (kb < g.ksteps) load(A, kb);
    rows_noise<double, NS, CT>(a, n, row0, col0, xs);
    while (kb < g.ksteps) {
        if (kb + kRowsWaves < g.ksteps) load(B, kb + kRowsWaves);
        use(A);
        kb += kRowsWaves;
        if (kb >= g.ksteps) break;
        if (kb + kRowsWaves < g.ksteps) load(A, kb + kRowsWaves);
        use(B);
        kb += kRowsWaves;
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[(wave * 16 + 4 * e + lg) * W + 16 * c + lr] = acc[c][e];
    rows_finish<double, NS, CT>(a, n, k, row0, col0, red, xs, trl, nullptr, nullptr, rg * g.cgroups + cg);
}

template <typename Real, int NS, int CT>
const void* rows_fn() {
    if constexpr (sizeof(Real) == 4)
        return reinterpret_cast<const void*>(&dense_rows_bf16x3_kernel<NS, CT>);
    else
        return reinterpret_cast<const void*>(&dense_rows_f64_kernel<NS, CT>);
}

// (four column tiles: n is beyond the FP64 form's range wherever they are chosen)
template <typename Real, int NS>
const void* pick_rows_ct(int ct) {
    switch (ct) {
        case 1: return rows_fn<Real, NS, 1>();
        case 2: return rows_fn<Real, NS, 2>();
        case 4:
            if constexpr (sizeof(Real) == 4) return rows_fn<Real, NS, 4>();
            return nullptr;
        default: return nullptr;
    }
}

template <typename Real>
const void* pick_rows(int ns, int ct) {
    switch (ns) {
        case 0: return pick_rows_ct<Real, 0>(ct);
        case 1: return pick_rows_ct<Real, 1>(ct);
        case 2: return pick_rows_ct<Real, 2>(ct);
        case 3: return pick_rows_ct<Real, 3>(ct);
        case 4: return pick_rows_ct<Real, 4>(ct);
        case 5: return pick_rows_ct<Real, 5>(ct);
        case 6: return pick_rows_ct<Real, 6>(ct);
        case 7: return pick_rows_ct<Real, 7>(ct);
        case 8: return pick_rows_ct<Real, 8>(ct);
        case 9: return pick_rows_ct<Real, 9>(ct);
        case 10: return pick_rows_ct<Real, 10>(ct);
        default: return nullptr;
    }
}

}  // namespace dev

template <typename Real>
int launch_dense_rows_impl(const StepArgs<Real>& a, const DenseRowsArgs& g0, int ct, int k, void* stream) {
    const bool f64 = sizeof(Real) == 8;
    DenseRowsArgs g = g0;
    if (a.R % (16 * ct) != 0 || (1 << a.lg_tpr) != a.R / 4 || a.R > 128) return -3;
    if (!f64 && (g.qt0 == nullptr || g.qt1 == nullptr)) return -4;
    g.cgroups = a.R / (16 * ct);
    const int64_t rgs = (a.N + 15) / 16;
    g.tiles = (rgs + 7) / 8 * 8 * g.cgroups;
    g.ksteps = int32_t(f64 ? (a.N + 15) / 16 : (a.N + 63) / 64);
    if (int64_t(g.ksteps) * (f64 ? 16 : 64) > g.rows_pad || g.rows_pad % 128 != 0) return -4;
    const int64_t per = dev::kRowsThreads >> a.lg_tpr;
    const int64_t ne = a.npairs + (a.dblk != nullptr ? a.N : 0);
    const int64_t grid = g.tiles + (ne + per - 1) / per;
    if (grid > 0x7FFFFFFF) return -3;
    const void* fn = dev::pick_rows<Real>(a.ns, ct);
    if (fn == nullptr) return -2;
    const size_t lds = 48 * sizeof(double) + size_t(dev::kRowsWaves + a.ns + 1) * 16 * 16 * size_t(ct) * sizeof(Real) +
                       (f64 ? 0 : 16 * (16 * size_t(ct) + 4) * sizeof(float));
    if (lds > 160 * 1024) return -3;
    StepArgs<Real> aa = a;
    void* args[] = {&aa, &g, &k};
    hipError_t e = hipLaunchKernel(fn, dim3(unsigned(grid)), dim3(dev::kRowsThreads), args, lds,
                                   static_cast<hipStream_t>(stream));
    return e == hipSuccess ? 0 : -1;
}

}  // namespace fth
