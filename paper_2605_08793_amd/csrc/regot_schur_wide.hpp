// The reduced solve of regot_schur.hpp for systems both of whose blocks are longer than a vector that fits the LDS there
// (kSchurCap): the kernels there gather what is not in LDS once per system, these once for both, the vectors of a pair side by
// side.  The line lies where the vectors cease to fit, not where the two meet, which is further on; 16 iterations here / there, us,
// single and pair:
//   22000 x 22000, 2e6 entries  490 / 459   621 / 532        32000 x 32000, 3e6  577 /  617    777 /  804
//   25000 x 25000, 5e5          496 / 305   629 / 370        40000 x 40000, 4e6  736 /  840    947 / 1240
//   26000 x 26000, 2e6          534 / 463   695 / 541        50000 x 50000, 5e6  936 / 1014   1168 / 1551
//   22000 x 120000, 3e6        1014 / 832  1273 / 1187
// Where one block is short those are faster: 40000 x 10000 with 4e6 entries 681 / 654 and 858 / 852, with 4e5 455 / 323 and
// 593 / 397; 15000 x 100000, 3e6 919 / 763 and 1156 / 1064; 100000 x 15000 885 / 737 and 1083 / 1024; a whole pair of 300000 x 60,
// 1.2e6 entries 2180 / 515, of 10^6 x 1000, 3e6 1896 / 1149.
// An iteration is four kernels: the half products by rows and by columns (the sweep of the product kernel with
// another last step per row), and the vector kernels of the iteration on the whole matrix, on the second block alone.
#pragma once

#include "regot_pcg.hpp"

namespace regot {

// R systems at once as in the kernels above: the vectors the iteration itself produces (u, p, S p, the iterate) are
// "packed", R side by side (see Pack); what the caller hands over or gets back (the right-hand sides, the solutions)
// and the right-hand sides of the reduced systems are plain arrays, one per system.
enum WideMode {
    kWideRows = 0,       // out_i = (sum_j T_ij in_j / eta) / D1_i             u = D1^{-1} B p      out packed
    kWideRowsFinal = 1,  // out_i = (own_i - sum_j T_ij in_j / eta) / D1_i     x1, own = g1         own, out plain
    kWideCols = 2,       // out_j = D2_j own_j - sum_i T_ij in_i / eta         S p, own = p         own, out packed;
                          //                                                    and own^T out
    kWideColsRhs = 3     // out_j = own_j - sum_i T_ij in_i / eta              own = g2             own, out plain
};

template <int R>
struct WideArgs {
    MatvecArgs mv;       // pattern, values, sums, eta, tau (x, y, row_waves unused)
    const double *in;    // packed: the vectors the entries are multiplied with, m - 1 entries (rows) or n (columns)
    const double *own[R];  // see WideMode; a packed vector is own[0]
    double *out[R];        // a packed vector is out[0]
    double *dot_part;    // kWideCols: partial sums of own^T out, one per system and group of kWaves waves
    const int *skip;     // the kernel does nothing if *skip is set (may be NULL)
};

template <int MODE, int R>
struct WideItem {
    static constexpr bool kPacked = MODE == kWideRows || MODE == kWideCols;
    const double *sums;
    const double *own[R];
    double *out[R];
    double eta, inv_eta, tau;
    double dg;
    Pack<R> mine;
    __device__ __forceinline__ void fetch(int64_t t)
    {
        dg = sums[t] / eta + tau;
        if (MODE == kWideCols) {
            mine = load_pack<R>(own[0], t);
        } else {
#pragma unroll
            for (int k = 0; k < R; ++k) mine.v[k] = MODE == kWideRows ? 0.0 : own[k][t];
        }
    }
    __device__ __forceinline__ Pack<R> finish(int64_t t, bool have, const Pack<R> &sum)
    {
        Pack<R> term, o;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            term.v[k] = 0.0;
            const double bs = sum.v[k] * inv_eta;
            if (MODE == kWideRows) o.v[k] = bs / dg;
            else if (MODE == kWideRowsFinal) o.v[k] = (mine.v[k] - bs) / dg;
            else if (MODE == kWideCols) o.v[k] = dg * mine.v[k] - bs;
            else o.v[k] = mine.v[k] - bs;
            if (MODE == kWideCols && have) term.v[k] = o.v[k] * mine.v[k];
        }
        if (have) {
            if (kPacked) {
                store_pack<R>(out[0], t, o);
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) out[k][t] = o.v[k];
            }
        }
        return term;
    }
};

template <int MODE, int R>
__global__ __launch_bounds__(kMatvecLdsThreads) void wide_half_kernel(WideArgs<R> S)
{
    __shared__ __attribute__((aligned(16))) double xs[kMatvecLdsCap];
    __shared__ double wave_dot[R][kMatvecLdsWaves];
    if (S.skip != nullptr && *S.skip) return;
    const MatvecArgs &A = S.mv;
    constexpr bool ROWS = MODE == kWideRows || MODE == kWideRowsFinal;
    const int lane = threadIdx.x & (kLanes - 1), w = threadIdx.x >> 6;
    const int mb = A.m - 1;
    const int limit = ROWS ? mb : A.n;
    const int nl = limit < kMatvecLdsCap / R ? limit : kMatvecLdsCap / R;
    double dot[R];
    WideItem<MODE, R> item;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        dot[k] = 0.0;
        item.own[k] = S.own[k];
        item.out[k] = S.out[k];
    }
    item.sums = ROWS ? A.row_sum : A.col_sum;
    item.eta = A.eta;
    item.inv_eta = 1.0 / A.eta;
    item.tau = A.tau;
    const int64_t *ptr = ROWS ? A.row_ptr : A.col_ptr;
    const int64_t count = ROWS ? A.n : mb;
    const int64_t first = (int64_t)blockIdx.x * kMatvecLdsWaves + w, stride = (int64_t)gridDim.x * kMatvecLdsWaves;
    const SweepHead head = lds_sweep_head(ptr, A.capacity, count, first, stride, lane, item);
    lds_fill(xs, S.in, nl * R);
    __syncthreads();
    lds_sweep<R, false>(ptr, ROWS ? A.col_idx : A.row_idx, ROWS ? A.val : A.val_csc, A.capacity, S.in, xs, nl, limit, count,
                      first, stride, lane, item, dot, head);
    if constexpr (MODE == kWideCols) lds_leave_dots<R>(dot, wave_dot, S.dot_part, (int)kPcgParts, lane, w);
}

// start of a reduced solve: u = D1^{-1} g1 (packed), and partial sums of ||rhs||^2 over both blocks -> rows 3R + k
// of `part`
template <int R>
struct WidePrepareArgs {
    int64_t n, N;
    const double *rhs[R];
    const double *row_sum;
    double eta, tau;
    double *u;
    double *part;
};
template <int R>
__global__ __launch_bounds__(kThreads) void wide_prepare_kernel(WidePrepareArgs<R> A)
{
    __shared__ double lds[kWaves];
    double gg[R];
#pragma unroll
    for (int k = 0; k < R; ++k) gg[k] = 0.0;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < A.N; t += (int64_t)gridDim.x * kThreads) {
        Pack<R> g;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            g.v[k] = A.rhs[k][t];
            gg[k] += g.v[k] * g.v[k];
        }
        if (t < A.n) {
            const double d1 = A.row_sum[t] / A.eta + A.tau;
#pragma unroll
            for (int k = 0; k < R; ++k) g.v[k] = g.v[k] / d1;
            store_pack<R>(A.u, t, g);
        }
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const double s = block_sum(gg[k], lds);
        if (threadIdx.x == 0) A.part[(size_t)(3 * R + k) * kPcgParts + blockIdx.x] = s;
    }
}

}  // namespace regot
