// The fused pass's second and third stage in one launch, for matrices whose counts of entries, one per row and panel, are few enough that
// every workgroup can add them all up for itself.
#ifndef REGOT_FINISH_SMALL_HPP
#define REGOT_FINISH_SMALL_HPP

#include "regot_kernels.hpp"

namespace regot {

// Behind the plan pass of a small matrix finalize_kernel and scatter_kernel are chains of memory latencies (4.8 and 4.0 us at 1000 x
// 1000, and the gap of a launch between them), and the second waits for the first only for the rows' places.  Those are sums over
// the counts of all rows before, 4 bytes for a row and panel: with at most kOnceCounts of them a workgroup has them in up to 24 loads a
// thread, 16 under way at once.  Workgroups, each of kFinThreads:
//   0: the objective (objective_at_once);
//   then one for 64 columns (finalize_columns);
//   then one for a row chunk (the first one also writes the scalars of the call): its rows' sums, its part of row_ptr, and the records of its waves' runs, a run to a wave; runs of
//   earlier flushes are looked for in the list of them, which is empty unless a wave had more than kRecCap records.
// Fused pass with 1 % of the entries, us a call, the two launches / this: 64 x 64 16.2 / 13.3, 1000 x 1000 19.2 / 16.1, 2000 x 2000 27.9 / 23.7,
// 3000 x 3000 38.8 / 35.4; sparsification alone 1000 x 1000 17.4 / 14.7.  Beyond kOnceCounts the sums over all counts and the
// objective's workgroup take what the launch took: 4999 x 3001 47.3 / 46.2, 4000 x 4000 47.4 / 48.0.  Nor for more than kOnceEntries a chunk, which
// is one workgroup's to place: 1000 x 1000 with half of its entries (7900 a chunk) 23.3 / 23.3, all of them 34 / 50, 33 x 4000 with 13000 a
// chunk 20.2 / 22.9.
constexpr int kOnceCounts = 24576;
constexpr int kOnceEntries = 6144;                         // of the capacity, for a chunk
constexpr int kOnceChunk = 2048;                           // counts of a chunk
constexpr int kOnceEach = kOnceChunk / kFinThreads;        // of a thread of its scan
constexpr int kOnceRecords = 4;                            // records of a lane under way at a time

// the records of run R (uniform in the wave) to their places; place: LDS, [row of the chunk][panel]
__device__ __forceinline__ void place_run(const ScatterArgs &S, const PoolRange &R, long long before, const int *place, int lane)
{
    const int col0 = (R.panel == S.g_c - 1 && S.m >= kPanel) ? S.m - kPanel : R.panel * kPanel;  // (as in scatter_kernel)
    for (int k0 = 0; k0 < R.count; k0 += kOnceRecords * kLanes) {
        unsigned pk[kOnceRecords];
        double v[kOnceRecords];
#pragma unroll
        for (int e = 0; e < kOnceRecords; ++e) {
            const int k = k0 + e * kLanes + lane;
            pk[e] = k < R.count ? S.pool_packed[(size_t)R.start + k] : 0u;
            v[e] = k < R.count ? S.pool_val[(size_t)R.start + k] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < kOnceRecords; ++e) {
            if (k0 + e * kLanes + lane >= R.count) break;
            const int at = min((int)(pk[e] >> 18) * S.g_c + R.panel, kOnceChunk - 1);
            const long long to = before + place[at] + (int)((pk[e] >> 9) & 511);
            if (to < S.capacity) {  // (always, without overflow)
                S.col_idx[to] = col0 + (int)(pk[e] & 511);
                S.val[to] = v[e];
            }
        }
    }
}

template <bool REDUCE>
__global__ __launch_bounds__(kFinThreads) void finish_small_kernel(ScatterArgs S, FinalizeArgs F)
{
    __shared__ double lds_part[kFinSub][kLanes];
    __shared__ int place[kOnceChunk];
    __shared__ int lds_all[2][kFinSub];
    const int tid = threadIdx.x, lane = tid & (kLanes - 1), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int block = (int)blockIdx.x;
    if constexpr (REDUCE) {
        if (block <= F.nblk_cols) {
            if (block == 0) objective_at_once(F);
            else finalize_columns(F, block - 1, lds_part);
            return;
        }
        block -= 1 + F.nblk_cols;
    }
    int r_begin, r_end;
    chunk_rows(block, S.g_r, S.n, r_begin, r_end);
    const int rows = r_end - r_begin;
    const int hdr_runs = S.header[HDR_RANGE_NEXT], hdr_overflow = S.header[HDR_POOL_OVERFLOW];
    // all counts, and those of the rows before; the chunk's own ones by row and panel
    int all = 0, before = 0;
    const int counts = S.n * S.g_c;
#pragma unroll 16
    for (int k = tid; k < counts; k += kFinThreads) {
        const int c = S.seg_rel[k];
        all += c;
        before += k % S.n < r_begin ? c : 0;
    }
    int mine[kOnceEach];
#pragma unroll
    for (int e = 0; e < kOnceEach; ++e) {
        const int at = kOnceEach * tid + e, row = at / S.g_c, p = at - row * S.g_c;
        mine[e] = row < rows ? S.seg_rel[(size_t)p * S.n + r_begin + row] : 0;
    }
    const int64_t rid = ((int64_t)block * S.g_c) * kWaves + w;  // the wave's first run
    const int runs = S.g_c * kWaves;
    PoolRange R{};
    if (w < runs) R = S.ranges[rid];
    if constexpr (REDUCE) {
        for (int i = tid; i < rows; i += kFinThreads) {
            const int row = r_begin + i;
            double v[kOncePanels];
#pragma unroll
            for (int p = 0; p < kOncePanels; ++p) v[p] = p < F.g_c ? F.rowpart[(size_t)p * F.n + row] : 0.0;
            const double a = F.a[row];
            double r = v[0];
#pragma unroll
            for (int p = 1; p < kOncePanels; ++p) r += v[p];
            if (F.row_sum) F.row_sum[row] = r;
            F.grad_alpha[row] = a - r;
        }
    }
    int sum = 0;
#pragma unroll
    for (int e = 0; e < kOnceEach; ++e) sum += mine[e];
    const int up_to = wave_scan(sum);
    all = wave_scan(all);
    before = wave_scan(before);
    __shared__ int lds_scan[kFinSub];
    if (lane == kLanes - 1) {
        lds_scan[w] = up_to;
        lds_all[0][w] = all;
        lds_all[1][w] = before;
    }
    __syncthreads();
    int run = up_to - sum;
    all = before = 0;
#pragma unroll
    for (int q = 0; q < kFinSub; ++q) {
        run += q < w ? lds_scan[q] : 0;
        all += lds_all[0][q];
        before += lds_all[1][q];
    }
    const bool overflow = all > S.capacity || hdr_overflow != 0;
    if (block == 0) {
        if (tid == 0) {
            S.info[0] = all;
            S.info[1] = overflow ? 1 : 0;
        }
        if (F.cu_table != nullptr)
            for (int i = tid; i < kCuKeys * (int)(sizeof(CuSlot) / sizeof(int)); i += kFinThreads) F.cu_table[i] = 0;
    }
#pragma unroll
    for (int e = 0; e < kOnceEach; ++e) {
        place[kOnceEach * tid + e] = run;
        run += mine[e];
    }
    __syncthreads();
    for (int i = tid; i < rows; i += kFinThreads) S.row_ptr[r_begin + i] = (int64_t)before + place[i * S.g_c];
    if (r_end == S.n && tid == 0) S.row_ptr[S.n] = all;
    if (overflow) return;
    for (int q = w; q < runs; q += kFinSub) {
        if (q != w) R = S.ranges[rid + (q - w)];
        place_run(S, R, before, place, lane);
    }
    const int extra = min(hdr_runs, S.max_ranges - S.fixed_runs);
    for (int e0 = w * kLanes; e0 < extra; e0 += kFinThreads) {
        PoolRange X{};
        if (e0 + lane < extra) X = S.ranges[S.fixed_runs + e0 + lane];
        for (uint64_t hits = __ballot(X.count > 0 && X.r_begin == r_begin); hits != 0; hits &= hits - 1) {
            const int from = __builtin_ctzll(hits);
            const PoolRange Y{__builtin_amdgcn_readlane(X.start, from), __builtin_amdgcn_readlane(X.count, from),
                              __builtin_amdgcn_readlane(X.panel, from), r_begin};
            place_run(S, Y, before, place, lane);
        }
    }
}

}  // namespace regot

#endif  // REGOT_FINISH_SMALL_HPP
