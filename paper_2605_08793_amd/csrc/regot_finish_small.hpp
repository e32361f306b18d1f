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
//   then one for a row chunk (the first one also writes the scalars of the call): its rows' sums, its part of row_ptr, and the records of
//   its waves' runs, a run to a wave.
// Where a chunk's runs are longer than a wave places at a time, or a wave had more than kRecCap records and listed runs of earlier flushes, the
// records are dealt out in portions, to the waves of as many workgroups as that takes (the grid's second dimension: most of
// them see that they are not needed, and return).  All entries of a matrix may be in one chunk, and one workgroup, which took runs of the list as
// they lay, so mostly by one wave, was slow at that.  3000 x 3000, 84000 entries in 28 rows, us, two launches / one workgroup a chunk / this:
// 43 / 242 / 47; 3072 x 4096, 118784 in 29 rows 44 / 262 / 50; 2000 x 2000, 36000 in 18 rows 28 / 81 / 30; 1000 x 1000, 9000 in 9 rows 21.7 / 32.1 / 21.9.
// Fused pass with 1 % of the entries all over the matrix, us a call, the two launches / this: 64 x 64 16.3 / 13.6, 1000 x 1000 19.2 / 16.1, 2000 x
// 2000 27.5 / 23.6, 3000 x 3000 38.0 / 34.8; sparsification alone 1000 x 1000 17.4 / 14.7.  Beyond kOnceCounts the sums over all counts and the
// objective's workgroup take what the launch took: 4999 x 3001 47.3 / 46.2, 4000 x 4000 47.4 / 48.0.  kOnceEntries lies where one workgroup a chunk
// met the two launches (1000 x 1000 with half of its entries, 7900 a chunk); with several it is still ahead behind that line, there 23.8 / 22.1, with all of
// the entries 33.9 / 32.4.  kOnceMost keeps a chunk of a few wide rows, whose workgroups have more than that each, with the launches.
constexpr int kOnceCounts = 24576;
constexpr int kOnceEntries = 6144;                         // of the capacity, for a chunk
constexpr int kOnceChunk = 2048;                           // counts of a chunk
constexpr int kOnceEach = kOnceChunk / kFinThreads;        // of a thread of its scan
constexpr int kOnceRecords = 4;                            // records of a lane under way at a time,
constexpr int kOncePortion = kOnceRecords * kLanes;        // and of a wave
constexpr int kOnceRunPortions = (kRecCap + kOncePortion - 1) / kOncePortion;
constexpr int kOnceEasy = 2;                               // portions a wave, up to which a chunk is one workgroup's
constexpr int kOnceMost = 6;                               // portions a wave with all workgroups of a chunk
static_assert(kOncePanels * kWaves <= kLanes, "a lane for a fixed run");
constexpr int kOnceTable = kFinSub * kLanes * (int)sizeof(double) / (int)sizeof(PoolRange);  // runs of the list looked at at a time
static_assert(kOnceTable <= kFinThreads && kOnceTable % kLanes == 0, "a thread for a run");

// a part of a run, at most kOncePortion records of it
struct Portion {
    int start, count, panel;
};

template <bool REDUCE>
__global__ __launch_bounds__(kFinThreads) void finish_small_kernel(ScatterArgs S, FinalizeArgs F, int most_parts)
{
    __shared__ __attribute__((aligned(16))) double lds_part[kFinSub][kLanes];
    __shared__ int place[kOnceChunk];        // where the records of a row and panel go
    __shared__ int lds_all[2][kFinSub], lds_scan[kFinSub];
    PoolRange *table = reinterpret_cast<PoolRange *>(lds_part);  // runs of the list, at most kOnceTable
    __shared__ int lds_runs[kFinSub];
    const int tid = threadIdx.x, lane = tid & (kLanes - 1), w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int block = (int)blockIdx.x;
    if constexpr (REDUCE) {
        if (block <= F.nblk_cols) {
            if (blockIdx.y > 0) return;
            if (block == 0) objective_at_once(F);
            else finalize_columns(F, block - 1, lds_part);
            return;
        }
        block -= 1 + F.nblk_cols;
    }
    const int part = (int)blockIdx.y;
    int r_begin, r_end;
    chunk_rows(block, S.g_r, S.n, r_begin, r_end);
    const int rows = r_end - r_begin;
    // The runs with a fixed number, of each wave a lane's, and those of the list.  Usually the former have a portion each and there are none of
    // the latter: then part 0 places a run a wave.
    const PoolRange *runs = S.ranges + ((int64_t)block * S.g_c) * kWaves;
    const int fixed_runs = S.g_c * kWaves;
    // (Asked for by lanes: the compiler would wait at once for what is the same in all of a wave.)
    int none = 0;
    asm volatile("" : "+v"(none));
    const int hdr_runs = S.header[HDR_RANGE_NEXT + none], hdr_overflow = S.header[HDR_POOL_OVERFLOW + none];
    PoolRange R{}, fixed{};
    if (w < fixed_runs) R = runs[w + none];
    if (lane < fixed_runs) fixed = runs[lane];
    int extra = 0;
    const auto listed = [&](int e) {  // run e of the list, if it is the chunk's
        PoolRange X{};
        if (e < extra) X = S.ranges[S.fixed_runs + e];
        if (X.r_begin != r_begin) X.count = 0;
        return X;
    };
    int fixed_up_to = 0, fixed_portions = 0, parts = 1;  // (parts: workgroups that have something to place)
    const auto share_out = [&] {
        fixed_up_to = wave_scan((min(fixed.count, kRecCap) + kOncePortion - 1) / kOncePortion);
        fixed_portions = __builtin_amdgcn_readlane(fixed_up_to, kLanes - 1);
        int portions = fixed_portions;
        if (extra > 0) {
            int found = 0;
            for (int e0 = 0; e0 < extra; e0 += kFinThreads) found += __builtin_popcountll(__ballot(listed(e0 + tid).count > 0));
            if (lane == 0) lds_runs[w] = found;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFinSub; ++q) portions += kOnceRunPortions * lds_runs[q];
            __syncthreads();
        }
        parts = max(1, min(most_parts, (portions + kOnceEasy * kFinSub - 1) / (kOnceEasy * kFinSub)));
    };
    if (part > 0) {
        extra = min(__builtin_amdgcn_readfirstlane(hdr_runs), S.max_ranges - S.fixed_runs);
        if (extra <= 0 && __ballot(fixed.count > kOncePortion) == 0) return;
        share_out();
        if (part >= parts) return;
    }
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
    if constexpr (REDUCE) {
        const int end = part == 0 ? rows : 0;
        for (int i = tid; i < end; i += kFinThreads) {
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
    extra = min(__builtin_amdgcn_readfirstlane(hdr_runs), S.max_ranges - S.fixed_runs);
    const bool usual = extra <= 0 && __ballot(fixed.count > kOncePortion) == 0;
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
    const bool overflow = all > S.capacity || __builtin_amdgcn_readfirstlane(hdr_overflow) != 0;
    if (block == 0 && part == 0) {
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
    if (part == 0) {
        for (int i = tid; i < rows; i += kFinThreads) S.row_ptr[r_begin + i] = (int64_t)before + place[i * S.g_c];
        if (r_end == S.n && tid == 0) S.row_ptr[S.n] = all;
    }
    if (overflow) return;
    const auto place_portions = [&](auto number_tag, const Portion *P) {
        constexpr int NUMBER = decltype(number_tag)::value;
        unsigned pk[NUMBER][kOnceRecords];
        double v[NUMBER][kOnceRecords];
#pragma unroll
        for (int h = 0; h < NUMBER; ++h)
#pragma unroll
            for (int e = 0; e < kOnceRecords; ++e) {
                const int k = e * kLanes + lane;
                pk[h][e] = k < P[h].count ? S.pool_packed[(size_t)P[h].start + k] : 0u;
                v[h][e] = k < P[h].count ? S.pool_val[(size_t)P[h].start + k] : 0.0;
            }
#pragma unroll
        for (int h = 0; h < NUMBER; ++h) {
            const int col0 = (P[h].panel == S.g_c - 1 && S.m >= kPanel) ? S.m - kPanel : P[h].panel * kPanel;  // (as in scatter_kernel)
#pragma unroll
            for (int e = 0; e < kOnceRecords; ++e) {
                if (e * kLanes + lane >= P[h].count) break;
                const int at = min((int)(pk[h][e] >> 18) * S.g_c + P[h].panel, kOnceChunk - 1);
                const long long to = (long long)before + place[at] + (int)((pk[h][e] >> 9) & 511);
                if (to < S.capacity) {  // (always, without overflow)
                    S.col_idx[to] = col0 + (int)(pk[h][e] & 511);
                    S.val[to] = v[h][e];
                }
            }
        }
    };
    if (part == 0) {
        if (usual) {
            for (int q = w; q < fixed_runs; q += kFinSub) {
                if (q != w) R = runs[q];
                const Portion P{__builtin_amdgcn_readfirstlane(R.start), __builtin_amdgcn_readfirstlane(R.count), __builtin_amdgcn_readfirstlane(R.panel)};
                place_portions(std::integral_constant<int, 1>{}, &P);
            }
            return;
        }
        share_out();
    }
    // portions to the waves of the chunk's workgroups in turn; a wave has two of them under way
    const int waves = parts * kFinSub;
    for (int u = part * kFinSub + w; u < fixed_portions; u += 2 * waves) {
        const auto portion = [&](int of) {
            if (of >= fixed_portions) return Portion{0, 0, 0};
            const int from = __builtin_popcountll(__ballot(fixed_up_to <= of));
            const int k0 = (of - (from > 0 ? __builtin_amdgcn_readlane(fixed_up_to, from - 1) : 0)) * kOncePortion;
            return Portion{__builtin_amdgcn_readlane(fixed.start, from) + k0, __builtin_amdgcn_readlane(fixed.count, from) - k0,
                           __builtin_amdgcn_readlane(fixed.panel, from)};
        };
        const Portion P[2] = {portion(u), portion(u + waves)};
        place_portions(std::integral_constant<int, 2>{}, P);
    }
    for (int e0 = 0; e0 < extra; e0 += kOnceTable) {
        // the chunk's runs of this part of the list, one behind the other
        const PoolRange X = listed(tid < kOnceTable ? e0 + tid : extra);
        const uint64_t hits = __ballot(X.count > 0);
        __syncthreads();  // the ones before are placed
        if (lane == 0) lds_runs[w] = __builtin_popcountll(hits);
        __syncthreads();
        int found = 0, to = __builtin_popcountll(hits & ((1ull << lane) - 1));
#pragma unroll
        for (int q = 0; q < kFinSub; ++q) {
            to += q < w ? lds_runs[q] : 0;
            found += lds_runs[q];
        }
        if (X.count > 0) table[to] = X;
        __syncthreads();
        if (found == 0) continue;
        // the first portions of all runs, then the second ones, ..
        const int wave = (part * kFinSub + w + fixed_portions) % waves;
        int at = wave % found, level = wave / found;
        const auto next = [&] {
            Portion P{0, 0, 0};
            while (P.count <= 0 && level < kOnceRunPortions) {
                const int k0 = level * kOncePortion;
                P = Portion{__builtin_amdgcn_readfirstlane(table[at].start) + k0, __builtin_amdgcn_readfirstlane(table[at].count) - k0,
                            __builtin_amdgcn_readfirstlane(table[at].panel)};
                for (at += waves; at >= found && level < kOnceRunPortions; at -= found) ++level;
            }
            return P;
        };
        for (;;) {
            const Portion P[2] = {next(), next()};
            if (P[0].count <= 0) break;
            place_portions(std::integral_constant<int, 2>{}, P);
        }
    }
}

}  // namespace regot

#endif  // REGOT_FINISH_SMALL_HPP
