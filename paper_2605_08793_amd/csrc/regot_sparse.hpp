// Kernels on a stored sparsity pattern (Sec. 4.2: the pattern of the sparse term is kept for S
// iterations and only its values are recomputed) and for the sparse term H_Omega itself
// (Sec. 3.1, eq. (7)):
//
//   H_Omega = (1/eta) [ diag(T 1_m)          T^Omega_{-m}        ]     x = (x_alpha[n], x_beta[m-1])
//                     [ (T^Omega_{-m})^T     diag(T_{-m}^T 1_n)  ]
//
// The pattern is the CSR the sparsify calls produce (all m columns, ascending inside a row);
// "-m" drops the last column, so its entries are skipped here.  All of this is O(nnz) work on
// data that is a few MB: tiles of consecutive entries where every entry is for itself (values,
// lower triangle), one wave per row (or column) and lanes over the entries where rows are summed,
// in a fixed order (bit-reproducible), no floating-point atomics -- the product with the transposed
// block reads the pattern by columns, which regot_pattern_transpose prepares once per pattern.
#pragma once

#include "regot_device.hpp"

namespace regot {

constexpr int kRowsPerScanBlock = 32;  // rows per block in the prefix count of dropped entries: a bit each in half a word
static_assert(kLanes % kRowsPerScanBlock == 0, "row blocks");

struct PatternArgs {
    int n, m;
    int64_t ldM;
    const double *M;
    const double *alpha;
    const double *beta;
    const int64_t *row_ptr;
    const int32_t *col_idx;
    const int64_t *csc_pos;  // optional
    int64_t capacity;        // length of col_idx / val: no entry beyond it is touched
    double *val;
    double *val_csc;         // optional
    ExpParams ex;
};

// entries [p0, p1) of row i, clamped to the arrays
__device__ __forceinline__ void row_range(const int64_t *row_ptr, int64_t i, int64_t capacity, int64_t &p0, int64_t &p1)
{
    p0 = row_ptr[i];
    p1 = row_ptr[i + 1];
    if (p0 < 0) p0 = 0;
    if (p1 > capacity) p1 = capacity;
}

// Kernels that take the entries of a pattern in tiles of consecutive ones, whatever rows they are in: where the tile's rows
// begin is found by a wave-wide search, and an entry's row by bisection in LDS, for all entries of a thread side by side.
// ITEMS entries to a thread: kTileItems (four: 2e6 entries 67 + 12.3 us for values and triangle, 4e6 in all calls of a new pattern
// 332; with eight, fewer waves to wait side by side, 70 + 13.4 and 340), or kTileFew up to three small tiles to a compute unit
// (values by twos / by fours: 300000 entries 13.9 / 15.8 us, 360000 13.1 / 15.3, 400000 19.2 / 17.2, 500000 20.1 / 18.7, 2e6
// 76 / 74).
// A workgroup per 32 rows writes the triangle on a stored structure faster where rows are many and short and alike (20000 x 20000,
// 50000 entries 3.3 us against 4.3; 100000 x 50, 30000 entries 4.4 / 6.1; 40000 x 10000, 4e6 17.9 / 18.8), and slower elsewhere
// (20000 x 20000, 2e6 12.2 / 11.9, 4e6 20.9 / 18.6; 10000 x 10000, 10^6 10.6 / 7.5; 4e6 in a fifth of the rows 39 / 18; 20 rows of
// 4400 173 / 3.7).
constexpr int kTileItems = 4, kTileFew = 2;
constexpr int64_t kTileFewBelow = 768 * kTileFew * kThreads;
constexpr int kTileHeld = 8 * kThreads;  // rows whose ends are held (a power of two): all of a tile's, unless many have no entries
static_assert((kTileHeld & (kTileHeld - 1)) == 0 && (kThreads & (kThreads - 1)) == 0, "bisection by halves");
template <int ITEMS>
struct TileRows {
    static constexpr int kEntries = ITEMS * kThreads;
    // the rows of entries base + k * kThreads + thread, k < ITEMS, of those below base + count; by the whole workgroup
    __device__ __forceinline__ static void find(int *ends /* LDS [kTileHeld] */, const int64_t *ptr, int n, int64_t base, int count,
                                                int64_t (&row)[ITEMS])
    {
        const int tid = (int)threadIdx.x;
        const int64_t row0 = wave_first(1, n, tid & (kLanes - 1), [&](int64_t r) { return ptr[r] > base; }, kThreads / 2) - 1;
        // where the rows from row0 on end (up to half of the first ones before the tile, which saves a load to wait for)
        int held = 0, want = kThreads;
        do {
            for (; held < want; held += kThreads) {
                const int64_t r = row0 + 1 + held + tid;
                const int64_t e = r <= n ? ptr[r] - base : kEntries;
                ends[held + tid] = (int)(e < 0 ? 0 : e > kEntries ? kEntries : e);
            }
            want *= 2;
            __syncthreads();
        } while (held < kTileHeld && ends[held - 1] < count);
        // the first end behind the entry
        int at[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) at[k] = 0;
        for (int half = held / 2; half > 0; half >>= 1) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) at[k] += ends[at[k] + half - 1] <= k * kThreads + tid ? half : 0;
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) row[k] = row0 + at[k];
        if (ends[held - 1] < count) {  // (more rows than are held: many without entries)
            for (int k = 0; k < ITEMS; ++k) {
                int64_t lo = row0, hi = (int64_t)n - 1;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (ptr[mid + 1] > base + k * kThreads + tid) hi = mid;
                    else lo = mid + 1;
                }
                row[k] = lo;
            }
        }
    }
};

// tiles of a pattern with room for `capacity` entries -> the workgroups of a kernel that takes them in turn
template <int ITEMS>
inline int64_t tile_blocks(int64_t capacity, int64_t most)
{
    const int64_t tiles = die_grid((capacity + TileRows<ITEMS>::kEntries - 1) / TileRows<ITEMS>::kEntries);
    return tiles < most ? tiles : most;
}

// val[p] = T_{i, col_idx[p]}: a random 8-byte read of M per entry, everything of a tile requested at once.  Neighbouring tiles run
// on one die, so that the lines of val_csc that neighbouring rows share are put together; a die has its share of the entries, not
// of the rows, so it does not matter where they are.
// What bounds it: 64-byte sectors of M at random places and 8-byte stores at random places (2e6 of them 48 and 37 us, each by
// itself).  20000 x 20000, 2e6 entries: 101 -> 67 us; a wave per row waits for its row's range, columns and costs one after the
// other, and the longest rows are the last to be ready.  4e6 entries in rows of equal length 155 -> 142.
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void pattern_values_kernel(PatternArgs A)
{
    constexpr int kEntries = TileRows<ITEMS>::kEntries;
    __shared__ int ends[kTileHeld];
    const int tid = (int)threadIdx.x;
    int64_t first, nnz, unused;
    row_range(A.row_ptr, 0, A.capacity, first, unused);
    nnz = A.row_ptr[A.n];
    nnz = nnz < 0 ? 0 : nnz > A.capacity ? A.capacity : nnz;
    const int64_t blocks = (nnz + kEntries - 1) / kEntries;
    for (int64_t b = blockIdx.x; b < die_grid(blocks); b += gridDim.x) {
        const int64_t tile = die_block(b, blocks);
        if (tile >= blocks) continue;
        const int64_t base = tile * kEntries;
        const int count = (int)(nnz - base < kEntries ? nnz - base : kEntries);
        int32_t j[ITEMS];
        int64_t to[ITEMS], row[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int q = k * kThreads + tid;
            j[k] = q < count ? A.col_idx[base + q] : -1;
            to[k] = A.val_csc && q < count ? A.csc_pos[base + q] : -1;
        }
        TileRows<ITEMS>::find(ends, A.row_ptr, A.n, base, count, row);
        double mij[ITEMS], s[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            // (anything else is not a column, or in no row: the entry is left alone)
            if ((uint32_t)j[k] >= (uint32_t)A.m || base + k * kThreads + tid < first) j[k] = -1;
            const bool on = j[k] >= 0;
            mij[k] = on ? __builtin_nontemporal_load(A.M + row[k] * A.ldM + j[k]) : 0.0;
            s[k] = on ? A.alpha[row[k]] + A.beta[j[k]] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            if (j[k] < 0) continue;
            const double t = exp_eta_any(s[k] - mij[k], A.ex);
            A.val[base + k * kThreads + tid] = t;
            if (to[k] >= 0 && to[k] < A.capacity) A.val_csc[to[k]] = t;
        }
        __syncthreads();  // (the next tile's rows)
    }
}

// The same for a small pattern (few_rows): a wave takes a row, and what is beyond its first trip (kRowTrip entries) is left to the
// whole workgroup, whose rows lie far apart.  of_row(i): what is needed of row i;  body(that, p, end, stride): entries p,
// p + stride, .. below `end`, kRowDepth of them.
//
// Few entries are a matter of loads that wait for one another (a row's range, its columns, its costs), and a tile has two more of
// them, for its number of entries and its rows.  Values, and triangle on a stored structure, by rows / by tiles, us:
//   1000 x 1000    10000 entries  3.0 / 4.3   2.9 / 3.9        3000 x 3000  276000  10.5 / 12.5  3.4 / 5.1
//   1000 x 1000    95000          4.2 / 4.7   2.9 / 4.0        4000 x 4000  375000  15.8 / 14.3  3.6 / 5.3
//   1000 x 1000   330000         12.7 / 6.9   5.7 / 4.8        6000 x 6000   60000   4.6 /  5.3  3.6 / 4.0
//   2000 x 8000   180000          7.5 / 9.0   3.1 / 4.4        8000 x 8000   80000   5.7 /  5.3    -
// (8000 x 8000: a wave per row without the rest for the workgroup).  All entries in a fiftieth of the rows, 1577 to each: 7.4 / 5.0
// and 4.3 / 4.0, where a wave by itself takes 16 us; with columns to kRowsColumns a row is at most eight more trips.
constexpr int kRowsMost = 6144, kRowsColumns = 8192;           // rows and columns
constexpr int kRowsEntries = 96, kRowsAll = 1024 * kThreads;   // entries to a row, on average, and together
constexpr int kRowDepth = 4, kRowTrip = kRowDepth * kLanes;
inline bool few_rows(int64_t n, int64_t m, int64_t capacity)
{
    return n <= kRowsMost && m <= kRowsColumns && capacity <= kRowsEntries * n && capacity <= kRowsAll;
}
template <typename G, typename F>
__device__ __forceinline__ void for_rows(const int64_t *row_ptr, int64_t n, int64_t capacity, int blocks, G of_row, F body)
{
    __shared__ int64_t begin[kWaves], end[kWaves];
    const int tid = (int)threadIdx.x, lane = tid & (kLanes - 1), w = tid >> 6;
    const int64_t i = (int64_t)w * blocks + blockIdx.x;
    int64_t p0 = 0, p1 = 0;
    if (i < n) {
        row_range(row_ptr, i, capacity, p0, p1);
        body(of_row(i), p0 + lane, p1 < p0 + kRowTrip ? p1 : p0 + kRowTrip, kLanes);
    }
    const bool more = p1 > p0 + kRowTrip;
    if (lane == 0) {
        begin[w] = p0 + kRowTrip;
        end[w] = p1;
    }
    if (__syncthreads_or(more) == 0) return;
    for (int k = 0; k < kWaves; ++k) {
        const int64_t e = end[k];
        int64_t p = begin[k];
        if (p >= e) continue;
        const auto row = of_row((int64_t)k * blocks + blockIdx.x);
        for (; p < e; p += kRowDepth * kThreads) body(row, p + tid, e, kThreads);
    }
}

__global__ __launch_bounds__(kThreads) void pattern_values_rows_kernel(PatternArgs A)
{
    struct Row {
        double al;
        const double *M;
    };
    for_rows(
        A.row_ptr, A.n, A.capacity, (int)gridDim.x, [&](int64_t i) { return Row{A.alpha[i], A.M + i * A.ldM}; },
        [&](const Row &row, int64_t p, int64_t end, int stride) {
            int32_t j[kRowDepth];
            int64_t to[kRowDepth];
            double mij[kRowDepth], be[kRowDepth];
#pragma unroll
            for (int d = 0; d < kRowDepth; ++d) {
                const int64_t q = p + d * stride;
                j[d] = q < end ? A.col_idx[q] : -1;
                to[d] = A.val_csc && q < end ? A.csc_pos[q] : -1;
            }
#pragma unroll
            for (int d = 0; d < kRowDepth; ++d) {
                if ((uint32_t)j[d] >= (uint32_t)A.m) j[d] = -1;  // (not a column: the entry is left alone)
                mij[d] = j[d] >= 0 ? __builtin_nontemporal_load(row.M + j[d]) : 0.0;
                be[d] = j[d] >= 0 ? A.beta[j[d]] : 0.0;
            }
#pragma unroll
            for (int d = 0; d < kRowDepth; ++d) {
                if (j[d] < 0) continue;
                const double t = exp_eta_any((row.al + be[d]) - mij[d], A.ex);
                A.val[p + d * stride] = t;
                if (to[d] >= 0 && to[d] < A.capacity) A.val_csc[to[d]] = t;
            }
        });
}

struct MatvecArgs {
    int n, m;
    double eta, tau;
    const int64_t *row_ptr;
    const int32_t *col_idx;
    const double *val;
    const int64_t *col_ptr;
    const int32_t *row_idx;
    const double *val_csc;
    int64_t capacity;
    const double *row_sum;
    const double *col_sum;
    const double *x;
    double *y;
    int64_t row_waves;  // waves that take rows; the rest take columns
};

// R vectors side by side: element t of vector k sits at [t * R + k], so one gather fetches the entry of
// every vector (R = 1: a plain array; R = 2: pairs, 16 bytes).
template <int R>
struct Pack {
    double v[R];
};
template <int R>
__device__ __forceinline__ Pack<R> load_pack(const double *a, int64_t t)
{
    static_assert(R == 1 || R == 2, "one vector or a pair");
    Pack<R> q;
    if constexpr (R == 2) {
        const dbl2 w = *reinterpret_cast<const dbl2 *>(a + 2 * t);
        q.v[0] = w.x;
        q.v[1] = w.y;
    } else {
        q.v[0] = a[t];
    }
    return q;
}
template <int R>
__device__ __forceinline__ void store_pack(double *a, int64_t t, const Pack<R> &q)
{
    if constexpr (R == 2) {
        *reinterpret_cast<dbl2 *>(a + 2 * t) = dbl2{q.v[0], q.v[1]};
    } else {
        a[t] = q.v[0];
    }
}

// This lane's share of sum_p val[p] * x[idx[p]] over entries [p0, p1) with idx[p] < limit.  Four
// entries per lane are loaded before the first is used: the longest rows (ten times the average)
// set the duration of the kernel, and their trips would otherwise each wait for a full memory latency.
template <int R>
__device__ __forceinline__ Pack<R> gather_dot(const int32_t *idx, const double *val, const double *x, int limit,
                                              int64_t p0, int64_t p1, int lane)
{
    constexpr int kDepth = 4;
    Pack<R> s;
#pragma unroll
    for (int k = 0; k < R; ++k) s.v[k] = 0.0;
    for (int64_t p = p0 + lane; p < p1; p += kDepth * kLanes) {
        int32_t j[kDepth];
        double v[kDepth];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            const int64_t q = p + d * kLanes;
            j[d] = q < p1 ? idx[q] : -1;
            v[d] = q < p1 ? val[q] : 0.0;
        }
        Pack<R> xv[kDepth];
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            if ((uint32_t)j[d] < (uint32_t)limit) {
                xv[d] = load_pack<R>(x, j[d]);
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) xv[d].v[k] = 0.0;
            }
        }
#pragma unroll
        for (int d = 0; d < kDepth; ++d)
#pragma unroll
            for (int k = 0; k < R; ++k) s.v[k] += v[d] * xv[d].v[k];
    }
    return s;
}

// NR rows (or columns) at once, for the product inside the iteration: the loads of all NR rows go out before the
// first value is used, so a wave waits for one memory latency per NR rows instead of per row.  Row r covers
// entries [p0[r], p1[r]); per row the operations and their order are those of gather_dot, hence the same bits
// (trips beyond a row's end add +0, which changes nothing).  The first `nl` entries of x are read from a copy in LDS
// (`xl`), the others from memory; ALL: every index below `limit` is in xl.
template <int R, int NR, bool ALL>
__device__ __forceinline__ void gather_dot_rows(const int32_t *idx, const double *val, const double *x, const double *xl,
                                                int nl, int limit, const int64_t (&p0)[NR], const int64_t (&p1)[NR],
                                                int lane, Pack<R> (&s)[NR])
{
    constexpr int kDepth = 4;
    int longest = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
#pragma unroll
        for (int k = 0; k < R; ++k) s[r].v[k] = 0.0;
        const int len = __builtin_amdgcn_readfirstlane((int)(p1[r] - p0[r]));
        longest = len > longest ? len : longest;
    }
    for (int t = 0; t < longest; t += kDepth * kLanes) {
        int32_t j[NR][kDepth];
        double v[NR][kDepth];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                const int64_t q = p0[r] + t + d * kLanes + lane;
                j[r][d] = q < p1[r] ? idx[q] : -1;
                v[r][d] = q < p1[r] ? val[q] : 0.0;
            }
        Pack<R> xv[NR][kDepth];
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (ALL ? (uint32_t)j[r][d] < (uint32_t)limit : (uint32_t)j[r][d] < (uint32_t)nl) {
                    xv[r][d] = load_pack<R>(xl, j[r][d]);
                } else if (!ALL && (uint32_t)j[r][d] < (uint32_t)limit) {
                    xv[r][d] = load_pack<R>(x, j[r][d]);
                } else {
#pragma unroll
                    for (int k = 0; k < R; ++k) xv[r][d].v[k] = 0.0;
                }
            }
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int d = 0; d < kDepth; ++d)
#pragma unroll
                for (int k = 0; k < R; ++k) s[r].v[k] += v[r][d] * xv[r][d].v[k];
    }
}

// y = (H_Omega + tau I) x.  Waves [0, row_waves) take the alpha block row by row from the CSR, the others
// the beta block column by column from the pattern by columns; one wave per row or column where the grid
// allows.  (The call on its own; the conjugate-gradient iteration uses hessian_matvec_lds_kernel.)
__global__ __launch_bounds__(kThreads) void hessian_matvec_kernel(MatvecArgs A)
{
    const int lane = threadIdx.x & (kLanes - 1);
    const int64_t wave = (int64_t)blockIdx.x * kWaves + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * kWaves;
    const int mb = A.m - 1;  // beta variables
    const double inv_eta = 1.0 / A.eta;
    if (wave < A.row_waves) {
        for (int64_t i = wave; i < A.n; i += A.row_waves) {
            int64_t p0, p1;
            row_range(A.row_ptr, i, A.capacity, p0, p1);
            const double s = wave_reduce1<OpSum>(gather_dot<1>(A.col_idx, A.val, A.x + A.n, mb, p0, p1, lane).v[0]);
            if (lane == 0) A.y[i] = (A.row_sum[i] * A.x[i] + s) * inv_eta + A.tau * A.x[i];
        }
    } else {
        const int64_t col_waves = nwaves - A.row_waves;
        for (int64_t j = wave - A.row_waves; j < mb; j += col_waves) {
            int64_t q0, q1;
            row_range(A.col_ptr, j, A.capacity, q0, q1);
            const double s = wave_reduce1<OpSum>(gather_dot<1>(A.row_idx, A.val_csc, A.x, A.n, q0, q1, lane).v[0]);
            if (lane == 0) A.y[A.n + j] = (A.col_sum[j] * A.x[A.n + j] + s) * inv_eta + A.tau * A.x[A.n + j];
        }
    }
}

// The product inside the conjugate-gradient iteration, for R vectors at once (x, y: R vectors side by side,
// see Pack), with the half of x that is gathered kept in LDS: workgroups of 16 waves, one per compute unit;
// the first row_blocks of them take the alpha block (they hold x's beta half, m - 1 entries), the others the
// beta block (they hold the alpha half, n entries).  What bounds the kernel above is not the bytes of the
// pattern but the gathers of x, each of which moves a cache line from L2 to a first-level cache far smaller
// than the vector; from LDS a gather costs a few cycles.  When a half has more than kMatvecLdsCap / R
// entries only its first entries are kept and the gathers of the others go to memory.
// The result does not depend on R or on what is kept in LDS: a row is summed by the same lanes in the same
// order as in the kernel above, wave W of the grid takes rows W, W + row waves, ..., and the workgroup writes
// its share of x_k^T y_k (for p^T A p) per group of kWaves waves to dot_part[k * dot_stride + ...], each the
// sum of its waves' shares in wave order.  Does nothing at all if *skip is set.
constexpr int kMatvecLdsCap = 20000;
constexpr int kMatvecLdsWaves = 16;
constexpr int kMatvecLdsThreads = kMatvecLdsWaves * kLanes;
constexpr int kMatvecRows = 2;                             // rows (columns) a wave has in flight
constexpr int kMatvecLdsGroup = kMatvecLdsWaves / kWaves;  // workgroups of the other kernel per workgroup of this one
static_assert(kMatvecLdsWaves % kWaves == 0, "whole workgroups of the other kernel");

// the first xlen doubles of src -> LDS; all loads of a thread go out before the first value is stored
// (16 bytes per load where src allows it)
__device__ __forceinline__ void lds_fill(double *xs, const double *src, int xlen)
{
    if ((reinterpret_cast<uintptr_t>(src) & 15) == 0) {
        constexpr int kPer = (kMatvecLdsCap / 2 + kMatvecLdsThreads - 1) / kMatvecLdsThreads;
        const int pairs = xlen / 2;
        dbl2 t[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = j * kMatvecLdsThreads + (int)threadIdx.x;
            t[j] = i < pairs ? reinterpret_cast<const dbl2 *>(src)[i] : dbl2{0.0, 0.0};
        }
        double last = 0.0;
        if ((xlen & 1) && threadIdx.x == 0) last = src[xlen - 1];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int i = j * kMatvecLdsThreads + (int)threadIdx.x;
            if (i < pairs) reinterpret_cast<dbl2 *>(xs)[i] = t[j];
        }
        if ((xlen & 1) && threadIdx.x == 0) xs[xlen - 1] = last;
        return;
    }
    constexpr int kPer = (kMatvecLdsCap + kMatvecLdsThreads - 1) / kMatvecLdsThreads;
    double t[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kMatvecLdsThreads + (int)threadIdx.x;
        t[j] = i < xlen ? src[i] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int i = j * kMatvecLdsThreads + (int)threadIdx.x;
        if (i < xlen) xs[i] = t[j];
    }
}

// One sweep of a wave over its items (rows of a CSR block or columns of the pattern by columns): items first,
// first + stride, ... below count.  A wave takes its items in batches of 64, lane l holding everything about item
// b0 + l * stride that one load can fetch (its range of entries and whatever `item.fetch` asks for), so the only
// memory latency left per group of kMatvecRows items is that of the entries themselves; the sums
// sum_p val[p] x[idx[p]] of an item are formed by the whole wave (gather_dot_rows), lane l keeps item l's and
// `item.finish` turns it into the item's result, stores it and returns the item's term of an inner product (or 0);
// dot[] (the same in every lane) grows by these terms item by item in ascending order.
//   Item: void fetch(int64_t t);  Pack<R> finish(int64_t t, bool have, const Pack<R> &sum)
// (the loads of a batch's first part: the kernels ask for those of their first batch before they fill the LDS)
struct SweepHead {
    int64_t q0, q1;
};
template <typename Item>
__device__ __forceinline__ SweepHead lds_sweep_head(const int64_t *ptr, int64_t capacity, int64_t count, int64_t b0,
                                                    int64_t stride, int lane, Item &item)
{
    SweepHead h{0, 0};
    const int64_t mine = b0 + lane * stride;
    if (mine < count) {
        row_range(ptr, mine, capacity, h.q0, h.q1);
        item.fetch(mine);
    }
    return h;
}

template <int R, bool ALL, typename Item>
__device__ __forceinline__ void lds_sweep(const int64_t *ptr, const int32_t *idx, const double *val, int64_t capacity,
                                          const double *xsrc, const double *xs, int nl, int limit, int64_t count,
                                          int64_t first, int64_t stride, int lane, Item &item, double (&dot)[R],
                                          SweepHead head /* of the batch at `first` */)
{
    for (int64_t b0 = first; b0 < count; b0 += kLanes * stride) {
        const int64_t mine = b0 + lane * stride;
        const bool have = mine < count;
        if (b0 != first) head = lds_sweep_head(ptr, capacity, count, b0, stride, lane, item);
        const int64_t q0 = head.q0, q1 = head.q1;
        Pack<R> sum;
#pragma unroll
        for (int k = 0; k < R; ++k) sum.v[k] = 0.0;
        const int64_t left = (count - b0 + stride - 1) / stride;
        const int items = __builtin_amdgcn_readfirstlane((int)(left < kLanes ? left : kLanes));
        for (int r0 = 0; r0 < items; r0 += kMatvecRows) {
            int64_t p0[kMatvecRows], p1[kMatvecRows];
#pragma unroll
            for (int r = 0; r < kMatvecRows; ++r) {
                const int src = r0 + r < items ? r0 + r : r0;  // (a surplus slot repeats item r0 with an empty range)
                p0[r] = read_lane_i64(q0, src);
                p1[r] = r0 + r < items ? read_lane_i64(q1, src) : p0[r];
            }
            Pack<R> s[kMatvecRows];
            gather_dot_rows<R, kMatvecRows, ALL>(idx, val, xsrc, xs, nl, limit, p0, p1, lane, s);
#pragma unroll
            for (int r = 0; r < kMatvecRows; ++r)
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    const double t = wave_reduce1<OpSum>(s[r].v[k]);
                    if (lane == r0 + r) sum.v[k] = t;
                }
        }
        const Pack<R> term = item.finish(mine, have, sum);
        for (int r = 0; r < items; ++r)
#pragma unroll
            for (int k = 0; k < R; ++k) dot[k] += read_lane(term.v[k], r);
    }
}

// the waves' shares of an inner product -> one partial sum per group of kWaves waves, added up in wave order
// (the order block_sum uses): dot_part[k * dot_stride + blockIdx.x * kMatvecLdsGroup + g]
template <int R>
__device__ __forceinline__ void lds_leave_dots(const double (&dot)[R], double (*wave_dot)[kMatvecLdsWaves],
                                               double *dot_part, int dot_stride, int lane, int w)
{
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (lane == 0) wave_dot[k][w] = dot[k];
    __syncthreads();
    if (threadIdx.x < kMatvecLdsGroup) {
        const int g = threadIdx.x;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            double r = wave_dot[k][g * kWaves];
#pragma unroll
            for (int q = 1; q < kWaves; ++q) r += wave_dot[k][g * kWaves + q];
            dot_part[(size_t)k * dot_stride + (size_t)blockIdx.x * kMatvecLdsGroup + g] = r;
        }
    }
}

// item of the full product: y_t = (diag_t x_t + sum) / eta + tau x_t, and its term x_t y_t of x^T y
template <int R>
struct ProductItem {
    const double *diag;   // row or column sums of the plan
    const double *x;      // the vector(s), offset to this half
    double *y;
    double inv_eta, tau;
    double dg;
    Pack<R> xt;
    __device__ __forceinline__ void fetch(int64_t t)
    {
        dg = diag[t];
        xt = load_pack<R>(x, t);
    }
    __device__ __forceinline__ Pack<R> finish(int64_t t, bool have, const Pack<R> &sum)
    {
        Pack<R> yt, term;
#pragma unroll
        for (int k = 0; k < R; ++k) {
            yt.v[k] = have ? (dg * xt.v[k] + sum.v[k]) * inv_eta + tau * xt.v[k] : 0.0;
            term.v[k] = have ? yt.v[k] * xt.v[k] : 0.0;
        }
        if (have) store_pack<R>(y, t, yt);
        return term;
    }
};

// ALL: both halves fit entirely (the host has checked), so no gather needs the test for where its entry is.
template <bool DOT, int R, bool ALL>
__global__ __launch_bounds__(kMatvecLdsThreads) void hessian_matvec_lds_kernel(MatvecArgs A, double *dot_part,
                                                                               int dot_stride, const int *skip,
                                                                               int row_blocks)
{
    __shared__ __attribute__((aligned(16))) double xs[kMatvecLdsCap];
    __shared__ double wave_dot[R][kMatvecLdsWaves];
    static_assert(sizeof(double) * (kMatvecLdsCap + R * kMatvecLdsWaves) <= 160 * 1024, "LDS per CU");
    if (DOT && *skip) return;
    const int lane = threadIdx.x & (kLanes - 1), w = threadIdx.x >> 6;
    const int mb = A.m - 1;  // beta variables
    const bool rows = (int)blockIdx.x < row_blocks;
    const double *xsrc = rows ? A.x + (int64_t)A.n * R : A.x;
    const int limit = rows ? mb : A.n;                                         // entries the gathers may ask for
    const int nl = limit < kMatvecLdsCap / R ? limit : kMatvecLdsCap / R;      // of which the first nl sit in LDS
    double dot[R];  // the wave's share of x^T y (the same in every lane)
#pragma unroll
    for (int k = 0; k < R; ++k) dot[k] = 0.0;
    ProductItem<R> item;
    item.inv_eta = 1.0 / A.eta;
    item.tau = A.tau;
    item.diag = rows ? A.row_sum : A.col_sum;
    item.x = rows ? A.x : A.x + (int64_t)A.n * R;
    item.y = rows ? A.y : A.y + (int64_t)A.n * R;
    const int64_t *ptr = rows ? A.row_ptr : A.col_ptr;
    const int64_t count = rows ? A.n : mb;
    const int64_t first = (int64_t)(rows ? (int)blockIdx.x : (int)blockIdx.x - row_blocks) * kMatvecLdsWaves + w;
    const int64_t stride = (int64_t)(rows ? row_blocks : (int)gridDim.x - row_blocks) * kMatvecLdsWaves;
    const SweepHead head = lds_sweep_head(ptr, A.capacity, count, first, stride, lane, item);
    lds_fill(xs, xsrc, nl * R);
    __syncthreads();
    lds_sweep<R, ALL>(ptr, rows ? A.col_idx : A.row_idx, rows ? A.val : A.val_csc, A.capacity, xsrc, xs, nl, limit, count,
                      first, stride, lane, item, dot, head);
    if constexpr (DOT) lds_leave_dots<R>(dot, wave_dot, dot_part, dot_stride, lane, w);
}

struct LowerArgs {
    int n, m;
    double eta, tau;
    const int64_t *row_ptr;
    const int32_t *col_idx;
    const double *val;
    int64_t capacity;
    const double *row_sum;
    const double *col_sum;
    int64_t *h_col_ptr;   // [n + m]
    int32_t *h_row_idx;
    double *h_val;
    int64_t h_capacity;
    int64_t *info;        // [2]: entries, overflow
    int64_t *blk;         // [nblk + 1] workspace: dropped entries in the blocks of rows before << 32 | a bit per row of the block
    int nblk;
    int values_only;
};

// does row i end with an entry in the dropped column (columns ascend, so it can only be the last one)
__device__ __forceinline__ int row_drops(const LowerArgs &A, int64_t i)
{
    int64_t p0, p1;
    row_range(A.row_ptr, i, A.capacity, p0, p1);
    return (p1 > p0 && A.col_idx[p1 - 1] == A.m - 1) ? 1 : 0;
}

// step 1: which rows of a block of kRowsPerScanBlock drop an entry; a thread per row, half a wave per block
__global__ __launch_bounds__(kThreads) void lower_count_kernel(LowerArgs A)
{
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const uint64_t drops = __ballot(i < A.n && row_drops(A, i));
    const int64_t rb = i / kRowsPerScanBlock;
    if ((threadIdx.x & (kRowsPerScanBlock - 1)) == 0 && rb < A.nblk)
        A.blk[rb] = (int64_t)(uint32_t)(drops >> (threadIdx.x & kRowsPerScanBlock & (kLanes - 1)));
}

// step 2: exclusive prefix over the blocks (one workgroup); all dropped entries in blk[nblk]
__global__ __launch_bounds__(kThreads) void lower_scan_kernel(LowerArgs A)
{
    __shared__ int wave_total[kWaves];
    constexpr int kPer = 4;  // blocks of a thread, asked for together
    const int lane = threadIdx.x & (kLanes - 1), w = threadIdx.x >> 6;
    int64_t carry = 0;
    for (int64_t first = 0; first < A.nblk; first += kPer * kThreads) {
        const int64_t b0 = first + (int64_t)threadIdx.x * kPer;
        uint32_t bits[kPer];
        int mine = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) bits[k] = b0 + k < A.nblk ? (uint32_t)A.blk[b0 + k] : 0u;
#pragma unroll
        for (int k = 0; k < kPer; ++k) mine += __builtin_popcount(bits[k]);
        const int incl = wave_scan(mine);
        if (lane == kLanes - 1) wave_total[w] = incl;
        __syncthreads();
        int before = incl - mine, all = 0;
#pragma unroll
        for (int q = 0; q < kWaves; ++q) {
            before += q < w ? wave_total[q] : 0;
            all += wave_total[q];
        }
        int64_t run = carry + before;
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (b0 + k < A.nblk) {
                A.blk[b0 + k] = run << 32 | bits[k];
                run += __builtin_popcount(bits[k]);
            }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) A.blk[A.nblk] = carry;
}

// entries dropped in the rows before row i
__device__ __forceinline__ int64_t dropped_before(const LowerArgs &A, int64_t i)
{
    const int64_t b = A.blk[i / kRowsPerScanBlock];
    return (b >> 32) + __builtin_popcount((uint32_t)b & ((1u << (i & (kRowsPerScanBlock - 1))) - 1u));
}

// step 3: column i < n of the lower triangle = diagonal, then row i of T^Omega_{-m} as rows n + j; columns n + j hold their
// diagonal only.  i diagonals and row_ptr[i] pattern entries come before column i, minus the dropped ones.  The first
// workgroups take tiles of consecutive pattern entries (TileRows); the others a column's beginning and its diagonal per
// thread.  2e6 entries 24 -> 12.3 us (48 MB read and written), 4e6 25.5 -> 22: a workgroup per 32 rows was ready when the
// longest 32 rows were.
// ITEMS 0: the entries by rows (for_rows).
template <int ITEMS>
__global__ __launch_bounds__(kThreads) void lower_fill_kernel(LowerArgs A, int entry_blocks)
{
    const int tid = (int)threadIdx.x;
    const int mb = A.m - 1;
    const double inv_eta = 1.0 / A.eta;
    int64_t first, pn, unused;
    row_range(A.row_ptr, 0, A.capacity, first, unused);
    pn = A.row_ptr[A.n];
    pn = pn < 0 ? 0 : pn > A.capacity ? A.capacity : pn;
    if constexpr (ITEMS == 0) {
        if ((int)blockIdx.x < entry_blocks) {
            for_rows(
                A.row_ptr, A.n, A.capacity, entry_blocks,
                [&](int64_t i) {  // place of entry p: that + p
                    int64_t p0, p1;
                    row_range(A.row_ptr, i, A.capacity, p0, p1);
                    return (A.values_only ? A.h_col_ptr[i] - p0 : i - dropped_before(A, i)) + 1;
                },
                [&](int64_t place, int64_t p, int64_t end, int stride) {
                    int32_t j[kRowDepth];
                    double v[kRowDepth];
#pragma unroll
                    for (int d = 0; d < kRowDepth; ++d) {
                        j[d] = p + d * stride < end ? A.col_idx[p + d * stride] : -1;
                        v[d] = p + d * stride < end ? A.val[p + d * stride] : 0.0;
                    }
#pragma unroll
                    for (int d = 0; d < kRowDepth; ++d) {
                        const int64_t q = place + p + d * stride;
                        if ((uint32_t)j[d] < (uint32_t)mb && q >= 0 && q < A.h_capacity) {
                            if (!A.values_only) A.h_row_idx[q] = A.n + j[d];
                            A.h_val[q] = v[d] * inv_eta;
                        }
                    }
                });
            return;
        }
    } else if ((int)blockIdx.x < entry_blocks) {
        constexpr int kEntries = TileRows<ITEMS>::kEntries;
        __shared__ int ends[kTileHeld];
        const int64_t blocks = (pn + kEntries - 1) / kEntries;
        for (int64_t b = blockIdx.x; b < die_grid(blocks); b += entry_blocks) {
            const int64_t tile = die_block(b, blocks);
            if (tile >= blocks) continue;
            const int64_t base = tile * kEntries;
            const int count = (int)(pn - base < kEntries ? pn - base : kEntries);
            int32_t j[ITEMS];
            double v[ITEMS];
            int64_t row[ITEMS], place[ITEMS];
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int q = k * kThreads + tid;
                j[k] = q < count ? A.col_idx[base + q] : -1;
                v[k] = q < count ? A.val[base + q] : 0.0;
            }
            TileRows<ITEMS>::find(ends, A.row_ptr, A.n, base, count, row);
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int64_t p = base + k * kThreads + tid;
                place[k] = -1;
                if ((uint32_t)j[k] >= (uint32_t)mb || p < first) continue;
                if (A.values_only) {
                    int64_t p0, p1;
                    row_range(A.row_ptr, row[k], A.capacity, p0, p1);
                    place[k] = A.h_col_ptr[row[k]] - p0 + p + 1;
                } else {
                    place[k] = row[k] - dropped_before(A, row[k]) + p + 1;
                }
            }
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int64_t q = place[k];
                if (q >= 0 && q < A.h_capacity) {
                    if (!A.values_only) A.h_row_idx[q] = A.n + j[k];
                    A.h_val[q] = v[k] * inv_eta;
                }
            }
            __syncthreads();  // (the next tile's rows)
        }
        return;
    }
    // total entries: n + (m-1) diagonals + pattern entries outside the dropped column
    const int64_t first_beta = A.values_only ? A.h_col_ptr[A.n + mb] - mb : (int64_t)A.n + pn - A.blk[A.nblk];
    const int64_t c = ((int64_t)blockIdx.x - entry_blocks) * kThreads + tid;
    if (c < A.n) {
        int64_t p = A.row_ptr[c];
        p = p < 0 ? 0 : p > A.capacity ? A.capacity : p;
        const int64_t q = A.values_only ? A.h_col_ptr[c] : c + p - dropped_before(A, c);
        if (!A.values_only) A.h_col_ptr[c] = q;
        if (q >= 0 && q < A.h_capacity) {
            if (!A.values_only) A.h_row_idx[q] = (int32_t)c;
            A.h_val[q] = A.row_sum[c] * inv_eta + A.tau;
        }
    } else if (c < (int64_t)A.n + mb) {
        const int64_t q = first_beta + (c - A.n);
        if (!A.values_only) A.h_col_ptr[c] = q;
        if (q >= 0 && q < A.h_capacity) {
            if (!A.values_only) A.h_row_idx[q] = (int32_t)c;
            A.h_val[q] = A.col_sum[c - A.n] * inv_eta + A.tau;
        }
    }
    if (c == 0) {
        const int64_t total = first_beta + mb;
        if (!A.values_only) A.h_col_ptr[A.n + mb] = total;
        A.info[0] = total;
        A.info[1] = total > A.h_capacity ? 1 : 0;
    }
}

// ---------------------------------------------------------------------------------------------
// Optimality measures of a dual point from its row and column sums (App. A.5), and the choice
// between two candidate iterates (Sec. 4.3).
// ---------------------------------------------------------------------------------------------

constexpr int kMetricParts = 256;   // workgroups of the first stage
constexpr int kMetricSums = 5;

struct MetricArgs {
    int64_t n, m;
    const double *a, *b, *alpha, *beta, *row_sum, *col_sum;
    double eta;
    double *part;     // [kMetricParts][kMetricSums]
    double *metrics;  // [4]: L_p, L_p - L_d, marginal error, || grad f ||_2
    int parts;
};

// sums over a slice of the n + m entries: alpha^T r + beta^T c, alpha^T (r - a) + beta^T (c - b),
// sum r, sum |r - a| + sum |c - b|, sum (r - a)^2 + sum_{j < m-1} (c - b)^2
__global__ __launch_bounds__(kThreads) void metric_parts_kernel(MetricArgs A)
{
    __shared__ double wsum[kWaves][kMetricSums];
    double s[kMetricSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
    const int64_t total = A.n + A.m;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        const bool row = t < A.n;
        const int64_t k = row ? t : t - A.n;
        const double dual = row ? A.alpha[k] : A.beta[k];
        const double sum = row ? A.row_sum[k] : A.col_sum[k];
        const double d = sum - (row ? A.a[k] : A.b[k]);
        s[0] += dual * sum;
        s[1] += dual * d;
        if (row) s[2] += sum;
        s[3] += fabs(d);
        if (row || k < A.m - 1) s[4] += d * d;
    }
#pragma unroll
    for (int e = 0; e < kMetricSums; ++e) s[e] = wave_reduce1<OpSum>(s[e]);
    if ((threadIdx.x & (kLanes - 1)) == 0)
        for (int e = 0; e < kMetricSums; ++e) wsum[threadIdx.x >> 6][e] = s[e];
    __syncthreads();
    if (threadIdx.x < kMetricSums) {
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += wsum[w][threadIdx.x];
        A.part[(size_t)blockIdx.x * kMetricSums + threadIdx.x] = v;
    }
}

__global__ void metric_final_kernel(MetricArgs A)
{
    if (threadIdx.x != 0) return;
    double s[kMetricSums] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int p = 0; p < A.parts; ++p)
        for (int e = 0; e < kMetricSums; ++e) s[e] += A.part[(size_t)p * kMetricSums + e];
    // L_p = <T, M> + eta sum T log T - eta sum T = sum_ij T_ij (alpha_i + beta_j) - eta sum T
    A.metrics[0] = s[0] - A.eta * s[2];
    A.metrics[1] = s[1];
    A.metrics[2] = s[3];
    A.metrics[3] = sqrt(s[4]);
}

struct ChooseArgs {
    int64_t n, m;
    const double *obj_q, *obj_s;
    const double *alpha_q, *beta_q, *alpha_s, *beta_s;
    double *alpha_out, *beta_out;
    int64_t *choice;
};

// keep the candidate with the larger dual objective (the quasi-Newton one unless the other is strictly better)
__global__ __launch_bounds__(kThreads) void choose_candidate_kernel(ChooseArgs A)
{
    const bool take_s = A.obj_s[0] > A.obj_q[0];
    const double *al = take_s ? A.alpha_s : A.alpha_q;
    const double *be = take_s ? A.beta_s : A.beta_q;
    const int64_t total = A.n + A.m;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        if (t < A.n) A.alpha_out[t] = al[t];
        else A.beta_out[t - A.n] = be[t - A.n];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) A.choice[0] = take_s ? 1 : 0;
}

}  // namespace regot
