// regot_pattern_transpose: the sparsity pattern by columns (symbolic work, once per pattern;
// Sec. 4.2 keeps a pattern for S iterations; the transposed block of H_Omega in Sec. 3.1 eq. (7) reads
// it).  The interface is documented in include/regot.h.
//
// The pattern by columns is the list of CSR positions p sorted by (column, p): CSR positions grow with
// the row and a column holds at most one entry per row, so inside a column ascending p is ascending row.
// There are two ways to it; by_counting says which one a pattern takes, and the text there why.
// Counting, for patterns that are not too sparse, is described further down, at its kernels.  The other:
// the positions start out in ascending order, so a STABLE sort by column alone gives that list: a
// least-significant-digit radix sort on the column index, 8 bits per pass, ceil(bits(m) / 8) passes (two
// for m < 65536):
//   0. entry_row[p] = row of CSR position p (one wave per row; in the launch of the first pass's step 1);
//   per pass:
//   1. every workgroup counts the digits of its tile of 2048 keys (LDS) -> table[digit][workgroup];
//   2. one workgroup per digit: exclusive scan of its row of the table, and the digit's total;
//   3. every workgroup ranks its keys stably (a wave takes 64 consecutive keys at a time; lanes with the
//      same digit find each other with eight ballots and rank by lane number behind the keys of that
//      digit the wave has already seen), orders the tile by digit in LDS and writes each digit's run to
//      its place: the digit's base + the table entry + the position inside the run; the last pass knows
//      where in the column order that is and writes row_idx[q] and csc_pos[p] = q instead of another list;
//   then, on the sorted columns:
//   4. col_ptr[j] = number of keys below j (a binary search per column).
// A col_idx outside [0, m) sorts as column m, behind every real column, and gets csc_pos = -1.
// Either way there are no atomics on memory and no order that depends on timing: the same bits on every call.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "regot.h"
#include "regot_device.hpp"

namespace {

using namespace regot;

constexpr int64_t kMaxDim = 2147483647LL;
constexpr size_t kAlign = 256;
constexpr int kBlock = 256;
constexpr int kWavesPerBlock = kBlock / kLanes;
constexpr int kItems = 8;                        // keys per thread
constexpr int kTile = kBlock * kItems;           // keys per workgroup
constexpr int kWaveKeys = kTile / kWavesPerBlock;  // consecutive keys a wave ranks
constexpr int kDigitBits = 8;
constexpr int kDigits = 1 << kDigitBits;
static_assert(kDigits == kBlock, "one thread per digit");
static_assert(kWaveKeys == kItems * kLanes, "a wave ranks kItems groups of 64 keys");

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
bool misaligned(const void *p, size_t a) { return ((uintptr_t)p % a) != 0; }

struct TransposeLayout {
    size_t table, digit_total, entry_row, key[2], pay[2];
    int64_t blocks;
    int passes;
    size_t total;
};

TransposeLayout make_transpose_layout(int64_t m, int64_t nnz)
{
    TransposeLayout L{};
    const size_t e = (size_t)(nnz > 0 ? nnz : 1);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = align_up(off + bytes);
        return at;
    };
    L.blocks = (int64_t)((e + kTile - 1) / kTile);
    int bits = 0;  // keys are 0 .. m
    while (bits < 32 && ((uint64_t)m >> bits) != 0) ++bits;
    L.passes = bits <= kDigitBits ? 1 : (bits + kDigitBits - 1) / kDigitBits;
    L.table = take((size_t)kDigits * (size_t)L.blocks * sizeof(uint32_t));
    L.digit_total = take(kDigits * sizeof(uint32_t));
    L.entry_row = take(e * sizeof(int32_t));
    for (int k = 0; k < 2; ++k) {
        L.key[k] = take(e * sizeof(uint32_t));
        L.pay[k] = take(e * sizeof(uint32_t));
    }
    L.total = off;
    return L;
}

struct TransposeArgs {
    int64_t n, m, nnz;
    const int64_t *row_ptr;
    const int32_t *col_idx;
    int64_t *col_ptr;
    int32_t *row_idx;
    int64_t *csc_pos;
    uint32_t *table;        // [kDigits][blocks]
    uint32_t *digit_total;  // [kDigits]
    int32_t *entry_row;     // [nnz]
    int64_t blocks;
};

// one pass of the sort: FIRST reads the keys from col_idx (positions are the payload), else from key_in / pay_in
struct PassArgs {
    const uint32_t *key_in, *pay_in;
    uint32_t *key_out, *pay_out;
    const int32_t *row_in;
    int32_t *row_out;
    int shift;
};

__device__ __forceinline__ uint32_t column_key(const TransposeArgs &A, int64_t p)
{
    const int64_t j = A.col_idx[p];
    return (uint32_t)(j >= 0 && j < A.m ? j : A.m);
}

template <bool FIRST>
__device__ __forceinline__ uint32_t load_key(const TransposeArgs &A, const PassArgs &P, int64_t i)
{
    return FIRST ? column_key(A, i) : P.key_in[i];
}

// Neighbouring tiles run on one die (die_block): a digit's run of a tile, a count or a position is written next to those of the
// tiles around it.  (With 2e6 entries a new pattern with its values and lower triangle took 257 us instead of 291, a third of the
// difference here; it takes 175 now.)

// step 1; behind the tiles' workgroups of the first pass, step 0: one wave per row
template <bool FIRST>
__global__ __launch_bounds__(kBlock) void digit_count_kernel(TransposeArgs A, PassArgs P)
{
    __shared__ unsigned hist[kDigits];
    const int64_t tiles = die_grid(A.blocks);
    if (FIRST && (int64_t)blockIdx.x >= tiles) {
        const int lane = threadIdx.x & (kLanes - 1);
        const int64_t wave = ((int64_t)blockIdx.x - tiles) * kWavesPerBlock + (threadIdx.x >> 6);
        for (int64_t i = wave; i < A.n; i += ((int64_t)gridDim.x - tiles) * kWavesPerBlock) {
            int64_t p0 = A.row_ptr[i], p1 = A.row_ptr[i + 1];
            if (p0 < 0) p0 = 0;
            if (p1 > A.nnz) p1 = A.nnz;
            for (int64_t p = p0 + lane; p < p1; p += kLanes) A.entry_row[p] = (int32_t)i;
        }
        return;
    }
    const int64_t tile = die_block(blockIdx.x, A.blocks);
    if (tile >= A.blocks) return;
    hist[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = tile * kTile;
    uint32_t key[kItems];
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int64_t i = base + k * kBlock + threadIdx.x;
        key[k] = i < A.nnz ? load_key<FIRST>(A, P, i) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kItems; ++k)
        if (base + k * kBlock + threadIdx.x < A.nnz) atomicAdd(&hist[(key[k] >> P.shift) & (kDigits - 1)], 1u);
    __syncthreads();
    A.table[(size_t)threadIdx.x * A.blocks + tile] = hist[threadIdx.x];
}

// exclusive scans of NV values per thread across the workgroup; total[] = the sums of all
template <int NV>
__device__ __forceinline__ void block_exclusive_scans(uint32_t (&v)[NV], uint32_t (&total)[NV], uint32_t (*lds)[kWavesPerBlock])
{
    const int lane = threadIdx.x & (kLanes - 1), w = threadIdx.x >> 6;
    uint32_t incl[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        incl[k] = (uint32_t)wave_scan((int)v[k]);
        if (lane == kLanes - 1) lds[k][w] = incl[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        uint32_t before = 0, all = 0;
#pragma unroll
        for (int q = 0; q < kWavesPerBlock; ++q) {
            const uint32_t t = lds[k][q];
            before += q < w ? t : 0u;
            all += t;
        }
        v[k] = before + incl[k] - v[k];
        total[k] = all;
    }
    __syncthreads();
}

// step 2: workgroup d turns row d of the table into its exclusive prefix and leaves the row's sum
__global__ __launch_bounds__(kBlock) void digit_scan_kernel(TransposeArgs A)
{
    __shared__ uint32_t lds[1][kWavesPerBlock];
    constexpr int kPer = 4;
    uint32_t *row = A.table + (size_t)blockIdx.x * A.blocks;
    uint32_t carry = 0;
    for (int64_t base = 0; base < A.blocks; base += kBlock * kPer) {
        const int64_t first = base + (int64_t)threadIdx.x * kPer;
        uint32_t c[kPer], mine = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            c[k] = first + k < A.blocks ? row[first + k] : 0u;
            mine += c[k];
        }
        uint32_t start[1] = {mine}, total[1];
        block_exclusive_scans<1>(start, total, lds);
        uint32_t run = carry + start[0];
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (first + k < A.blocks) {
                row[first + k] = run;
                run += c[k];
            }
        carry += total[0];
    }
    if (threadIdx.x == 0) A.digit_total[blockIdx.x] = carry;
}

// step 3.  LAST: the positions are those of the column order.  CARRY: the entries' rows go along (as many passes as the workspace
// has room for: two), else the last pass looks them up.
template <bool FIRST, bool LAST, bool CARRY>
__global__ __launch_bounds__(kBlock) void digit_scatter_kernel(TransposeArgs A, PassArgs P)
{
    __shared__ uint32_t seen[kWavesPerBlock][kDigits];  // keys of a digit a wave has ranked so far; then the wave's offset
    __shared__ uint32_t run_start[kDigits];             // where the digit's run starts inside the tile
    __shared__ uint32_t run_dest[kDigits];              // where it goes in the output
    __shared__ uint32_t scan_lds[2][kWavesPerBlock];
    __shared__ uint32_t tile_key[kTile], tile_pay[kTile];
    __shared__ int32_t tile_row[CARRY ? kTile : 1];
    const int lane = threadIdx.x & (kLanes - 1), w = threadIdx.x >> 6;
    const int64_t tile = die_block(blockIdx.x, A.blocks);
    if (tile >= A.blocks) return;
    const int64_t base = tile * kTile;
    const int64_t left = A.nnz - base;
    const int count = (int)(left < kTile ? left : kTile);
    auto wave_sync = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); };

#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) seen[k][threadIdx.x] = 0;
    __syncthreads();

    // the wave's keys in input order: group g, lane l is key w * kWaveKeys + g * 64 + l of the tile
    uint32_t key[kItems], pay[kItems], rank[kItems];
    int32_t row[kItems];
#pragma unroll
    for (int g = 0; g < kItems; ++g) {
        const int t = w * kWaveKeys + g * kLanes + lane;
        const bool valid = t < count;
        key[g] = valid ? load_key<FIRST>(A, P, base + t) : 0u;
        pay[g] = valid ? (FIRST ? (uint32_t)(base + t) : P.pay_in[base + t]) : 0u;
        if (CARRY) row[g] = valid ? (FIRST ? A.entry_row[base + t] : P.row_in[base + t]) : 0;
    }
    const uint32_t digit_total = A.digit_total[threadIdx.x], digit_before = A.table[(size_t)threadIdx.x * A.blocks + tile];
#pragma unroll
    for (int g = 0; g < kItems; ++g) {
        const int t = w * kWaveKeys + g * kLanes + lane;
        const bool valid = t < count;
        const unsigned d = (key[g] >> P.shift) & (kDigits - 1);
        // lanes that hold the same digit
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kDigitBits; ++b) {
            const bool set = ((d >> b) & 1u) != 0;
            const uint64_t m = __ballot(set);
            peers &= set ? m : ~m;
        }
        const int before = __builtin_popcountll(peers & ((1ull << lane) - 1ull));
        uint32_t first = 0;
        if (valid) first = seen[w][d];
        wave_sync();
        if (valid && before == 0) seen[w][d] = first + (uint32_t)__builtin_popcountll(peers);
        wave_sync();
        rank[g] = first + (uint32_t)before;
    }
    __syncthreads();

    // thread d: the waves' offsets inside the run of digit d, the run's place in the tile and in the output
    {
        const int d = threadIdx.x;
        uint32_t run = 0;
#pragma unroll
        for (int k = 0; k < kWavesPerBlock; ++k) {
            const uint32_t c = seen[k][d];
            seen[k][d] = run;
            run += c;
        }
        uint32_t start[2] = {run, digit_total}, total[2];
        block_exclusive_scans<2>(start, total, scan_lds);
        run_start[d] = start[0];
        run_dest[d] = start[1] + digit_before;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kItems; ++g) {
        const int t = w * kWaveKeys + g * kLanes + lane;
        if (t < count) {
            const unsigned d = (key[g] >> P.shift) & (kDigits - 1);
            const uint32_t at = run_start[d] + seen[w][d] + rank[g];
            tile_key[at] = key[g];
            tile_pay[at] = pay[g];
            if (CARRY) tile_row[at] = row[g];
        }
    }
    __syncthreads();
    // neighbouring threads now hold neighbouring keys of a run
#pragma unroll
    for (int k = 0; k < kItems; ++k) {
        const int t = k * kBlock + threadIdx.x;
        if (t < count) {
            const uint32_t kk = tile_key[t];
            const unsigned d = (kk >> P.shift) & (kDigits - 1);
            const int64_t at = (int64_t)run_dest[d] + (t - (int)run_start[d]);
            if (at < A.nnz) {  // always; a guard against a table that does not add up
                const uint32_t p = tile_pay[t];
                P.key_out[at] = kk;
                if (!LAST) {
                    P.pay_out[at] = p;
                    if (CARRY) P.row_out[at] = tile_row[t];
                } else if ((int64_t)p < A.nnz) {  // always: the payloads are a permutation of the positions
                    if ((int64_t)kk < A.m) {
                        A.row_idx[at] = CARRY ? tile_row[t] : A.entry_row[p];
                        A.csc_pos[p] = at;
                    } else {
                        A.csc_pos[p] = -1;  // not an entry of any column
                    }
                }
            }
        }
    }
}

// step 4: col_ptr[j] = number of sorted keys below j, j = 0 .. m.  (Two halves at a time: eight parts mean fewer loads one after
// the other but a line of its own for each, 13.5 instead of 7.6 us with 2e6 entries.)
__global__ __launch_bounds__(kBlock) void col_ptr_kernel(TransposeArgs A, const uint32_t *sorted_key)
{
    const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (j > A.m) return;
    int64_t lo = 0, hi = A.nnz;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo) / 2;
        if ((int64_t)sorted_key[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    A.col_ptr[j] = lo;
}

// ---------------------------------------------------------------------------
// The same by counting.  The entries are taken in blocks: the entry at position p in row r comes to r / 32 + p / E, and block b
// has the entries where that is in [b, b + 1), so they are at most E and of at most 32 rows, and a long row is several blocks' (five full rows
// of 1000 x 40000, us: 31; with blocks of whole rows 68, by sorting 49, as many entries in all rows 28).  Per
// block a bit mask for every column says which of its rows have an entry there, so that an entry's rank among the block's
// entries of its column is a count of bits, whatever order they come in, and nothing has to be sorted:
//   1. column_count_kernel: the masks of a block in LDS; rank[p] of its entries and count[block][column];
//   2. column_scan_kernel: per column, the counts of the blocks before (base[block][column]), and the column's place among 128;
//   3. column_place_kernel: csc_pos[p] = column's beginning + base + rank, row_idx[csc_pos[p]]; col_ptr.
// Every access is consecutive but the gathers from LDS and the stores of row_idx.  Those go to the next free place of a column, one
// line for 32 rows' entries or more, so blocks that lie next to each other run on one die, whose L2 puts the lines together; the dies
// share the blocks by entries, since rows without any also make blocks (20000 x 20000, all 2e6 entries in 4000 of the rows, us:
// 53, with the same number of blocks to a die 74).  E is nnz / 128, in 2048 .. 16384: more entries to a block are fewer rows of the
// table, as long as there are blocks enough for the compute units (2e6 entries in 20000 x 20000, E = 8192 / 16384: 51 / 46 us; 0.9e6
// in 200 x 40000, 41 / 51).
// What bounds it: 6 bytes of table traffic per column and block (0.2 an entry of the matrix) and 37 bytes an entry of the pattern, which
// at 20000 x 20000 and 2e6 entries are 149 MB, 22 us at a copy's rate; count, scan and place take 14 + 11 + 24 in a trace, where the last
// waits for its scattered stores.
// A row holds a column at most once, as the pattern's definition has it.  The masks can't hold a second one, so where any block finds
// one (the bit is set already) column_scan_kernel lists every column entry by entry instead, with the result that the sort has:
// correct, but 128 columns for the time of a look at all entries.
// ---------------------------------------------------------------------------
constexpr int kCountThreads = 1024;
constexpr int kBlockRows = 32, kBlockLeastEntries = 2048, kBlockMostEntries = 16384;
constexpr int kCountHeld = 4;                    // entries of a thread at a time
constexpr int kGroupCols = 128;                  // columns of a workgroup of the scan,
constexpr int kScanCols = 8;                     // of a thread
constexpr int kScanParts = kCountThreads * kScanCols / kGroupCols;  // shares of the blocks in it
constexpr int kScanHeld = 10;                    // blocks of a share requested at once
constexpr int kCountMaxCols = 40000, kCountMostRows = 65535;   // (the masks in LDS; base has 16 bits)
constexpr int padded(int cols) { return (cols + kGroupCols - 1) / kGroupCols * kGroupCols; }
constexpr int kMaxGroups = (kCountMaxCols + kGroupCols - 1) / kGroupCols, kGroupsPerLane = (kMaxGroups + kLanes - 1) / kLanes;

struct BlockRows {  // of a block: its first entry, how many, their first row, how many
    int32_t first, count, row, rows;
};

struct CountLayout {
    size_t count, base, rank, col_off, group_total, rows, repeats, die_start;
    int64_t blocks, pitch, entries;
    int64_t room;  // blocks that the tables have room for
    size_t total;
};

// By counting / by sorting, us: 20000 x 20000, 2e6 entries 46 / 72, 790000 40 / 50; 40000 x 10000, 4e6 67 / 118; 10000 x 10000, 200000 22 / 34;
// 1000 x 1000, 9000 14 / 28; 5000 x 5000, 12000 15 / 28; 100 x 40000, 1.6e6 50 / 64.  Not (the table) where the pattern of a large matrix
// has fewer entries than one in 512, at 20000 x 20000 with 390000 40.0 / 39.5, or one in 200 where m > 20000 leaves room for one workgroup
// on a compute unit, at 5000 x 40000 with 600000 44.9 / 45.3, 30000 x 40000 with 2.5e6 105 / 85; nor where there are more blocks than the
// compute units take at once and (few columns to share the scan) 65000 x 100, 35 / 21, or (few entries in a block) 65535 x 2048 with
// 327000, 51 / 40 (65535 x 3000 with 1e6: 56 / 58); nor (as a row was one block's: 32 x 40000 with 480000 54 / 43,
// 30 / 42 since it is not) for more than 512 n columns; nor where the sort has
// one pass over few entries, at 64 x 64 with 98, 11.0 / 10.5 (2135: 11 / 17).
bool by_counting(int64_t n, int64_t m, int64_t nnz)
{
    if (n < 1 || m < 1 || nnz < 1 || n > kCountMostRows || m > kCountMaxCols) return false;
    return n * m <= std::max<int64_t>(40'000'000, (m <= kCountMaxCols / 2 ? 512 : 200) * nnz) && (n <= 20480 || (m >= 2048 && nnz >= 16 * n)) && m <= 512 * n && (m >= kDigits || nnz >= kTile);
}

CountLayout make_count_layout(int64_t n, int64_t m, int64_t nnz)
{
    CountLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = align_up(off + bytes);
        return at;
    };
    L.entries = std::clamp<int64_t>(nnz / 128, kBlockLeastEntries, kBlockMostEntries);
    L.blocks = (n * L.entries + nnz * kBlockRows) / (kBlockRows * L.entries) + 1;
    // (blocks = floor(n / 32 + nnz / E) + 1 may fall as nnz grows, by one where E = nnz / 128 is rounded down to less; a caller's workspace for
    // more entries has to do for fewer, so the tables' size goes by a bound of it that does not)
    L.room = n / kBlockRows + std::max(nnz / kBlockMostEntries, std::min<int64_t>(nnz / kBlockLeastEntries, 128)) + 2;
    L.pitch = (m + kGroupCols - 1) / kGroupCols * kGroupCols;
    L.count = take((size_t)(L.room * L.pitch));
    L.base = take((size_t)(L.room * L.pitch) * sizeof(uint16_t));
    L.rank = take((size_t)nnz);
    L.col_off = take((size_t)L.pitch * sizeof(uint32_t));
    L.group_total = take((size_t)(L.pitch / kGroupCols) * sizeof(uint32_t));
    L.rows = take((size_t)L.room * sizeof(BlockRows));
    L.repeats = take((size_t)L.room);
    L.die_start = take((kDies + 2) * sizeof(int32_t));
    L.total = off;
    return L;
}

struct CountArgs {
    int n, m, blocks, pitch, entries;  // (entries: as a block may have)
    int64_t nnz;
    const int64_t *row_ptr;
    const int32_t *col_idx;
    int64_t *col_ptr;
    int32_t *row_idx;
    int64_t *csc_pos;
    uint8_t *count;         // [blocks][pitch]
    uint16_t *base;         // [blocks][pitch]
    uint8_t *rank;          // [nnz]
    uint32_t *col_off;      // [pitch] entries of the columns before in the group of 128
    uint32_t *group_total;  // [pitch / 128]
    BlockRows *rows;        // [blocks]
    uint8_t *repeats;       // [blocks] a row of it holds a column twice
    int32_t *die_start;     // [kDies + 1] first blocks of the dies in column_place_kernel; behind them: a block has repeats
};

__device__ __forceinline__ int64_t entries_before(const CountArgs &A, int64_t r)
{
    const int64_t p = A.row_ptr[r];
    return p < 0 ? 0 : p > A.nnz ? A.nnz : p;
}

struct BlockStart {
    int64_t entry;
    int row;
    bool inside;  // of the row: some of its entries are the block before's
};

// Where block b begins, by a wave: the first row that is the block's is among the 64 around where it would be if all had the same number of
// entries, or else among all.
__device__ __forceinline__ BlockStart block_start(const CountArgs &A, int b, int lane)
{
    const int64_t target = (int64_t)b * kBlockRows * A.entries;
    const auto reached = [&](int64_t r) { return r >= A.n || r * A.entries + entries_before(A, r) * kBlockRows >= target; };
    int64_t r = (int64_t)b * A.n / A.blocks - kLanes / 2;
    r = r < 0 ? 0 : r;
    const uint64_t mask = __ballot(reached(r + lane));
    if (mask != 0 && (r == 0 || (mask & 1) == 0)) r += __builtin_ctzll(mask);
    else r = wave_first(0, A.n, lane, reached);
    r = r < A.n ? r : A.n;
    // the end of the row before may be
    const int64_t p = entries_before(A, r), in_row = r > 0 ? (target - (r - 1) * A.entries + kBlockRows - 1) / kBlockRows : p;
    if (in_row < p && in_row >= entries_before(A, r - 1)) return BlockStart{in_row, (int)r - 1, true};
    return BlockStart{p, (int)r, false};
}

// The entries of a block of rows, one to a thread whatever rows they are in.
struct BlockEntries {
    int64_t first;
    int r0, count;
    // ends: LDS [kBlockRows], complete after the next barrier
    __device__ __forceinline__ BlockEntries(const CountArgs &A, const BlockRows &B, int *ends) : first(B.first), r0(B.row), count(B.count)
    {
        if ((int)threadIdx.x < kBlockRows) ends[threadIdx.x] = (int)threadIdx.x < B.rows ? (int)(entries_before(A, r0 + threadIdx.x + 1) - first) : INT32_MAX;
    }
    // the row of the block that entry q is in
    static __device__ __forceinline__ int row(const int *ends, int q)
    {
        int r = 0;
#pragma unroll
        for (int half = kBlockRows / 2; half > 0; half >>= 1) r += ends[r + half - 1] <= q ? half : 0;
        return r;
    }
};

template <int COLS>
__global__ __launch_bounds__(kCountThreads) void column_count_kernel(CountArgs A)
{
    __shared__ __attribute__((aligned(16))) uint32_t mask[padded(COLS)];
    __shared__ int ends[kBlockRows];
    __shared__ BlockStart cut[2];
    __shared__ int repeats;
    const int tid = (int)threadIdx.x, block = (int)blockIdx.x;
    if (tid < 2 * kLanes) {
        const int k = tid / kLanes;
        const BlockStart start = block_start(A, block + k, tid % kLanes);
        if (tid % kLanes == 0) cut[k] = start;
    }
    __syncthreads();
    const int rows = max(0, min(kBlockRows, cut[1].row - cut[0].row + (cut[1].inside ? 1 : 0)));  // (never more, unless row_ptr does not ascend)
    const int64_t first = cut[0].entry, after = cut[1].entry;
    const BlockRows B{(int32_t)first, (int32_t)(after > first ? after - first : 0), cut[0].row, rows};
    const BlockEntries E(A, B, ends);
    if (tid == 0) {
        A.rows[block] = B;
        repeats = 0;
    }
    if (tid <= kDies) {  // the dies that begin behind this block: the next one is the first whose entries begin in their shares
        const auto die_of = [&](int64_t p) { return min((int)(p * kDies / A.nnz), kDies - 1); };
        const int here = block == 0 ? -1 : die_of(first), next = block + 1 == A.blocks ? kDies : die_of(after);
        if (block == 0 && tid == 0) A.die_start[0] = 0;
        else if (tid > max(here, 0) && tid <= next) A.die_start[tid] = block + 1;
    }
    int32_t j[kCountHeld];
    int r[kCountHeld];
    // kCountHeld entries a thread from q0 on: their columns (none: -1), and the rows of those that are in one
    const auto fetch = [&](int q0) {
#pragma unroll
        for (int k = 0; k < kCountHeld; ++k) {
            const int q = q0 + k * kCountThreads + tid;
            j[k] = q < E.count ? A.col_idx[E.first + q] : -1;
            j[k] = (uint32_t)j[k] < (uint32_t)A.m ? j[k] : -1;
        }
    };
    const auto find_rows = [&](int q0) {
#pragma unroll
        for (int k = 0; k < kCountHeld; ++k) r[k] = BlockEntries::row(ends, q0 + k * kCountThreads + tid);
    };
    fetch(0);
    for (int c = 4 * tid; c < A.pitch; c += 4 * kCountThreads) *reinterpret_cast<uint4 *>(mask + c) = uint4{0, 0, 0, 0};
    __syncthreads();
    constexpr int kTrip = kCountHeld * kCountThreads;
    const int last = E.count > 0 ? (E.count - 1) / kTrip * kTrip : 0;
    for (int q0 = 0;; q0 += kTrip) {
        find_rows(q0);
#pragma unroll
        for (int k = 0; k < kCountHeld; ++k)
            if (j[k] >= 0 && (atomicOr(&mask[j[k]], 1u << r[k]) >> r[k] & 1u) != 0) repeats = 1;
        if (q0 >= last) break;
        fetch(q0 + kTrip);
    }
    __syncthreads();
    // A row that begins in a block before this one, and holds a column there and here, is two entries to the column's place in base: right, unless
    // they add up to more than its 16 bits.  (65535 x 10000, 6e6 entries, us, without a look / with one: 98.2 / 99.2.)
    if (A.n + A.blocks > kCountMostRows && cut[0].inside) {
        for (int64_t p = entries_before(A, cut[0].row) + tid; p < first; p += kCountThreads) {
            const int32_t c = A.col_idx[p];
            if ((uint32_t)c < (uint32_t)A.m && (mask[c] & 1u) != 0) repeats = 1;
        }
        __syncthreads();
    }
    if (tid == 0) A.repeats[block] = (uint8_t)repeats;
    for (int q0 = last;; q0 -= kTrip) {  // (what was fetched last first)
#pragma unroll
        for (int k = 0; k < kCountHeld; ++k) {
            const int q = q0 + k * kCountThreads + tid;
            if (q < E.count) A.rank[E.first + q] = j[k] >= 0 ? (uint8_t)__builtin_popcount(mask[j[k]] & ((1u << r[k]) - 1u)) : (uint8_t)0;
        }
        if (q0 == 0) break;
        fetch(q0 - kTrip);
        find_rows(q0 - kTrip);
    }
    uint8_t *count = A.count + (size_t)block * A.pitch;
    for (int c = 4 * tid; c < A.pitch; c += 4 * kCountThreads) {
        const uint4 four = *reinterpret_cast<const uint4 *>(mask + c);
        *reinterpret_cast<uint32_t *>(count + c) = (uint32_t)__builtin_popcount(four.x) | (uint32_t)__builtin_popcount(four.y) << 8 |
                                                   (uint32_t)__builtin_popcount(four.z) << 16 | (uint32_t)__builtin_popcount(four.w) << 24;
    }
}

// The columns of a group in the order of their entries, whatever the rows hold: for patterns with repeats.  Every wave takes a share of the
// blocks; its entries of a column go behind those of the shares before.
__device__ __forceinline__ void list_columns(const CountArgs &A, int c0)
{
    constexpr int kShares = kCountThreads / kLanes;
    __shared__ int32_t next[kShares][kGroupCols];
    __shared__ int32_t before;  // entries of the columns before the group
    const int tid = (int)threadIdx.x, lane = tid % kLanes, share = tid / kLanes;
    const int b0 = (int)((int64_t)A.blocks * share / kShares), b1 = (int)((int64_t)A.blocks * (share + 1) / kShares);
    for (int k = tid; k < kShares * kGroupCols; k += kCountThreads) next[k / kGroupCols][k % kGroupCols] = 0;
    if (tid == 0) before = 0;
    __syncthreads();
    int32_t less = 0;
    for (int b = b0; b < b1; ++b) {
        const BlockRows B = A.rows[b];
        for (int q = lane; q < B.count; q += kLanes) {
            const int32_t j = A.col_idx[(int64_t)B.first + q];
            less += (uint32_t)j < (uint32_t)c0 ? 1 : 0;
            if ((uint32_t)j < (uint32_t)A.m && j >= c0 && j < c0 + kGroupCols) atomicAdd(&next[share][j - c0], 1);
        }
    }
    if (less != 0) atomicAdd(&before, less);
    __syncthreads();
    if (share == 0) {  // two columns a lane: where the shares' entries of each begin
        int32_t sum[2] = {0, 0};
        for (int k = 0; k < kShares; ++k)
            for (int h = 0; h < 2; ++h) sum[h] += next[k][2 * lane + h];
        const int32_t up_to = before + wave_scan(sum[0] + sum[1]);
        int32_t run[2] = {up_to - sum[1] - sum[0], up_to - sum[1]};
        for (int h = 0; h < 2; ++h) {
            const int c = c0 + 2 * lane + h;
            if (c < A.m) A.col_ptr[c] = run[h];
            if (c == A.m - 1) A.col_ptr[A.m] = (int64_t)run[h] + sum[h];
        }
        for (int k = 0; k < kShares; ++k)
            for (int h = 0; h < 2; ++h) {
                const int32_t count = next[k][2 * lane + h];
                next[k][2 * lane + h] = run[h];
                run[h] += count;
            }
    }
    __syncthreads();
    for (int b = b0; b < b1; ++b) {
        const BlockRows B = A.rows[b];
        const int end = lane < B.rows ? (int)(entries_before(A, B.row + lane + 1) - B.first) : INT32_MAX;
        for (int q0 = 0; q0 < B.count; q0 += kLanes) {
            const int q = q0 + lane;
            const int32_t j = q < B.count ? A.col_idx[(int64_t)B.first + q] : -1;
            const bool real = (uint32_t)j < (uint32_t)A.m, mine = real && j >= c0 && j < c0 + kGroupCols;
            if (q < B.count && !real && c0 == 0) A.csc_pos[(int64_t)B.first + q] = -1;
            for (uint64_t open = __ballot(mine); open != 0;) {  // a column at a time, lanes in order
                const int32_t column = __builtin_amdgcn_readlane(j, __builtin_ctzll(open));
                const uint64_t same = __ballot(mine && j == column);
                const int32_t first = next[share][column - c0];
                if ((same >> lane & 1) != 0) {
                    const int32_t to = first + __builtin_popcountll(same & ((1ull << lane) - 1));
                    int row = 0;  // how many of the block's rows end at or before q
                    for (int k = 0; k < kBlockRows; ++k) row += __builtin_amdgcn_readlane(end, k) <= q ? 1 : 0;
                    if (to < A.nnz) A.row_idx[to] = B.row + row;
                    A.csc_pos[(int64_t)B.first + q] = to;
                }
                next[share][column - c0] = first + __builtin_popcountll(same);  // (the same from all lanes)
                open &= ~same;
            }
        }
    }
}

// Eight columns to a thread, two to a word: a column has at most kCountMostRows entries.  The blocks are shared out among groups of
// 16 threads.
__global__ __launch_bounds__(kCountThreads) void column_scan_kernel(CountArgs A)
{
    __shared__ __attribute__((aligned(16))) uint16_t part[kScanParts][kGroupCols];
    __shared__ int wave_repeats[kCountThreads / kLanes];
    const int tid = (int)threadIdx.x, share = tid / (kGroupCols / kScanCols), at = kScanCols * (tid % (kGroupCols / kScanCols));
    const int c = (int)blockIdx.x * kGroupCols + at;
    const int per = (A.blocks + kScanParts - 1) / kScanParts, g0 = min(A.blocks, share * per), g1 = min(A.blocks, g0 + per);
    const uint8_t *count = A.count + c;
    int repeats = 0;
    for (int b = tid; b < A.blocks; b += kCountThreads) repeats |= A.repeats[b];
    uint4 s{0, 0, 0, 0};
    const auto add = [&](uint2 eight) {
        s.x += __builtin_amdgcn_perm(0u, eight.x, 0x0c010c00u);
        s.y += __builtin_amdgcn_perm(0u, eight.x, 0x0c030c02u);
        s.z += __builtin_amdgcn_perm(0u, eight.y, 0x0c010c00u);
        s.w += __builtin_amdgcn_perm(0u, eight.y, 0x0c030c02u);
    };
    uint2 eight[kScanHeld];  // (all requested at once; the first ones are kept)
    const auto fetch = [&](int g) {
#pragma unroll
        for (int k = 0; k < kScanHeld; ++k) eight[k] = g + k < g1 ? *reinterpret_cast<const uint2 *>(count + (size_t)(g + k) * A.pitch) : uint2{0, 0};
    };
    for (int g = g0 + kScanHeld; g < g1; g += kScanHeld) {
        fetch(g);
#pragma unroll
        for (int k = 0; k < kScanHeld; ++k) add(eight[k]);
    }
    fetch(g0);
#pragma unroll
    for (int k = 0; k < kScanHeld; ++k) add(eight[k]);
    *reinterpret_cast<uint4 *>(&part[share][at]) = s;
    const uint64_t in_wave = __ballot(repeats != 0);
    if (tid % kLanes == 0) wave_repeats[tid / kLanes] = in_wave != 0 ? 1 : 0;
    __syncthreads();
    repeats = 0;
#pragma unroll
    for (int k = 0; k < kCountThreads / kLanes; ++k) repeats |= wave_repeats[k];
    if (blockIdx.x == 0 && tid == 0) A.die_start[kDies + 1] = repeats;
    if (repeats != 0) {
        list_columns(A, (int)blockIdx.x * kGroupCols);
        return;
    }
    if (tid < kLanes) {  // two columns a lane: what is before each share, and their sums
        uint32_t run = 0;
#pragma unroll 16
        for (int k = 0; k < kScanParts; ++k) {
            uint32_t *two = reinterpret_cast<uint32_t *>(&part[k][2 * tid]);
            const uint32_t t = *two;
            *two = run;
            run += t;
        }
        const uint32_t t0 = run & 0xffffu, t1 = run >> 16, up_to = (uint32_t)wave_scan((int)(t0 + t1));
        uint32_t *col_off = A.col_off + (int)blockIdx.x * kGroupCols + 2 * tid;
        col_off[0] = up_to - t1 - t0;
        col_off[1] = up_to - t1;
        if (tid == kLanes - 1) A.group_total[blockIdx.x] = up_to;
    }
    __syncthreads();
    s = *reinterpret_cast<const uint4 *>(&part[share][at]);
    uint16_t *base = A.base + c;
    for (int g = g0; g < g1; g += kScanHeld) {
        if (g != g0) fetch(g);
#pragma unroll
        for (int k = 0; k < kScanHeld; ++k) {
            if (g + k < g1) *reinterpret_cast<uint4 *>(base + (size_t)(g + k) * A.pitch) = s;
            add(eight[k]);
        }
    }
}

template <int COLS>
__global__ __launch_bounds__(kCountThreads) void column_place_kernel(CountArgs A)
{
    __shared__ __attribute__((aligned(16))) uint32_t at[padded(COLS)];  // where the block's first entry of a column goes
    __shared__ uint32_t group_at[kGroupsPerLane * kLanes + 1];
    __shared__ int ends[kBlockRows];
    if (A.die_start[kDies + 1] != 0) return;  // (all is done)
    const int die = (int)blockIdx.x % kDies;
    int block = max(A.die_start[die], 0) + (int)blockIdx.x / kDies;
    const int end = min(A.die_start[die + 1], A.blocks);
    for (bool first = true; first || block < end; first = false, block += (int)gridDim.x / kDies) {
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));  // (no addresses kept over the loop: with more than 64 registers a compute unit has one workgroup)
        const BlockEntries E(A, block < end ? A.rows[block] : BlockRows{}, ends);
        if (!first && E.count == 0) continue;
        int32_t j[kCountHeld];
        uint32_t rank[kCountHeld];
        const auto fetch = [&](int q0) {
#pragma unroll
            for (int k = 0; k < kCountHeld; ++k) {
                const int q = q0 + k * kCountThreads + tid;
                j[k] = q < E.count ? A.col_idx[E.first + q] : -1;
                rank[k] = q < E.count ? A.rank[E.first + q] : 0u;
            }
        };
        fetch(0);
        constexpr int kStage = (padded(COLS) / kScanCols + kCountThreads - 1) / kCountThreads;
        const uint16_t *base = A.base + (size_t)min(block, A.blocks - 1) * A.pitch;
        uint4 b[kStage];
#pragma unroll
        for (int k = 0; k < kStage; ++k) {
            const int c = kScanCols * (k * kCountThreads + tid);
            b[k] = c < A.pitch ? *reinterpret_cast<const uint4 *>(base + c) : uint4{0, 0, 0, 0};
        }
        if (first && tid < kLanes) {
            const int groups = A.pitch / kGroupCols;
            uint32_t t[kGroupsPerLane], sum = 0;
#pragma unroll
            for (int k = 0; k < kGroupsPerLane; ++k) {
                const int i = tid * kGroupsPerLane + k;
                t[k] = i < groups ? A.group_total[i] : 0u;
                sum += t[k];
            }
            const uint32_t up_to = (uint32_t)wave_scan((int)sum);
            uint32_t run = up_to - sum;
#pragma unroll
            for (int k = 0; k < kGroupsPerLane; ++k) {
                group_at[tid * kGroupsPerLane + k] = run;
                run += t[k];
            }
            if (tid == kLanes - 1) group_at[kGroupsPerLane * kLanes] = up_to;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kStage; ++k) {
            const int c = kScanCols * (k * kCountThreads + tid);
            if (c >= A.pitch) break;
            const uint32_t g = group_at[c / kGroupCols];
            const uint4 o0 = *reinterpret_cast<const uint4 *>(A.col_off + c), o1 = *reinterpret_cast<const uint4 *>(A.col_off + c + 4);
            *reinterpret_cast<uint4 *>(at + c) = uint4{g + o0.x + (b[k].x & 0xffffu), g + o0.y + (b[k].x >> 16), g + o0.z + (b[k].y & 0xffffu), g + o0.w + (b[k].y >> 16)};
            *reinterpret_cast<uint4 *>(at + c + 4) = uint4{g + o1.x + (b[k].z & 0xffffu), g + o1.y + (b[k].z >> 16), g + o1.z + (b[k].w & 0xffffu), g + o1.w + (b[k].w >> 16)};
        }
        if (first)
            for (int64_t c = (int64_t)blockIdx.x * kCountThreads + tid; c <= A.m; c += (int64_t)gridDim.x * kCountThreads)
                A.col_ptr[c] = c < A.m ? group_at[c / kGroupCols] + A.col_off[c] : group_at[kGroupsPerLane * kLanes];
        __syncthreads();
        constexpr int kTrip = kCountHeld * kCountThreads;
        for (int q0 = 0; q0 < E.count; q0 += kTrip) {
            if (q0 != 0) fetch(q0);
#pragma unroll
            for (int k = 0; k < kCountHeld; ++k) {
                const int q = q0 + k * kCountThreads + tid;
                if (q >= E.count) break;
                int64_t to = -1;  // (not an entry of any column)
                if ((uint32_t)j[k] < (uint32_t)A.m) {
                    to = (int64_t)at[j[k]] + rank[k];
                    if (to < A.nnz) A.row_idx[to] = E.r0 + BlockEntries::row(ends, q);  // (always, unless row_ptr does not add up)
                }
                A.csc_pos[E.first + q] = to;
            }
        }
        if (block + (int)gridDim.x / kDies >= end) break;
        __syncthreads();  // at and ends are read
    }
}

int check_dims(int64_t n, int64_t m, int64_t nnz)
{
    if (n < 0 || m < 0 || n > kMaxDim || m > kMaxDim) return REGOT_ERR_DIM;
    if (nnz < 0 || nnz > kMaxDim) return REGOT_ERR_ARG;
    return REGOT_OK;
}

}  // namespace

extern "C" {

int regot_pattern_transpose_workspace_bytes(int64_t n, int64_t m, int64_t nnz, size_t *bytes)
{
    if (!bytes) return REGOT_ERR_NULL;
    const int st = check_dims(n, m, nnz);
    if (st != REGOT_OK) return st;
    *bytes = make_transpose_layout(m, nnz).total;
    if (by_counting(n, m, nnz)) *bytes = std::max(*bytes, make_count_layout(n, m, nnz).total);
    return REGOT_OK;
}

int regot_pattern_transpose(int64_t n, int64_t m, int64_t nnz, const int64_t *row_ptr, const int32_t *col_idx,
                            int64_t *col_ptr, int32_t *row_idx, int64_t *csc_pos, void *workspace,
                            size_t workspace_bytes, regot_stream_t stream)
{
    int st = check_dims(n, m, nnz);
    if (st != REGOT_OK) return st;
    if (!row_ptr || !col_ptr || (nnz > 0 && (!col_idx || !row_idx || !csc_pos))) return REGOT_ERR_NULL;
    if (misaligned(row_ptr, 8) || misaligned(col_ptr, 8) || misaligned(csc_pos, 8) || misaligned(col_idx, 4) ||
        misaligned(row_idx, 4))
        return REGOT_ERR_ALIGN;
    const TransposeLayout L = make_transpose_layout(m, nnz);
    if (!workspace) return REGOT_ERR_NULL;
    if (misaligned(workspace, kAlign)) return REGOT_ERR_ALIGN;
    const bool counting = by_counting(n, m, nnz);
    if (workspace_bytes < (counting ? std::max(L.total, make_count_layout(n, m, nnz).total) : L.total)) return REGOT_ERR_WORKSPACE;

    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    if (counting) {
        const CountLayout K = make_count_layout(n, m, nnz);
        const CountArgs C{(int)n, (int)m, (int)K.blocks, (int)K.pitch, (int)K.entries, nnz, row_ptr, col_idx, col_ptr, row_idx, csc_pos,
                          reinterpret_cast<uint8_t *>(ws + K.count), reinterpret_cast<uint16_t *>(ws + K.base),
                          reinterpret_cast<uint8_t *>(ws + K.rank), reinterpret_cast<uint32_t *>(ws + K.col_off),
                          reinterpret_cast<uint32_t *>(ws + K.group_total), reinterpret_cast<BlockRows *>(ws + K.rows),
                          reinterpret_cast<uint8_t *>(ws + K.repeats), reinterpret_cast<int32_t *>(ws + K.die_start)};
        const bool narrow = m <= kCountMaxCols / 2;  // (two workgroups to a compute unit)
        const dim3 threads(kCountThreads);
        hipLaunchKernelGGL(narrow ? column_count_kernel<kCountMaxCols / 2> : column_count_kernel<kCountMaxCols>, dim3((unsigned)K.blocks), threads, 0, s, C);
        hipLaunchKernelGGL(column_scan_kernel, dim3((unsigned)(K.pitch / kGroupCols)), threads, 0, s, C);
        hipLaunchKernelGGL(narrow ? column_place_kernel<kCountMaxCols / 2> : column_place_kernel<kCountMaxCols>, dim3((unsigned)die_grid(K.blocks)), threads, 0, s, C);
        return hipGetLastError() == hipSuccess ? REGOT_OK : REGOT_ERR_HIP;
    }
    TransposeArgs A{};
    A.n = n;
    A.m = m;
    A.nnz = nnz;
    A.row_ptr = row_ptr;
    A.col_idx = col_idx;
    A.col_ptr = col_ptr;
    A.row_idx = row_idx;
    A.csc_pos = csc_pos;
    A.table = reinterpret_cast<uint32_t *>(ws + L.table);
    A.digit_total = reinterpret_cast<uint32_t *>(ws + L.digit_total);
    A.entry_row = reinterpret_cast<int32_t *>(ws + L.entry_row);
    A.blocks = L.blocks;
    uint32_t *key[2] = {reinterpret_cast<uint32_t *>(ws + L.key[0]), reinterpret_cast<uint32_t *>(ws + L.key[1])};
    uint32_t *pay[2] = {reinterpret_cast<uint32_t *>(ws + L.pay[0]), reinterpret_cast<uint32_t *>(ws + L.pay[1])};

    const unsigned col_blocks = (unsigned)((m + 1 + kBlock - 1) / kBlock);
    if (nnz == 0) {
        // no keys: every column starts and ends at 0
        hipLaunchKernelGGL(col_ptr_kernel, dim3(col_blocks), dim3(kBlock), 0, s, A, (const uint32_t *)key[0]);
        return hipGetLastError() == hipSuccess ? REGOT_OK : REGOT_ERR_HIP;
    }
    int64_t row_blocks = (n + kWavesPerBlock - 1) / kWavesPerBlock;
    if (row_blocks > 16 * 256) row_blocks = 16 * 256;
    const unsigned tiles = (unsigned)die_grid(L.blocks);
    const bool carry = L.passes <= 2;
    for (int pass = 0; pass < L.passes; ++pass) {
        PassArgs P{};
        P.key_in = pass == 0 ? nullptr : key[(pass - 1) & 1];
        P.pay_in = pass == 0 ? nullptr : pay[(pass - 1) & 1];
        P.key_out = key[pass & 1];
        P.pay_out = pay[pass & 1];
        P.row_in = P.row_out = reinterpret_cast<int32_t *>(pay[1]);  // (two passes: the second writes no list of positions)
        P.shift = pass * kDigitBits;
        const bool first = pass == 0, last = pass == L.passes - 1;
        if (first) hipLaunchKernelGGL(digit_count_kernel<true>, dim3(tiles + (unsigned)row_blocks), dim3(kBlock), 0, s, A, P);
        else hipLaunchKernelGGL(digit_count_kernel<false>, dim3(tiles), dim3(kBlock), 0, s, A, P);
        hipLaunchKernelGGL(digit_scan_kernel, dim3(kDigits), dim3(kBlock), 0, s, A);
        if (first && last) hipLaunchKernelGGL((digit_scatter_kernel<true, true, true>), dim3(tiles), dim3(kBlock), 0, s, A, P);
        else if (carry && first) hipLaunchKernelGGL((digit_scatter_kernel<true, false, true>), dim3(tiles), dim3(kBlock), 0, s, A, P);
        else if (carry) hipLaunchKernelGGL((digit_scatter_kernel<false, true, true>), dim3(tiles), dim3(kBlock), 0, s, A, P);
        else if (first) hipLaunchKernelGGL((digit_scatter_kernel<true, false, false>), dim3(tiles), dim3(kBlock), 0, s, A, P);
        else if (!last) hipLaunchKernelGGL((digit_scatter_kernel<false, false, false>), dim3(tiles), dim3(kBlock), 0, s, A, P);
        else hipLaunchKernelGGL((digit_scatter_kernel<false, true, false>), dim3(tiles), dim3(kBlock), 0, s, A, P);
    }
    const uint32_t *sorted_key = key[(L.passes - 1) & 1];
    hipLaunchKernelGGL(col_ptr_kernel, dim3(col_blocks), dim3(kBlock), 0, s, A, sorted_key);
    return hipGetLastError() == hipSuccess ? REGOT_OK : REGOT_ERR_HIP;
}

}  // extern "C"
