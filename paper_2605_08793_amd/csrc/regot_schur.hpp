// H_Omega + tau I solved through its Schur complement (regot_pcg_solve_reduced, regot_pcg_solve2_reduced).  With
//     H_Omega + tau I = [ D1   B  ]     D1 = diag(T 1) / eta + tau        (n)
//                       [ B^T  D2 ]     D2 = diag(T_{-m}^T 1) / eta + tau (m - 1),   B = T^Omega_{-m} / eta
// (eq. (7)) and rhs = (g1, g2), eliminating the first block leaves S x2 = g2 - B^T D1^{-1} g1 with
// S = D2 - B^T D1^{-1} B (symmetric positive definite as the whole matrix is, Theorem 1), and
// x1 = D1^{-1} (g1 - B x2).  Conjugate gradients on S preconditioned with D2 take about half the iterations
// of the iteration on the whole matrix (the classical result for matrices whose diagonal blocks are diagonal).
// (regot_schur_wide.hpp has the same for systems whose blocks are both longer than kSchurCap.)
//
// An iteration is three kernels: the half product by rows, which forms p = z + ratio p_old and u = D1^{-1} B p, the latter from
// D1^{-1} B z and the u of the iteration before (so its gathers need z, and not what the ratio is still to be found for; see
// kSchurRecurrent); the half product S p = D2 p - B^T u by columns, with p^T S p; and x, r, z with their inner products.  Scalars
// are worked out by every wave that needs them from the partial sums the kernel before left, in a fixed order; they live on the
// device, and after convergence the remaining kernels return at once.
//
// A pair of systems is the same kernels with a second row of workgroups (blockIdx.y): a system's arithmetic does not
// depend on the other one, and the two workgroups that read the same entries run on one die (the linear ids differ by
// half of kSchurParts, a multiple of the number of dies), so the entries come from memory once.
#pragma once

#include "regot_sparse.hpp"

namespace regot {

// The half products.  The rows (columns) are cut into kSchurParts contiguous parts with about the same number of
// entries, once per solve (schur_prepare_kernel), eight waves to a part.  Inside a part the ENTRIES are dealt out, not the
// rows: a slice of 256 consecutive entries to a wave, 4 to a lane, whatever rows they belong to; a bit mask says where rows
// end, and a segmented scan over the wave puts them together.  So all that a workgroup reads is requested at once, a long
// row is as good as many short ones, and one vector fits the LDS for up to kSchurCap entries (a pair of vectors side by
// side fitted half of that).  One system: a workgroup per part.  Two: two parts and one system to a workgroup, half of the
// workgroups for either system; the chip is full both times, and what happens to a part is the same.
//
// What bounds it (pair of systems, 20000 x 20000, 2e6 entries; time stamps): 4.3 us until 350 KB a workgroup have come (the
// vector from L2, the entries from the last-level cache, both near the rate of a compute unit), 1.3 us for the mask, 2.3 us of
// instructions for four slices a wave (64 entries of the scan cost as much as 256 gathers from LDS), 1 us to the results, and
// about 2 us of launch.  12.0 us by columns, 13.5 by rows between those stamps, 13.3 and 14.4 in a
// kernel trace (update 4.1 to 4.8), an iteration 28.1 in launches one behind the other; a wave per row with the pair side by side,
// half of its gathers going to L2, took 16.4 and 20.2, and an iteration 36 in four kernels.  On the way: the row of a lane's
// first entry by bisection, 64-bit positions throughout 20.9 us (8.8 of them instructions); two trips of two slices 12.2.
constexpr int kSchurParts = 256;
constexpr int kSchurPartWaves = 8;
constexpr int kSchurPartThreads = kSchurPartWaves * kLanes;
constexpr int kSchurLaneEntries = 4;                              // consecutive entries of a lane
constexpr int kSchurSlice = kSchurLaneEntries * kLanes;           // of a wave
constexpr int kSchurWaveSlices = 4;                               // slices of a wave per trip
constexpr int kSchurTripSlices = kSchurPartWaves * kSchurWaveSlices;
constexpr int kSchurTrip = kSchurTripSlices * kSchurSlice;        // entries of a part per trip
constexpr int kSchurHeld = 128;                                   // rows of a part whose sums are held at a time
constexpr int kSchurCap = 20000;                                  // entries of the vector in LDS
constexpr int kSchurRowCost = 16;                                 // what a row costs besides its entries, in entries
constexpr int kSchurVecBlocks = 256;                              // most workgroups of the vector kernels
// From so many steps on every second u = D1^{-1} B p is the product again instead of the recurrence, whose rounding errors add
// up: where the solution takes hundreds of iterations (a small tau, values over several orders of magnitude), the recurrence
// throughout took 1.2 to 1.4 times as many of them, and left 3 to 7 times the residual of the whole system.  So it is neither
// more iterations nor a larger residual than with products throughout, beyond what other orders of the sums make of either
// (with every fourth a product 3 to 5 % more iterations, with every eighth 8 to 10 %).
// A step with p in LDS instead of z takes longer: on average 25.1 -> 26.6 us at 20000 x 20000 with 2e6 entries, a pair 28.3 -> 30.1;
// where z is longer than the LDS as well, 15000 x 100000 with 3e6, 45.3 -> 54 and 62.5 -> 82.
constexpr int kSchurRecurrent = 32;
static_assert(kSchurLaneEntries == 4 && kSchurTripSlices * 2 == kLanes, "four bits of the mask per lane and slice; two lanes per slice");

// where a part begins: its first row (column) and that one's first entry
struct SchurCut {
    int64_t item, entry;
};

// What the kernels of an iteration read and hand on.  Two slots per system, alternating: a kernel that writes the one
// leaves the other alone, which its other workgroups may still be reading.
struct SchurState {
    double rz, rr, bb;    // r^T z, ||r||^2, ||rhs||^2 of the whole system
    long long steps;      // steps whose partial sums are there, or will be before this is read
    int done;             // converged (or nothing to do)
    int first;            // no step yet: the partial sums are those of the start, and of ||rhs||^2
    int flip;             // which of the two buffers holds p; S p is formed in the other
    int pad;
};

struct SchurArgs {
    int n, mb;            // rows, columns that are variables (m - 1)
    double eta, tau, rtol;
    const int64_t *row_ptr, *col_ptr;
    const int32_t *col_idx, *row_idx;
    const double *val, *val_csc;
    int64_t capacity;
    const double *row_sum, *col_sum;
    // per system:
    const double *rhs[2];     // [n + mb]
    double *x_out[2];         // [n + mb]
    double *x[2];             // [mb] the iterate (may be x_out + n)
    double *u[2];             // [n]
    double *r[2], *z[2];      // [mb]
    double *buf[2][2];        // [system][flip][mb]: p and S p
    double *part[2];          // partial sums: p^T S p [kSchurParts]
    double *part_rz[2], *part_rr[2], *part_norm[2];  // [kSchurVecBlocks]
    SchurState *state;        // [2 slots][2 systems]
    SchurCut *row_cut, *col_cut;  // [kSchurParts + 1]
    double *info;             // [4] per system
    int it;                   // iteration of this call; the final kernel: the number of them
    int vec_blocks, norm_blocks;
};

// The beginning of share `part` of [0, count) cut into kSchurParts (part == kSchurParts: the end), for what every part does to
// its share of a vector.
__host__ __device__ constexpr int64_t schur_share(int64_t count, int part)
{
    const int64_t at = (count + kSchurParts - 1) / kSchurParts * part;
    return at < count ? at : count;
}

__device__ __forceinline__ int64_t clamp_entry(int64_t p, int64_t capacity) { return p < 0 ? 0 : p > capacity ? capacity : p; }

// Sum of part[0 .. count), count <= kSchurVecBlocks, in a fixed order; every lane gets it.  In two steps, so that the loads
// can be on their way while something else is waited for.
struct WaveParts {
    double v[kSchurVecBlocks / kLanes];
    __device__ __forceinline__ void fetch(const double *part, int count, int lane)
    {
#pragma unroll
        for (int k = 0; k < kSchurVecBlocks / kLanes; ++k) v[k] = k * kLanes + lane < count ? part[k * kLanes + lane] : 0.0;
    }
    __device__ __forceinline__ double sum() const
    {
        double s = v[0];
#pragma unroll
        for (int k = 1; k < kSchurVecBlocks / kLanes; ++k) s += v[k];
        return wave_reduce1<OpSum>(s);
    }
};

// For what the running kernel does not write and all lanes read alike: by scalar loads, which do not wait for vector loads
// requested before them.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T *scalar_at(const T *p)
{
    return (const __attribute__((address_space(4))) T *)p;
}
__device__ __forceinline__ SchurState schur_state(const SchurState *slot)
{
    const auto *at = scalar_at(slot);
    return SchurState{at->rz, at->rr, at->bb, at->steps, at->done, at->first, at->flip, 0};
}

// the state after the partial sums `rz`, `rr` (and `norm`, for a first one) have become known
__device__ __forceinline__ SchurState schur_advance(const SchurState &cur, double rz, double rr, double norm, double rtol)
{
    SchurState nx = cur;
    nx.rz = rz;
    nx.rr = rr;
    if (cur.first) nx.bb = norm;
    nx.done = rr <= rtol * rtol * nx.bb || (cur.first && rr == 0.0) ? 1 : 0;
    if (!nx.done) {
        nx.first = 0;
        nx.steps = cur.steps + 1;
        nx.flip = cur.flip ^ 1;
    }
    return nx;
}

// u = D1^{-1} g1, partial sums of ||rhs||^2; and, by the workgroups behind the first norm_blocks, the cuts: a wave finds the
// first row r at which ptr[r] + kSchurRowCost r reaches its share of the whole, 64 places at a time.
constexpr int kSchurCutWaves = 2 * (kSchurParts + 1);
__global__ __launch_bounds__(kThreads) void schur_prepare_kernel(SchurArgs A)
{
    __shared__ double lds[kWaves];
    const int lane = threadIdx.x & (kLanes - 1);
    if ((int)blockIdx.x >= A.norm_blocks) {
        const int wave = ((int)blockIdx.x - A.norm_blocks) * kWaves + (int)(threadIdx.x >> 6);
        if (wave >= kSchurCutWaves || blockIdx.y != 0) return;
        const bool rows = wave <= kSchurParts;
        const int t = rows ? wave : wave - (kSchurParts + 1);
        const int64_t *ptr = rows ? A.row_ptr : A.col_ptr;
        const int64_t count = rows ? A.n : A.mb;
        const int64_t w0 = clamp_entry(ptr[0], A.capacity), w1 = clamp_entry(ptr[count], A.capacity) + kSchurRowCost * count;
        // (whole parts and the rest apart: the product would not fit for any number of entries)
        const int64_t whole = (w1 - w0) / kSchurParts, rest = (w1 - w0) % kSchurParts;
        const int64_t target = w0 + whole * t + rest * t / kSchurParts;
        const auto reached = [&](int64_t r) { return clamp_entry(ptr[r], A.capacity) + kSchurRowCost * r >= target; };
        const int64_t at = wave_first(t == kSchurParts ? count : 0, t == 0 ? 0 : count, lane, reached);
        if (lane == 0) (rows ? A.row_cut : A.col_cut)[t] = SchurCut{at, clamp_entry(ptr[at], A.capacity)};
        return;
    }
    const int sys = (int)blockIdx.y;
    const double *rhs = A.rhs[sys];
    double gg = 0.0;
    const int64_t N = (int64_t)A.n + A.mb;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < N; t += (int64_t)A.norm_blocks * kThreads) {
        const double g = rhs[t];
        gg += g * g;
        if (t < A.n) A.u[sys][t] = g / (A.row_sum[t] / A.eta + A.tau);
    }
    const double s = block_sum(gg, lds);
    if (threadIdx.x == 0) A.part_norm[sys][blockIdx.x] = s;
}

enum SchurMode {
    kSchurRows = 0,       // p = z + ratio p_old and u = D1^{-1} B p, as u_i = (sum_j T_ij z_j / eta) / D1_i + ratio u_old_i
    kSchurRowsFinal = 1,  // x1_i = (g1_i - sum_j T_ij x2_j / eta) / D1_i; x2 to the caller, the record of the iteration
    kSchurCols = 2,       // (S p)_j = D2_j p_j - sum_i T_ij u_i / eta; p^T S p
    kSchurColsRhs = 3,    // r_j = g2_j - sum_i T_ij u_i / eta; x = 0, z = D2^{-1} r; r^T z, r^T r
    kSchurRowsLater = 4   // kSchurRows where the step may be kSchurRecurrent or a later one, and u_i (sum_j T_ij p_j / eta) / D1_i
};

// sums over a part's waves of NV values per thread, in a fixed order; its first thread gets them
template <int NV>
__device__ __forceinline__ void schur_part_sums(double (&v)[NV], double (*lds)[kSchurPartWaves], int lane, int w)
{
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = wave_reduce1<OpSum>(v[k]);
        if (lane == 0) lds[k][w] = v[k];
    }
    __syncthreads();
    if (lane == 0 && w == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            v[k] = lds[k][0];
#pragma unroll
            for (int q = 1; q < kSchurPartWaves; ++q) v[k] += lds[k][q];
        }
    }
}

// Segmented inclusive sum over the wave: lane l ends with the sum of lanes l - dist .. l, where a segment begins.
struct SegmentedScan {
    int to15, to31;  // distances from which on a segment reaches into the row of lanes, and the half, before
    __device__ __forceinline__ explicit SegmentedScan(int lane)
        : to15((lane & 16) != 0 ? (lane & 15) + 1 : kLanes), to31(lane >= 32 ? lane - 31 : kLanes) {}
    __device__ __forceinline__ double operator()(double v, int dist) const
    {
        double up = dpp_f64<kDppRowShr + 1>(v);
        v += dist >= 1 ? up : 0.0;
        up = dpp_f64<kDppRowShr + 2>(v);
        v += dist >= 2 ? up : 0.0;
        up = dpp_f64<kDppRowShr + 4>(v);
        v += dist >= 4 ? up : 0.0;
        up = dpp_f64<kDppRowShr + 8>(v);
        v += dist >= 8 ? up : 0.0;
        up = dpp_f64<kDppRowBcast15>(v);
        v += dist >= to15 ? up : 0.0;
        up = dpp_f64<kDppRowBcast31>(v);
        v += dist >= to31 ? up : 0.0;
        return v;
    }
};

struct SchurPartShared {
    union __attribute__((aligned(16))) {
        uint32_t ends[kSchurTrip / 32];       // bit q: entry q of the trip is its row's last; then, when all have their share of it:
        double sums[kSchurHeld];              // the last pieces of the rows in hand, in the order of the rows that have entries
    };
    double tails[kSchurTripSlices];           // what a slice has of the row it ends in
    double carry[2];                          // what the trips so far have of the row they end in, by parity of the trip
    int filled[kSchurHeld / kLanes];          // rows with entries among 64
};
struct SchurShared {
    __attribute__((aligned(16))) double xs[kSchurCap + 2];  // behind the vector a 0 for indices that are none
    SchurPartShared part[2];
};
static_assert(sizeof(SchurShared) <= 160 * 1024, "LDS per CU");
static_assert(2 * kSchurPartWaves <= kSchurHeld, "schur_part_sums in sums");
static_assert(kSchurTrip / 32 <= kSchurPartThreads && kSchurHeld <= kSchurPartThreads, "a thread per word, and per row");

// ALL: the vector fits the LDS.
template <int KIND, int R, bool ALL>
__global__ __launch_bounds__(R *kSchurPartThreads) REGOT_WAVES_ATTR(4) void schur_half_kernel(SchurArgs A)
{
    constexpr int MODE = KIND == kSchurRowsLater ? kSchurRows : KIND;
    constexpr bool ROWS = MODE == kSchurRows || MODE == kSchurRowsFinal;
    typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));
    typedef int32_t int4u __attribute__((ext_vector_type(4), aligned(4)));
    constexpr int kThreadsAll = R * kSchurPartThreads, kWavesAll = R * kSchurPartWaves;  // (a workgroup has as many parts as there are systems)
    __shared__ SchurShared S;
    const int all_tid = (int)threadIdx.x, lane = all_tid & (kLanes - 1), all_w = __builtin_amdgcn_readfirstlane(all_tid >> 6);
    const int sub = all_w / kSchurPartWaves, w = all_w % kSchurPartWaves, tid = all_tid - sub * kSchurPartThreads;
    const int sys = (int)blockIdx.y, me = (int)blockIdx.x * R + sub;
    SchurPartShared &L = S.part[sub];

    // (a wave's base and a lane's 32-bit offset)
    const auto lane_at = [&](const void *p, int bytes) { return static_cast<const char *>(p) + (unsigned)(lane * bytes); };

    // Everything is requested before anything is waited for (but the state, by scalar loads, so that the kernels behind the
    // last step end early).  The vector, straight to LDS:
    SchurState cur{};
    if (MODE != kSchurColsRhs) cur = schur_state(A.state + 2 * ((MODE == kSchurCols ? A.it + 1 : A.it) & 1) + sys);
    if ((MODE == kSchurRows || MODE == kSchurCols) && cur.done) {
        if (MODE == kSchurRows && me == 0 && tid == 0) A.state[2 * ((A.it + 1) & 1) + sys] = cur;
        return;
    }
    const bool fresh = KIND == kSchurRowsLater && cur.steps >= kSchurRecurrent && (cur.steps & 1) == 0;  // u from p, not from z and the u before
    const int limit = ROWS ? A.mb : A.n;
    const int nl = limit < kSchurCap ? limit : kSchurCap;
    const double *xs = MODE == kSchurRows ? A.z[sys] : MODE == kSchurRowsFinal ? A.x[sys] : A.u[sys];
    constexpr int kPer = (kSchurCap / 2 + kThreadsAll - 1) / kThreadsAll;
    const int pairs = nl / 2;
    if (MODE != kSchurRowsFinal || (reinterpret_cast<uintptr_t>(xs) & 15) == 0) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int first = (k * kWavesAll + all_w) * kLanes;  // the wave's 64 pairs, 16 bytes a lane, one after the other
            if (first + lane < pairs)
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(lane_at(xs + 2 * first, 16)),
                                                 (__attribute__((address_space(3))) void *)(S.xs + 2 * first), 16, 0, 0);
        }
    } else {  // (an iterate of the caller's, at an odd multiple of 8 bytes)
        for (int i = all_tid; i < 2 * pairs; i += kThreadsAll) S.xs[i] = xs[i];
    }
    const double *p_old = cur.flip ? A.buf[sys][1] : A.buf[sys][0];  // (kSchurCols: p)
    double *other = cur.flip ? A.buf[sys][0] : A.buf[sys][1];        // p, or S p
    // fresh: p_old as well, to registers as far as there are any
    constexpr int kAhead = KIND == kSchurRowsLater ? (R == 1 ? kPer : 2) : 1;
    dbl2u p_ahead[kAhead];
    const auto p_pair = [&](int k) {
        const int at = (k * kWavesAll + all_w) * kLanes + lane;
        return *reinterpret_cast<const dbl2u *>(p_old + 2 * (at < pairs ? at : 0));
    };
    if (fresh && pairs > 0) {
#pragma unroll
        for (int k = 0; k < kAhead; ++k) p_ahead[k] = p_pair(k);
    }
    const double last = (nl & 1) != 0 && all_tid == 0 ? xs[nl - 1] : 0.0;
    if (tid < kSchurTrip / 32) L.ends[tid] = 0;
    __syncthreads();

    // this workgroup's part, and the entries of its first trip (what lies behind the part is not used)
    const auto *cut = scalar_at((ROWS ? A.row_cut : A.col_cut) + me);
    const int64_t r0 = cut[0].item, r1 = cut[1].item, e0 = cut[0].entry, e1 = cut[1].entry;
    const int64_t *ptr = ROWS ? A.row_ptr : A.col_ptr;
    // (the waves of the two parts of a workgroup go through the same barriers: the longer part says how many)
    const auto *cut_b = scalar_at((ROWS ? A.row_cut : A.col_cut) + (R == 2 ? me ^ 1 : me));
    const int64_t r0_b = cut_b[0].item, r1_b = cut_b[1].item, e0_b = cut_b[0].entry, e1_b = cut_b[1].entry;
    const int64_t rows_max = r1 - r0 > r1_b - r0_b ? r1 - r0 : r1_b - r0_b;
    const int32_t *idx = ROWS ? A.col_idx : A.row_idx;
    const double *val = ROWS ? A.val : A.val_csc;
    int32_t bj[kSchurWaveSlices][kSchurLaneEntries];
    double bv[kSchurWaveSlices][kSchurLaneEntries];
    auto load_slice = [&](int h, int64_t base) {
        const int64_t q_wave = base + (h * kSchurPartWaves + w) * kSchurSlice, q = q_wave + kSchurLaneEntries * lane;
        if (q_wave + kSchurSlice <= A.capacity) {
            const int4u jj = *reinterpret_cast<const int4u *>(lane_at(idx + q_wave, 16));
            const dbl2u *vv = reinterpret_cast<const dbl2u *>(lane_at(val + q_wave, 32));
            const dbl2u va = vv[0], vb = vv[1];
            bj[h][0] = jj.x;
            bj[h][1] = jj.y;
            bj[h][2] = jj.z;
            bj[h][3] = jj.w;
            bv[h][0] = va.x;
            bv[h][1] = va.y;
            bv[h][2] = vb.x;
            bv[h][3] = vb.y;
        } else {
#pragma unroll
            for (int e = 0; e < kSchurLaneEntries; ++e) {
                bj[h][e] = q + e < A.capacity ? idx[q + e] : -1;
                bv[h][e] = q + e < A.capacity ? val[q + e] : 0.0;
            }
        }
    };
#pragma unroll
    for (int h = 0; h < kSchurWaveSlices; ++h)
#pragma unroll
        for (int e = 0; e < kSchurLaneEntries; ++e) bj[h][e] = -1;
    auto load_trip = [&](int64_t base, int64_t end) {
#pragma unroll
        for (int h = 0; h < kSchurWaveSlices; ++h)
            if (base + h * (kSchurPartWaves * kSchurSlice) < end) load_slice(h, base);
    };
    load_trip(e0, e1);

    // the partial sums the state is advanced with
    const bool first = cur.first != 0;
    WaveParts prz, prr;
    if (ROWS) {
        const int count = first ? kSchurParts : A.vec_blocks;
        prz.fetch(A.part_rz[sys], count, lane);
        prr.fetch(A.part_rr[sys], count, lane);
    }

    // rows ra .. of the part, a thread per row: its entries, and what its result is made with
    const double *diag = ROWS ? A.row_sum : A.col_sum;
    const double *own = MODE == kSchurRows ? A.u[sys] : MODE == kSchurRowsFinal ? A.rhs[sys] : MODE == kSchurCols ? p_old : A.rhs[sys] + A.n;
    int64_t b0 = 0, b1 = 0;
    double dg = 1.0, mine = 0.0;
    auto load_rows = [&](int64_t ra, int cnt) {
        b0 = b1 = 0;
        if (tid < cnt) {
            b0 = ptr[ra + tid];
            b1 = ptr[ra + tid + 1];
            dg = diag[ra + tid];
            mine = own[ra + tid];
        }
    };
    int cnt = (int)(r1 - r0 < kSchurHeld ? r1 - r0 : kSchurHeld);
    load_rows(r0, cnt);
    // a share of p = z + ratio p_old is formed with every part (kSchurRows), or a share of x handed on (kSchurRowsFinal)
    const int64_t share0 = schur_share(A.mb, me);
    const int share = (int)(schur_share(A.mb, me + 1) - share0);
    double p_mine = 0.0, z_mine = 0.0;
    if (MODE == kSchurRows && tid < share) {
        p_mine = (p_old + share0)[tid];
        z_mine = (xs + share0)[tid];
    }

    double ratio = 0.0;
    bool done = false;
    if (ROWS) {
        SchurState nx = cur;
        if (!cur.done) {
            double norm = 0.0;
            if (first) {
                WaveParts parts;
                parts.fetch(A.part_norm[sys], A.norm_blocks, lane);
                norm = parts.sum();
            }
            nx = schur_advance(cur, prz.sum(), prr.sum(), norm, A.rtol);
        }
        if (MODE == kSchurRows) {
            if (me == 0 && tid == 0) A.state[2 * ((A.it + 1) & 1) + sys] = nx;
            done = nx.done != 0;
            ratio = nx.rz / cur.rz;
        } else if (me == 0 && tid == 0) {
            if ((A.it & 1) != 0) A.state[sys] = cur;  // (a later call goes on from there, with the partial sums as they are)
            double *info = A.info + 4 * sys;
            info[0] = (double)cur.steps;
            info[1] = (double)nx.done;
            info[2] = sqrt(nx.rr);
            info[3] = sqrt(nx.bb);
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the vector is in LDS
    if (MODE == kSchurRows && done) return;
    if (all_tid == 0) {
        if (nl & 1) S.xs[nl - 1] = fresh ? __builtin_fma(ratio, p_old[nl - 1], last) : last;
        S.xs[nl] = 0.0;
    }
    if (fresh && pairs > 0) {  // p in place of z (what this wave has put there)
        const auto put = [&](int k, const dbl2u &p) {
            const int at = (k * kWavesAll + all_w) * kLanes + lane;
            if (at < pairs) {
                S.xs[2 * at] = __builtin_fma(ratio, p.x, S.xs[2 * at]);
                S.xs[2 * at + 1] = __builtin_fma(ratio, p.y, S.xs[2 * at + 1]);
            }
        };
#pragma unroll
        for (int k = 0; k < kAhead; ++k) put(k, p_ahead[k]);
#pragma unroll 4
        for (int k = kAhead; k < kPer; ++k) put(k, p_pair(k));
    }
    if (MODE == kSchurRows) {
        for (int i = tid; i < share; i += kSchurPartThreads) {
            const double p = i == tid ? p_mine : (p_old + share0)[i], z = i == tid ? z_mine : (xs + share0)[i];
            (other + share0)[i] = first ? z : __builtin_fma(ratio, p, z);
        }
    }
    if (MODE == kSchurRowsFinal && A.x[sys] != A.x_out[sys] + A.n)
        for (int i = tid; i < share; i += kSchurPartThreads) (A.x_out[sys] + A.n + share0)[i] = (xs + share0)[i];

    const double inv_eta = 1.0 / A.eta;
    const SegmentedScan scan_wave(lane);
    const uint64_t up_to = ~0ull >> (kLanes - 1 - lane);  // this lane and the ones before it
    constexpr int kSums = MODE == kSchurColsRhs ? 2 : 1;
    double total[kSums] = {};
    for (int64_t rows = 0; rows < rows_max; rows += kSchurHeld) {
        const int64_t ra = r0 + rows;
        // the entries of the rows in hand, of a part with rows [q0, q1) and entries [p0, p1)
        auto begin = [&](int64_t q0, int64_t q1, int64_t p0, int64_t p1, int64_t at) {
            return at == 0 ? p0 : q0 + at < q1 ? clamp_entry(ptr[q0 + at], A.capacity) : p1;
        };
        const int64_t ea = begin(r0, r1, e0, e1, rows), eb = begin(r0, r1, e0, e1, rows + kSchurHeld);
        int64_t len = eb - ea;
        if (R == 2) {
            const int64_t len_b = begin(r0_b, r1_b, e0_b, e1_b, rows + kSchurHeld) - begin(r0_b, r1_b, e0_b, e1_b, rows);
            len = len > len_b ? len : len_b;
        }
        if (rows != 0) {
            cnt = (int)(r1 - ra < kSchurHeld ? r1 - ra : kSchurHeld);
            load_rows(ra, cnt);
            load_trip(ea, eb);
        }
        b0 = clamp_entry(b0, A.capacity);
        b1 = clamp_entry(b1, A.capacity);
        // the place of the row's sum: rows with entries before it
        const uint64_t filled = __ballot(b1 > b0);
        int rank = __builtin_popcountll(filled & (up_to >> 1));
        int ended = 0;  // rows that ended in the trips before
        double sum = 0.0;
        int par = 0;
        for (int64_t base = ea; base < ea + len; base += kSchurTrip, par ^= 1) {
            if (rows != 0 || base != ea) {
                __syncthreads();  // (what is in LDS of the trip before is done with)
                if (tid < kSchurTrip / 32) L.ends[tid] = 0;
                __syncthreads();
            }
            const bool open = b1 > b0 && b1 > base && b0 < base + kSchurTrip;  // the row has entries in this trip
            const int q0 = b0 >= base ? (int)(b0 - base) : -1, q1 = b1 - base > kSchurTrip ? kSchurTrip : (int)(b1 - base) - 1;
            if (open && q1 < kSchurTrip) atomicOr(&L.ends[q1 >> 5], 1u << (q1 & 31));
            if (lane == 0 && w < kSchurHeld / kLanes) L.filled[w] = __builtin_popcountll(filled);
            __syncthreads();
            if (base == ea) {
#pragma unroll
                for (int k = 0; k < kSchurHeld / kLanes - 1; ++k) rank += k < w ? L.filled[k] : 0;
            }
            // rows that end before the wave's slices: lane l counts half a slice; and the lane's four bits of each of the wave's
            unsigned bits[kSchurWaveSlices];
            const uint4 words = reinterpret_cast<const uint4 *>(L.ends)[lane];
            const int here = __builtin_popcount(words.x) + __builtin_popcount(words.y) + __builtin_popcount(words.z) + __builtin_popcount(words.w);
#pragma unroll
            for (int h = 0; h < kSchurWaveSlices; ++h)
                bits[h] = (L.ends[(h * kSchurPartWaves + w) * (kSchurSlice / 32) + (lane >> 3)] >> (4 * (lane & 7))) & 15u;
            const int ends_up_to = wave_scan(here), ends_before = ends_up_to - here;
            __syncthreads();
            // (entries of the vector that are not in LDS are asked for a slice ahead; lanes that need none read its first)
            double far[2][kSchurLaneEntries], far_p[2][kSchurLaneEntries];
            auto load_far = [&](int h) {
#pragma unroll
                for (int e = 0; e < kSchurLaneEntries; ++e) {
                    const unsigned j = (unsigned)bj[h][e];
                    const unsigned at = j >= (unsigned)nl && j < (unsigned)limit ? j : 0u;
                    far[h & 1][e] = xs[at];
                    if (fresh) far_p[h & 1][e] = p_old[at];
                }
            };
            if (!ALL) load_far(0);
#pragma unroll
            for (int h = 0; h < kSchurWaveSlices; ++h) {
                const int s = h * kSchurPartWaves + w;
                if (!ALL && h + 1 < kSchurWaveSlices) load_far(h + 1);
                if (base + h * (kSchurPartWaves * kSchurSlice) >= eb) break;
                const unsigned m = bits[h];
                double x[kSchurLaneEntries];
#pragma unroll
                for (int e = 0; e < kSchurLaneEntries; ++e) {
                    const unsigned j = (unsigned)bj[h][e];
                    x[e] = S.xs[j < (unsigned)nl ? j : (unsigned)nl];
                    if (!ALL && j >= (unsigned)nl && j < (unsigned)limit)
                        x[e] = fresh ? __builtin_fma(ratio, far_p[h & 1][e], far[h & 1][e]) : far[h & 1][e];
                }
                // t_e: of entry e's row, as far as it lies in the lane
                const double(&v)[kSchurLaneEntries] = bv[h];
                const double t0 = v[0] * x[0];
                const double t1 = __builtin_fma(v[1], x[1], (m & 1) ? 0.0 : t0);
                const double t2 = __builtin_fma(v[2], x[2], (m & 2) ? 0.0 : t1);
                const double t3 = __builtin_fma(v[3], x[3], (m & 4) ? 0.0 : t2);
                const double tail = (m & 8) ? 0.0 : t3;
                const uint64_t ends = __ballot(m != 0);
                int at = ended + __builtin_amdgcn_readlane(ends_before, 2 * s);
                if (__ballot((m & (m - 1)) != 0) != 0) {  // lanes in which several rows end
                    const int mine_ends = __builtin_popcount(m);
                    at += wave_scan(mine_ends) - mine_ends;
                    int k = at + 1;
                    if ((m & 2) && (m & 1)) L.sums[k++] = t1;
                    if ((m & 4) && (m & 3)) L.sums[k++] = t2;
                    if ((m & 8) && (m & 7)) L.sums[k] = t3;
                } else {
                    at += lanes_below(ends);
                }
                const double head = (m & 1) ? t0 : (m & 2) ? t1 : (m & 4) ? t2 : t3;
                // the tail together with the lanes before it, back to the last one in which a row ends
                const uint64_t before = ends & up_to;
                const double scan = scan_wave(tail, before != 0 ? lane - (63 - __builtin_clzll(before)) : lane);
                const double carry = dpp_f64<kDppWaveShr1>(scan);
                if (m != 0) L.sums[at] = carry + head;
                if (lane == kLanes - 1) L.tails[s] = scan;
                if (base + kSchurTrip + h * (kSchurPartWaves * kSchurSlice) < eb) load_slice(h, base + kSchurTrip);
            }
            ended += __builtin_amdgcn_readlane(ends_up_to, kLanes - 1);
            __syncthreads();
            // a row over several slices: the slices in order, then the end that is in sums[]
            if (open) {
                const int s_hi = q1 / kSchurSlice;  // (kSchurTripSlices: goes on in the next trip)
                int s = q0 / kSchurSlice;
                if (q0 < 0 || s < s_hi) {
                    double f;
                    if (q0 < 0) {
                        f = L.carry[par ^ 1];
                        s = 0;
                    } else {
                        f = L.tails[s];
                        ++s;
                    }
                    for (; s < s_hi; ++s) f += L.tails[s];
                    if (q1 < kSchurTrip) sum = f + L.sums[rank];
                    else L.carry[par] = f;
                } else {
                    sum = L.sums[rank];
                }
            }
        }
        if (tid < cnt) {
            const int64_t i = ra + tid;
            const double d = dg / A.eta + A.tau, bs = sum * inv_eta;
            if (MODE == kSchurRows) {
                const double v = bs / d;
                A.u[sys][i] = first || fresh ? v : __builtin_fma(ratio, mine, v);
            } else if (MODE == kSchurRowsFinal) {
                A.x_out[sys][i] = (mine - bs) / d;
            } else if (MODE == kSchurCols) {
                const double o = d * mine - bs;
                other[i] = o;
                total[0] += o * mine;
            } else {
                const double r = mine - bs, z = r / d;
                A.r[sys][i] = r;
                A.z[sys][i] = z;
                A.x[sys][i] = 0.0;
                total[0] += r * z;
                total[kSums - 1] += r * r;
            }
        }
    }
    if (!ROWS) {
        __syncthreads();
        schur_part_sums<kSums>(total, reinterpret_cast<double(*)[kSchurPartWaves]>(L.sums), lane, w);
        if (tid == 0) {
            if (MODE == kSchurCols) {
                A.part[sys][me] = total[0];
            } else {
                A.part_rz[sys][me] = total[0];
                A.part_rr[sys][me] = total[kSums - 1];
                if (me == 0) {
                    SchurState s{};
                    s.first = 1;
                    A.state[sys] = s;
                }
            }
        }
    }
}

// x += step p, r -= step S p, z = r / D2; partial sums of the new r^T z and r^T r
__global__ __launch_bounds__(kThreads) void schur_update_kernel(SchurArgs A)
{
    __shared__ double lds[2][kWaves];
    const int lane = threadIdx.x & (kLanes - 1), sys = (int)blockIdx.y;
    const int stride = (int)gridDim.x * kThreads;
    int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double d = 1.0, x = 0.0, r = 0.0, b0 = 0.0, b1 = 0.0;
    auto fetch = [&]() {
        d = A.col_sum[t];
        x = A.x[sys][t];
        r = A.r[sys][t];
        b0 = A.buf[sys][0][t];
        b1 = A.buf[sys][1][t];
    };
    // (everything is asked for before the state says which buffer is which)
    if (t < A.mb) fetch();
    WaveParts parts;
    parts.fetch(A.part[sys], kSchurParts, lane);
    const SchurState st = schur_state(A.state + 2 * ((A.it + 1) & 1) + sys);
    if (st.done) return;
    const double step = st.rz / parts.sum();
    double rz = 0.0, rr = 0.0;
    while (t < A.mb) {
        const double p = st.flip ? b1 : b0, Sp = st.flip ? b0 : b1;
        x += step * p;
        r = r - step * Sp;
        const double z = r / (d / A.eta + A.tau);
        rz += r * z;
        rr += r * r;
        A.x[sys][t] = x;
        A.r[sys][t] = r;
        A.z[sys][t] = z;
        t += stride;
        if (t < A.mb) fetch();
    }
    rz = wave_reduce1<OpSum>(rz);
    rr = wave_reduce1<OpSum>(rr);
    const int w = (int)(threadIdx.x >> 6);
    if (lane == 0) {
        lds[0][w] = rz;
        lds[1][w] = rr;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double s = lds[threadIdx.x][0];
#pragma unroll
        for (int q = 1; q < kWaves; ++q) s += lds[threadIdx.x][q];
        (threadIdx.x == 0 ? A.part_rz[sys] : A.part_rr[sys])[blockIdx.x] = s;
    }
}

}  // namespace regot
