// One Sinkhorn sweep (alpha half-step, then beta half-step) from ONE read of the cost matrix.
//
// Run as two half-steps a sweep reads M twice, because the beta update of a column needs the new alpha of every row.
// But the entries of a row are still on chip when the row's log-sum-exp is complete, and its exponentials are already
// formed: with e_ij = exp((beta_j - M_ij - max_i) / eta), S_i = sum_j e_ij and the new alpha_i = eta log a_i -
// (max_i + eta log S_i), the plan entry at (new alpha, old beta) is
//     T_ij = exp((alpha_i + beta_j - M_ij) / eta) = e_ij a_i / S_i,
// one multiplication instead of another exponential, and with c_j = sum_i T_ij the exact maximiser in beta is
//     beta_j + eta (log b_j - log c_j).
// T_ij <= a_i, so nothing overflows for masses that are anywhere near 1; a column whose c_j is so small that terms may have
// been lost to underflow, or that has no T (beta = -inf), is done again from alpha and M in the log domain
// (sweep_finalize_kernel).
//
// A row of 20000 doubles is 160 KB, too much for one compute unit to hold twice (the row being worked on and the one
// in flight) next to the column sums, so K = ceil(m / 3840) workgroups -- a cluster, one workgroup per compute unit --
// share a block of rows, each owning `width` columns.  Fifteen waves work on the matrix: a lane owns up to 4 columns, keeps
// their sums in registers for all rows of the block, has two batches of 4 rows in registers (the one whose exponentials are
// being formed and the one in flight) and the exponentials of the batch before in LDS.  The sixteenth wave
// finds the factors a_i / S_i: it publishes the workgroup's (max, sum) per row in the workspace, reads the other members',
// and has the time the workers take for the next batch to do it.  (It has to be a wave of its own: memory loads return in
// order, so a wave that also streams the matrix would see the other members' numbers only behind its own prefetch.)
// One barrier per batch.
//
// Where half the columns per workgroup make better use of the fifteen waves, K = ceil(m / 1920) workgroups take batches of
// eight rows instead: 4999 columns are 2500 of 3840 in two workgroups and 1667 of 1920 in three, and a workgroup has that
// much more in flight.  7001 x 4999 75 -> 69 us a sweep, 20000 x 4000 168 -> 151, 9000 x 9500 151 -> 141, 30000 x 1800
// 110 -> 96.  Not where the exchange is among more than kSweepMaxK8 workgroups (9000 x 12500, seven: 189 -> 195;
// 20000 x 20000, eleven: 607 -> 667), and not where a block has fewer than kSweepRows8 rows: a few batches of eight
// overlap less than twice as many of four (5000 x 1900, 20 rows: 28.3 -> 29.1; 2000 x 4999, 24: 32.2 -> 33.7;
// 8192 x 1500, 32: 32.4 -> 31.8).
//
// That is the first sweep of a call.  The ones behind it know how large their terms are and need no maxima: regot_sweep_near.hpp.
//
// What bounds it: instructions (32 an entry: with the loads taken out 447 us at 20000 x 20000) beside the memory.  20000 x 20000:
// 596 us a sweep = 5.4 TB/s of M against 975 us for the two half-steps (two reads at 6.6 TB/s; the sweeps behind the first one
// take 540); with the exponentials replaced by one operation 550 us.  A member's numbers take 0.8 us to reach the others, but the members of a cluster
// drift apart by up to the one batch (5 us) they are allowed; a cluster of one (m <= 3840) runs at 5.8 TB/s.  Measured on
// the way: seven workers with twice the columns each 616 us; all of a batch's loads requested at once 673 us (the waves then
// stand in line to issue them); counters in LDS instead of the barrier: no change; members on one die: no change.
// (With two groups of columns a wave two or three of the 128 registers are spilled: addresses of the results, written before the loops and
// read behind them.)
#pragma once

#include "regot_kernels.hpp"

namespace regot {

constexpr int kSweepWaves = 15;                              // that work on the matrix; one more finds the factors
constexpr int kSweepLanes = kSweepWaves * kLanes;
constexpr int kSweepThreads = kSweepLanes + kLanes;
constexpr int kSweepCols1 = kSweepWaves * 2 * kLanes;       // columns of a workgroup with one group of 128 per wave (1920)
constexpr int kSweepCols = 2 * kSweepCols1;                 // most columns a workgroup can own: two groups per wave (3840)
constexpr int kSweepMaxK8 = 5;                              // most members and fewest rows of a cluster whose batches are
constexpr int kSweepRows8 = 32;                             // eight rows (see above)
constexpr int64_t kSweepKeepTwo = 27000000;                 // most entries of a matrix whose sweeps alternate: two in a call,
constexpr int64_t kSweepKeep = 36000000;                    // and more of them (see SweepRows)
constexpr int kSweepMaxK = 16;                              // members of a cluster: one lane of a DPP row each
static_assert(kSweepWaves <= 16, "a DPP row of 16 lanes per row in sweep_factors");

// What an unpublished word holds: a NaN with all bits set.  Published NaNs have other bits.
constexpr unsigned long long kUnpublished = ~0ull;
constexpr int kSweepLooks = 1 << 14;  // at the words of the other members, one to two us each, before they are done without

// c_j below this is recomputed: what underflow takes from a term is below 3e-308 kSweepHuge, so from up to 2^31 of them
// less than 1e-16 of it.  Where a row's mass is beyond kSweepHuge (marginals are not asked to sum to 1), every column is.
constexpr double kSweepTiny = 1e-270;
constexpr double kSweepHuge = 1e12;
constexpr int kSweepHugeMark = 0x48554745;
// What sweep_finalize_kernel asks of masses, of b_j / c_j and of the duals before the terms of the next sweep are plan entries
// (regot_sweep_near.hpp).
constexpr double kNearLeastMass = 1e-150, kNearMostMass = 1e100, kNearLeastRatio = 1e-12, kNearMostDual = 1e13;  // the latter in units of eta

struct SweepArgs {
    int n, m;
    int64_t ldM;
    const double *M;
    const double *a, *b;
    double *alpha, *beta;
    double eta;
    int K, P;         // members of a cluster, clusters
    int width;        // columns per member (even; the last member may have fewer)
    double *exch;     // [n][K][2] published (max, sum); K > 1
    double *colpart;  // [P][m] column sums of a cluster's rows
    int *ticket;      // K > 1: number of workgroups that have started
    int looks;        // K > 1: kSweepLooks, or what a test asked for
    int splits;       // workgroups of sweep_finalize_kernel per 64 columns
    double *redo;     // splits > 1: [splits][2][m] (max, sum) of the columns that are done again
    int *redo_count;  // splits > 1: [groups of 64 columns] workgroups that have written theirs
    double floor, floor_max;  // see sweep_wave
    ExpParams ex;
    int *huge;        // [2] kSweepHugeMark in [turn]: a mass beyond kSweepHuge was met
    int *far;         // [2] [turn] not 0: it found that this sweep cannot
    double *alpha_out;  // what the pass writes: alpha, or an array that sweep_finalize_kernel copies to alpha
    int turn;         // parity of the sweep
    int up;           // the clusters take their rows from the last to the first (see SweepRows)
};

// The rows of a cluster in the order it takes them: t-th row of `count`, t beyond the last being the last again.
// Every other sweep of a call takes them from the last to the first, and M is read with ordinary loads (STREAM false): a sweep
// begins with the 32 MB that the one before it has left in the L2s.  (The last-level cache gives no more than the memory does:
// what limits either is between the dies.)  That takes a workgroup whose rows were last read on its own die: with one member the
// workgroup's id says which rows it has, and the grids are whole rounds over the dies; with several it is their order of arrival,
// which mostly comes out alike.
// All sweeps in order, with non-temporal loads, -> these, us a sweep in calls one behind the other: 2000 x 1900 16.0 -> 15.1, 3000^2
// 28.5 -> 26.9, 5000 x 3000 36.2 -> 33.7, 6000^2 64.7 -> 60.7.  Ordinary loads of a stream cost something (a single sweep of
// 10000^2, which has nothing to begin with, 152 -> 160), so the matrix must not be too large for 32 MB to make up for it, above
// all with two sweeps, of which one has a beginning.  us a call, of a caller that goes on with the matrix / has just written it /
// has new arrays:
//   two,   4000 x 5000   119 -> 114    124 -> 115    114 -> 112        6000^2   170 -> 156    165 -> 163    153 -> 155
//          6000 x 5000   149 -> 142    151 -> 151    143 -> 145        2000 x 20000   174 -> 165    172 -> 179    161 -> 161
//   three, 6000 x 5000   213 -> 204    219 -> 215    207 -> 205        6000^2   231 -> 213    235 -> 236    217 -> 218
//          7001 x 4999   238 -> 228    243 -> 246    225 -> 222        2000 x 20000   243 -> 223    246 -> 250    230 -> 227
//   four,  7000^2   365 -> 338    394 -> 413    -        10000^2   637 -> 624    672 -> 691    643 -> 693
//   ten,   5000^2   543 -> 521    580 -> 560    545 -> 531        6000^2   690 -> 633    698 -> 690    645 -> 639
struct SweepRows {
    int first, step, count;
    __device__ __forceinline__ int at(int t) const { return first + step * min(t, count - 1); }
};


// The arguments of the running kernel, fetched where this stands.  For code that hardly ever runs: what it needs would
// otherwise be fetched when the kernel starts, and there is not room for it (0.2 us a launch).
__device__ __forceinline__ SweepArgs sweep_args_here()
{
    typedef const __attribute__((address_space(4))) SweepArgs ArgsAt;
    ArgsAt *at = (ArgsAt *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    return *(const SweepArgs *)at;
}

__global__ __launch_bounds__(kThreads) void sweep_init_kernel(unsigned long long *exch, int64_t words, int *ticket)
{
    const int64_t i0 = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i0 == 0) *ticket = 0;
    for (int64_t i = i0; i < words; i += (int64_t)gridDim.x * kThreads) exch[i] = kUnpublished;
}

template <int NU, int R>
struct SweepShared {
    dbl2 prev[R][NU][kSweepLanes];  // a lane's exponentials of the batch before; read back by the same lane
    dbl2 beta[NU][kSweepLanes];                // a lane's beta; likewise
    dbl2 pairs[2][R][kSweepWaves];  // (max, sum) per row and wave, by parity of the batch
    double fac[2][R][kSweepWaves];  // what a wave's exponentials of a row are to be multiplied by
    int huge;                       // a row's mass is beyond kSweepHuge
};

// Batches a cluster works through; rows beyond the last are its last row again, with a factor of 0.  An even number of batches
// of four: eight rows are little to round up to.
template <int R>
__device__ __forceinline__ int sweep_batches(int rows)
{
    const int nb = (rows + R - 1) / R;
    return R == 4 ? (nb + 1) & ~1 : nb;
}

// The same for sweeps behind the first: an even number of batches where there are two sets of them.
template <int R, int LAG>
__device__ __forceinline__ int near_batches(int rows)
{
    const int nb = (rows + R - 1) / R;
    return LAG == 1 ? (nb + 1) & ~1 : nb;
}

// Reductions of 2 or 4 rows at once: row r ends up in lane 32 (r & 1) + 16 (r >> 1)
template <typename Op>
__device__ __forceinline__ double wave_reduce_rows(const double (&v)[2]) { return wave_reduce2<Op>(v[0], v[1]); }
template <typename Op>
__device__ __forceinline__ double wave_reduce_rows(const double (&v)[4]) { return wave_reduce4<Op>(v[0], v[1], v[2], v[3]); }

// R: rows of a batch, G of them at a time.
// NU: groups of 128 columns per wave, group u of wave w being columns c0 + 128 (15 u + w) + 2 lane + e.
// MASKED: not all of the wave's groups are full (the last columns of the member).
// The loads of a batch are issued by every wave unconditionally and in the same number, so that waiting for one batch
// never waits for the one requested behind it: where the member has no column a lane reads its last two again.
template <int NU, int R, bool STREAM, bool MASKED>
__device__ __forceinline__ void sweep_wave(const SweepArgs &A, SweepShared<NU, R> &L, int cluster, const SweepRows &rows,
                                           int c0, int ncol, int w, int lane)
{
    typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));  // 16 bytes wherever a double may lie
    constexpr int kStride = 2 * kLanes * kSweepWaves, G = R / 2;
    const int first = 2 * kLanes * w + 2 * lane;
    int nu = 0;         // groups that hold any column
    unsigned off[NU];   // byte offset of the pair a lane loads
    bool cv[NU][2], last[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int c = first + u * kStride;
        if (2 * kLanes * (u * kSweepWaves + w) < ncol) nu = u + 1;
        cv[u][0] = !MASKED || c < ncol;
        cv[u][1] = !MASKED || c + 1 < ncol;
        last[u] = MASKED && c == ncol - 1;                // its column is the second of the pair it loads
        off[u] = (unsigned)(MASKED ? min(c, ncol - 2) : c) * (unsigned)sizeof(double);
    }
    nu = MASKED ? __builtin_amdgcn_readfirstlane(nu) : NU;
    double csum[NU][2];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        csum[u][0] = csum[u][1] = 0.0;
        const double *src = A.beta + c0 + first + u * kStride;
        L.beta[u][threadIdx.x] = dbl2{cv[u][0] ? src[0] : 0.0, cv[u][1] ? src[1] : 0.0};
    }
    int floor_on = 0;  // (see before the loops below)
    double floor = -INFINITY, floor_max = -kDblMax;

    const double *M0 = A.M + (int64_t)rows.first * A.ldM + c0;
    const int64_t ld = rows.step * A.ldM;
    auto load_row = [&](double (&v)[NU][2], int row) {
        const double *prow = M0 + (int64_t)min(row, rows.count - 1) * ld;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const dbl2u *src = reinterpret_cast<const dbl2u *>(reinterpret_cast<const char *>(prow) + off[u]);
            const dbl2u x = STREAM ? __builtin_nontemporal_load(src) : *src;
            v[u][0] = x.x;
            v[u][1] = x.y;
        }
    };

    // One row: costs relative to wmax -> exponentials; returns the lane's sum
    auto exponentials = [&](double (&v)[NU][2], double wmax, int row) -> double {
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (MASKED && u >= nu) continue;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double t = exp_eta(v[u][e] - wmax, A.ex);
                if constexpr (MASKED) t = cv[u][e] ? t : 0.0;
                v[u][e] = t;
                acc += t;
            }
        }
        if (__ballot(not_finite(acc)) != 0) {
            // an infinite cost or an infinite beta in the row: again from memory, with the IEEE limits of exp
            acc = 0.0;
            floor_on = 1;
            const double *prow = M0 + (int64_t)min(row, rows.count - 1) * ld + first;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const dbl2 bet = L.beta[u][threadIdx.x];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    double t = 0.0;
                    if (first + u * kStride + e < ncol) {
                        t = exp_eta_any((bet[e] - prow[u * kStride + e]) - wmax, A.ex);
                        acc += t;
                    }
                    v[u][e] = t;
                }
            }
            // without this the code after the branch has to assume that these loads are still on their way, and waits
            // for everything requested since, the next batch included
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
        }
        return acc;
    };

    // Column sums of one row: its exponentials (in LDS, of two batches ago) times its factor
    auto accumulate = [&](const dbl2 (&x)[NU], double f) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            csum[u][0] = __builtin_fma(f, x[u].x, csum[u][0]);
            csum[u][1] = __builtin_fma(f, x[u].y, csum[u][1]);
            // (here and now: sunk to where the sums are needed next, the additions would keep all they read in registers)
            asm volatile("" : "+v"(csum[u][0]), "+v"(csum[u][1]));
        }
    };

    // Batch b: its costs are in `cur`, the exponentials of batch b - 1 in `old`, those of batch b - 2 in LDS, and their
    // factors are known.  Row by row: the column sums of batch b - 2, batch b - 1 to LDS, the costs of batch b + 1 requested
    // into its registers (behind the last batch: the last row again), and, G rows at a time, the exponentials of batch b.
    // The requests are spread over the batch because all waves are in step: requested at once they fill the memory
    // pipeline of the compute unit, and the waves wait to issue them instead of computing.
    auto batch = [&](auto floor_tag, int b, double (&cur)[R][NU][2], double (&old)[R][NU][2]) {
        constexpr bool FLOOR = decltype(floor_tag)::value;
        const int row0 = b * R, par = b & 1;
#pragma unroll
        for (int h = 0; h < R; h += G) {
            auto turn = [&](int r, dbl2 (&x)[NU]) {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    x[u] = L.prev[r][u][threadIdx.x];
                    L.prev[r][u][threadIdx.x] = dbl2{old[r][u][0], old[r][u][1]};
                }
                load_row(old[r], row0 + R + r);
                __builtin_amdgcn_sched_barrier(0);  // (in this order: what is waited for is counted from the youngest load)
            };
            dbl2 x[NU];
            turn(h, x);
            double lmax[G], lsum[G];
#pragma unroll
            for (int r = 0; r < G; ++r) lmax[r] = -INFINITY;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (MASKED && u >= nu) continue;
                const dbl2 bet = L.beta[u][threadIdx.x];
#pragma unroll
                for (int r = 0; r < G; ++r) {
                    double(&c)[2] = cur[h + r][u];
                    // (the subtraction stays here: moved to where the costs are requested it would have to wait for them)
                    asm volatile("" : "+v"(c[0]), "+v"(c[1]));
                    if (MASKED && last[u]) c[0] = c[1];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        c[e] = bet[e] - c[e];
                        if constexpr (FLOOR) c[e] = c[e] < floor ? floor : c[e];
                        if (cv[u][e]) lmax[r] = fmax(lmax[r], c[e]);
                    }
                }
            }
            // (at least -DBL_MAX, or above the floor: a segment of infinite costs gives terms 0 and an empty partial sum)
            const double mx = fmax(wave_reduce_rows<OpMax>(lmax), FLOOR ? floor_max : -kDblMax);
            accumulate(x, L.fac[par][h][w]);
            lsum[0] = exponentials(cur[h], read_lane(mx, 0), row0 + h);
#pragma unroll
            for (int r = 1; r < G; ++r) {
                turn(h + r, x);
                lsum[r] = exponentials(cur[h + r], read_lane(mx, 32 * (r & 1) + 16 * (r >> 1)), row0 + h + r);
                accumulate(x, L.fac[par][h + r][w]);
            }
            const double sm = wave_reduce_rows<OpSum>(lsum);
            if (lane % (kLanes / G) == 0) L.pairs[par][h + quad_row(lane)][w] = dbl2{mx, sm};
        }
        __syncthreads();
    };
    const int nb = sweep_batches<R>(rows.count);
    double v0[R][NU][2], v1[R][NU][2];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            L.prev[r][u][threadIdx.x] = dbl2{0.0, 0.0};
            v1[r][u][0] = v1[r][u][1] = 0.0;
        }
    // (the two batches before the first; read back by this wave only, before anyone writes it)
    if (lane < 2 * R) L.fac[lane / R][lane % R][w] = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) load_row(v0[r], r);
    __builtin_amdgcn_sched_barrier(0);
    // Terms that are -inf (an infinite cost, a column without mass) make the reduction of exp_eta a NaN.  A wave that has
    // met one, or has such a column, puts a finite floor under its terms from then on, low enough to give exactly 0 and to lie
    // below whatever a row can hold, so that it goes back to memory (below) once, not in every row: 1 % of the costs
    // infinite 1580 -> 647 us a sweep at 20000 x 20000 (the two half-steps 1106), a sixth of the columns without mass 1830 ->
    // 612 (1009), 100000 x 1000 with 1 % without 466 -> 214 (352).  Other waves do not pay for it: it is a loop of its own,
    // since three more operations an entry, or a branch around them, cost 2.5 %.  (A NaN stays one.)
    bool massless = false;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const dbl2 bet = L.beta[u][threadIdx.x];
        massless = massless || bet.x == -INFINITY || bet.y == -INFINITY;
    }
    if (__ballot(massless) != 0) floor_on = 1;
    int b = 0;
    for (; b + 1 < nb && floor_on == 0; b += 2) {
        batch(std::false_type{}, b, v0, v1);
        batch(std::false_type{}, b + 1, v1, v0);
    }
    if (b < nb) {
        const SweepArgs C = sweep_args_here();
        floor = C.floor;
        floor_max = C.floor_max;
    }
    for (; b + 1 < nb; b += 2) {
        batch(std::true_type{}, b, v0, v1);
        batch(std::true_type{}, b + 1, v1, v0);
    }
    if (R != 4 && (nb & 1)) {
        batch(std::true_type{}, nb - 1, v0, v1);  // (the floor changes no result; once is enough here)
        // (copied, so that what follows is there once: written out for either, it takes registers from the loop)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                v1[r][u][0] = v0[r][u][0];
                v1[r][u][1] = v0[r][u][1];
            }
    }
    // the last two batches: one in LDS, one in registers
    const int par = (nb - 1) & 1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        dbl2 x[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) x[u] = L.prev[r][u][threadIdx.x];
        accumulate(x, L.fac[par ^ 1][r][w]);
    }
    __syncthreads();
    const int huge = L.huge;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        dbl2 x[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) x[u] = dbl2{v1[r][u][0], v1[r][u][1]};
        accumulate(x, L.fac[par][r][w]);
    }
    if (__builtin_amdgcn_readfirstlane(huge) != 0) {  // these sums are not to be used
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) csum[u][e] = csum[u][e] == csum[u][e] ? -INFINITY : csum[u][e];
    }
    double *out = A.colpart + (int64_t)cluster * A.m + c0 + first;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (cv[u][0]) out[u * kStride] = csum[u][0];
        if (cv[u][1]) out[u * kStride + 1] = csum[u][1];
    }
}

// (max, sum) of the 16 lanes of a DPP row, each with a pair of its own.  (The products are rounded before they are added, so
// that two places in the code cannot differ in that.)
__device__ __forceinline__ dbl2 merge_pairs16(dbl2 pair, const ExpParams &ex)
{
#pragma clang fp contract(off)
    const double mx = row16_reduce<OpMax>(pair.x);
    const double scaled = pair.y * exp_eta_any(pair.x - mx, ex);
    return dbl2{mx, row16_reduce<OpSum>(scaled)};
}

// What a member publishes for a row: the (max, sum) of each of its waves as sweep_wave forms them, and of those as
// sweep_factors does, operation by operation, by one wave.  For a member that is not there in time.
template <int NU, int R>
__device__ __forceinline__ dbl2 sweep_member_row(const SweepArgs &A, int row, int member, int lane)
{
    const int c0 = member * A.width, ncol = min(A.width, A.m - c0);
    const double *src = A.M + (int64_t)row * A.ldM + c0, *beta = A.beta + c0;
    dbl2 mine{-kDblMax, 0.0};
#pragma unroll 1
    for (int w = 0; w < kSweepWaves; ++w) {
        double v[NU][2], all[R / 2], acc = 0.0, lmax = -INFINITY;
        bool in[NU][2];
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = 2 * kLanes * (u * kSweepWaves + w) + 2 * lane + e;
                in[u][e] = c < ncol;
                v[u][e] = in[u][e] ? beta[c] - src[c] : 0.0;
                if (in[u][e]) lmax = fmax(lmax, v[u][e]);
            }
#pragma unroll
        for (int r = 0; r < R / 2; ++r) all[r] = lmax;
        const double mx = fmax(wave_reduce_rows<OpMax>(all), -kDblMax);
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) acc += in[u][e] ? exp_eta_any(v[u][e] - mx, A.ex) : 0.0;
#pragma unroll
        for (int r = 0; r < R / 2; ++r) all[r] = acc;
        const double sum = wave_reduce_rows<OpSum>(all);
        if ((lane & 15) == w) mine = dbl2{mx, sum};
    }
    return merge_pairs16(mine, A.ex);
}

// The factors of every batch, by one wave: lanes 16 r + j work on rows r, r + 4 of the batch, j being a wave of the
// workgroup or a member of the cluster.
template <int NU, int R>
__device__ __forceinline__ void sweep_factors(const SweepArgs &A, SweepShared<NU, R> &L, int member, const SweepRows &rows, int lane)
{
    constexpr int Q = R / 4;
    const int r16 = lane >> 4, j16 = lane & 15;
    const int nb = sweep_batches<R>(rows.count);
    unsigned long long *exch = reinterpret_cast<unsigned long long *>(A.exch);
    int patience = A.looks;
    // (now, while the workers wait for their first rows)
    bool huge = false;
    for (int t = lane; t < rows.count; t += kLanes) huge = huge || A.a[rows.at(t)] > kSweepHuge;
    if (__ballot(huge) != 0 && lane == 0) {
        L.huge = 1;
        A.huge[A.turn] = kSweepHugeMark;
    }
    __builtin_amdgcn_s_setprio(3);  // a few instructions that fifteen waves wait for (50000 x 50000: 4.23 -> 4.00 ms a sweep)
    for (int b = 0; b < nb; ++b) {
        const int par = b & 1;
        int row[Q];
        bool live[Q];
        double ai[Q], mx[Q], sum[Q];
        dbl2 mine[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int t = b * R + 4 * q + r16;
            live[q] = t < rows.count;
            row[q] = rows.at(t);
            ai[q] = A.a[row[q]];
        }
        __syncthreads();  // the workers' (max, sum) of batch b are there
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            mine[q] = j16 < kSweepWaves ? L.pairs[par][4 * q + r16][j16] : dbl2{-kDblMax, 0.0};
            const dbl2 own = merge_pairs16(mine[q], A.ex);
            mx[q] = own.x;
            sum[q] = own.y;
        }
        if (A.K > 1) {
            unsigned long long x[Q], y[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                unsigned long long word = (unsigned long long)__double_as_longlong(j16 == 0 ? mx[q] : sum[q]);
                if (word == kUnpublished) word = 0x7ff8000000000000ull;
                if (j16 < 2 && live[q])
                    __hip_atomic_store(exch + ((int64_t)row[q] * A.K + member) * 2 + j16, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                x[q] = y[q] = 0;
            }
            // The other members run, or will as soon as a compute unit is free (see sweep_pass_kernel).  How long that takes is
            // up to whatever else is on the device, so nothing depends on it: what is not there after kSweepLooks looks
            // (some 20 ms) is computed from M, the same bits, and then after one look a batch until all are there again.
            // (Looks, not time: a queue that is switched out does not look.)
            bool late = false;
            for (int left = patience;; --left) {
                bool missing = false;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (live[q] && j16 < A.K) {
                        const unsigned long long *src = exch + ((int64_t)row[q] * A.K + j16) * 2;
                        x[q] = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        y[q] = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) missing = missing || x[q] == kUnpublished || y[q] == kUnpublished;
                late = __ballot(missing) != 0;
                if (!late || left <= 0) break;
            }
            patience = late ? 0 : A.looks;
            if (late) {
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    unsigned long long open = __ballot(x[q] == kUnpublished || y[q] == kUnpublished);
                    while (open != 0) {
                        const int at = __builtin_ctzll(open);
                        open &= open - 1;
                        const dbl2 pair = sweep_member_row<NU, R>(A, rows.at(b * R + 4 * q + (at >> 4)), at & 15, lane);
                        if (lane == at) {
                            x[q] = (unsigned long long)__double_as_longlong(pair.x);
                            y[q] = (unsigned long long)__double_as_longlong(pair.y);
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const bool take = live[q] && j16 < A.K;
                const double px = take ? __longlong_as_double((long long)x[q]) : -kDblMax;
                const double py = take ? __longlong_as_double((long long)y[q]) : 0.0;
                const dbl2 whole = merge_pairs16(dbl2{px, py}, A.ex);
                mx[q] = whole.x;
                sum[q] = whole.y;
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool fine = sum[q] > 0.0 && sum[q] <= kDblMax && ai[q] >= 0.0 && ai[q] <= kDblMax;
            const double scale = fine ? ai[q] / sum[q] : __builtin_nan("");  // NaN: every column is done again from alpha and M
            if (j16 < kSweepWaves) L.fac[par][4 * q + r16][j16] = live[q] ? scale * exp_eta_any(mine[q].x - mx[q], A.ex) : 0.0;
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (b % A.K == member && j16 == 0 && live[q]) A.alpha_out[row[q]] = A.eta * log(ai[q]) - (mx[q] + A.eta * log(sum[q]));
    }
    __syncthreads();
}

}  // namespace regot

#include "regot_sweep_near.hpp"

namespace regot {

// Which member of which cluster a workgroup is follows from the order in which the workgroups start (a counter in the
// workspace): only the cluster formed last can be incomplete while its members wait for each other, and the clusters
// before it finish whatever happens, so a place for the missing members comes free unless other kernels hold all that is
// left, or the stream may use fewer compute units than a cluster has members; then they are waited for for a while and
// done without (see sweep_factors).  Which workgroup does what has no influence on the results.
// R: rows of a batch of a sweep that finds its rows' maxima; the others take four.  NEAR: it may be one of those (a kernel of its own, since
// what it has to look up first and the registers it takes cost the others 0.4 us).
template <int NU, int R, bool STREAM, bool NEAR>
__global__ __launch_bounds__(kSweepThreads) REGOT_WAVES_ATTR(4) void sweep_pass_kernel(SweepArgs A)
{
    static_assert(NU * R <= 8 && (R == 4 || R == 8), "registers and LDS of a lane; rows of sweep_factors");
    constexpr int LAG = NU == 1 && R == 8 ? 3 : 1;
    typedef SweepNear<NU, 4, LAG> Near;
    union Shared {
        SweepShared<NU, R> first;
        Near near;
    };
    __shared__ __attribute__((aligned(16))) char lds[NEAR ? sizeof(Shared) : sizeof(SweepShared<NU, R>)];
    __shared__ int lds_role;
    SweepShared<NU, R> &L = *reinterpret_cast<SweepShared<NU, R> *>(lds);
    Near &N = *reinterpret_cast<Near *>(lds);
    const int lane = threadIdx.x & (kLanes - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool near = NEAR && *((const __attribute__((address_space(4))) int *)A.far + A.turn) == 0;
    if (threadIdx.x == 0) {
        if (!near) L.huge = 0;
        lds_role = A.K > 1 ? atomicAdd(A.ticket, 1) : (int)blockIdx.x;
    }
    __syncthreads();
    const int role = __builtin_amdgcn_readfirstlane(lds_role);
    if (role < 0 || role >= A.P * A.K) return;
    const int cluster = role / A.K, member = role - cluster * A.K;
    int r_begin, r_end;
    chunk_rows(cluster, A.P, A.n, r_begin, r_end);
    const SweepRows rows{A.up ? r_end - 1 : r_begin, A.up ? -1 : 1, r_end - r_begin};
    const int c0 = member * A.width;
    const int ncol = min(A.width, A.m - c0);
    if (w == kSweepWaves) {
        const SweepArgs C = sweep_args_here();
        if (role == 0 && lane == 0) C.huge[C.turn ^ 1] = C.far[C.turn ^ 1] = 0;  // (last read behind the sweep before)
        if (role == 0 && C.splits > 1)  // (for sweep_finalize_kernel)
            for (int i = lane; i < (C.m + kLanes - 1) / kLanes; i += kLanes) C.redo_count[i] = 0;
        if (NEAR && near) near_factors<NU, 4, LAG>(C, N, member, rows, lane);
        else sweep_factors<NU, R>(C, L, member, rows, lane);
        return;
    }
    const bool full = 2 * kLanes * ((NU - 1) * kSweepWaves + w + 1) <= ncol;  // the wave's last group is
    if (NEAR && near) {
        if (full) near_wave<NU, 4, LAG, STREAM, false>(A, N, cluster, rows, c0, ncol, w, lane);
        else near_wave<NU, 4, LAG, STREAM, true>(A, N, cluster, rows, c0, ncol, w, lane);
    } else {
        if (full) sweep_wave<NU, R, STREAM, false>(A, L, cluster, rows, c0, ncol, w, lane);
        else sweep_wave<NU, R, STREAM, true>(A, L, cluster, rows, c0, ncol, w, lane);
    }
}

// Column sums over the clusters and the new beta; 64 columns per workgroup, one wave per share of the clusters.  Also
// clears the exchange words and the counter for the next sweep.
//
// A column whose sum is too small is done again from alpha and M, as the beta half-step is written.  That is every column
// whose beta is -inf (mass 0: there is no T), where one finite cost settles it, and columns so far below the others that all
// of their T underflow: with eta = 1e-4 some in the first sweep from zero.  For those the `splits` workgroups of a group of
// 64 columns share the rows; the last of them to be ready puts the parts together.  All but the first see from a few of
// the sums that there is nothing to do, nearly always, and cost next to nothing then.  Gaussian clouds in ten dimensions,
// one sweep from zero, us, eta = 1e-3 / 1e-4 / 3e-5: 3000^2 33 / 52 / 54, 10000^2 166 / 190 / 265, 20000^2 619 / 646 /
// 976; by the one workgroup that has a column, row after row: 33 / 352 / 340, 164 / 1190 / 1061, 616 / 2690 / 4220; the
// two half-steps: 53, 275, 988.
constexpr int kSweepFinWaves = 16;
constexpr int kSweepFinRows = 8;       // rows of a column that a lane asks for at a time
constexpr int kSweepMaxSplits = 16;
constexpr int kSweepMerge = 4;         // of their results asked for at a time

// NEAR: for calls whose later sweeps may be those of regot_sweep_near.hpp.  (What it does for them costs 0.3 us.)
template <bool NEAR>
__global__ __launch_bounds__(kSweepFinWaves *kLanes) REGOT_WAVES_ATTR(8) void sweep_finalize_kernel(SweepArgs A)
{
    __shared__ double lds_a[kSweepFinWaves][kLanes], lds_b[kSweepFinWaves][kLanes];
    __shared__ unsigned long long lds_bad;
    const int l = threadIdx.x & (kLanes - 1);
    const int sub = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int group = (int)blockIdx.x, split = (int)blockIdx.y;
    const int64_t j = (int64_t)group * kLanes + l;
    const bool live = j < A.m;
    if (A.K > 1) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *A.ticket = 0;
        const int64_t words = split == 0 ? (int64_t)A.n * A.K * 2 : 0;
        unsigned long long *ex = reinterpret_cast<unsigned long long *>(A.exch);
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += (int64_t)gridDim.x * blockDim.x)
            ex[i] = kUnpublished;
    }
    double bo = 0.0, bj = 1.0;  // (asked for before the sums are there)
    if (live && sub == 0 && split == 0) {
        bo = A.beta[j];
        bj = A.b[j];
    }
    // what becomes of row i0, asked for now and looked at behind the columns
    const int64_t i0 = (int64_t)group * blockDim.x + threadIdx.x;
    double mass0 = 0.0, alpha0 = 0.0;
    if (NEAR && split == 0 && i0 < A.n) {
        mass0 = A.a[i0];
        alpha0 = A.alpha_out[i0];
    }
    if (split > 0) {
        const int huge = A.huge[A.turn];
        // nothing to do, usually: sixteen of the clusters' sums are enough to see it (a sum of all is no smaller than a part
        // of it, up to rounding)
        lds_a[sub][l] = live ? A.colpart[(int64_t)(sub * A.P / kSweepFinWaves) * A.m + j] : 1.0;
        __syncthreads();
        if (sub == 0) {
            double c = lds_a[0][l];
            if (A.P >= kSweepFinWaves)
#pragma unroll
                for (int q = 1; q < kSweepFinWaves; ++q) c += lds_a[q][l];
            const unsigned long long open = __ballot(!(c >= 2.0 * kSweepTiny) || huge == kSweepHugeMark);
            if (l == 0) lds_bad = open;
        }
        __syncthreads();
        if (lds_bad == 0) return;
        __syncthreads();
    }
    double s = 0.0;
    if (live) {
#pragma unroll 4
        for (int p = sub; p < A.P; p += kSweepFinWaves) s += A.colpart[(int64_t)p * A.m + j];
    }
    lds_a[sub][l] = s;
    __syncthreads();
    if (sub == 0) {
        double c = lds_a[0][l];
#pragma unroll
        for (int q = 1; q < kSweepFinWaves; ++q) c += lds_a[q][l];
        // (c is NaN only where an alpha is NaN or +inf -- a NaN among a row's costs, or no finite one -- and so is then every
        // log-sum-exp of a column: NaN is the result)
        const bool ok = !live || c >= kSweepTiny || c != c;
        const double bn = bo + A.eta * (log(bj) - log(c));
        if (live && ok && split == 0) A.beta[j] = bn;
        const unsigned long long bad = __ballot(!ok);
        if (l == 0) lds_bad = bad;
        // (a column without mass must have been -inf, so that no T of it is in the rows' sums; what becomes of it is seen below)
        const bool near = bj > 0.0 ? ok && bj <= kNearMostMass && bj >= kNearLeastRatio * c && __builtin_fabs(bn) <= kNearMostDual * A.eta
                                   : bj == 0.0 && bo == -INFINITY;
        if (NEAR && split == 0 && __ballot(live && !near) != 0 && l == 0) A.far[A.turn ^ 1] = 1;
    }
    if (NEAR && split == 0) {
        // the new alpha, for the caller and the next sweep, which may have to find its maxima for some row's sake
        bool far = false;
        for (int64_t i = i0; i < A.n; i += (int64_t)gridDim.x * blockDim.x) {
            if (i != i0) {
                mass0 = A.a[i];
                alpha0 = A.alpha_out[i];
            }
            far = far || !(mass0 > 0.0 ? mass0 >= kNearLeastMass && mass0 <= kSweepHuge && __builtin_fabs(alpha0) <= kNearMostDual * A.eta
                                       : mass0 == 0.0 && alpha0 == -INFINITY);
            if (A.alpha_out != A.alpha) A.alpha[i] = alpha0;
        }
        if (__ballot(far) != 0 && l == 0) A.far[A.turn ^ 1] = 1;
    }
    __syncthreads();
    const unsigned long long bad = lds_bad;
    if (bad == 0) return;
    const SweepArgs C = sweep_args_here();
    const bool redo = ((bad >> l) & 1) != 0;
    bj = redo ? A.b[j] : 1.0;
    const int64_t per = ((int64_t)C.n + C.splits - 1) / C.splits, r0 = split * per, r1 = r0 + per < C.n ? r0 + per : C.n;
    const auto *alpha = (const __attribute__((address_space(4))) double *)C.alpha_out;  // (complete: written by the pass)
    double mx = -kDblMax, sum = 0.0;
    for (int64_t i = r0 + sub; i < r1; i += kSweepFinWaves * kSweepFinRows) {
        // (a column without mass is -inf as soon as it has one finite cost)
        const bool need = redo && (bj != 0.0 || sum == 0.0);
        if (__ballot(need) == 0) break;
        double v[kSweepFinRows], nm = mx;
        const double *src = C.M + i * C.ldM + j;
#pragma unroll
        for (int q = 0; q < kSweepFinRows; ++q) v[q] = need && i + q * kSweepFinWaves < r1 ? src[q * kSweepFinWaves * C.ldM] : INFINITY;
#pragma unroll
        for (int q = 0; q < kSweepFinRows; ++q) {
            const int64_t row = i + q * kSweepFinWaves;
            v[q] = alpha[row < r1 ? row : r1 - 1] - v[q];
        }
#pragma unroll
        for (int q = 0; q < kSweepFinRows; ++q) nm = fmax(nm, v[q]);
        if (__ballot(nm > mx) != 0) {
            sum *= exp_eta_any(mx - nm, C.ex);
            mx = nm;
        }
#pragma unroll
        for (int q = 0; q < kSweepFinRows; ++q) {
            const double d = v[q] - mx;
            // (where eta is so small that columns are done again, most terms are 0)
            if (__ballot(d * C.ex.c1 >= -1100.0) != 0) sum += exp_eta_any(d, C.ex);
        }
    }
    __syncthreads();
    lds_a[sub][l] = mx;
    lds_b[sub][l] = sum;
    __syncthreads();
    if (sub != 0) return;
#pragma unroll
    for (int q = 1; q < kSweepFinWaves; ++q) mx = fmax(mx, lds_a[q][l]);
    sum = 0.0;
#pragma unroll
    for (int q = 0; q < kSweepFinWaves; ++q) sum += lds_b[q][l] * exp_eta_any(lds_a[q][l] - mx, C.ex);
    if (C.splits > 1) {
        unsigned long long *mine = reinterpret_cast<unsigned long long *>(C.redo) + 2 * (int64_t)split * C.m + j;
        if (redo) {
            __hip_atomic_store(mine, (unsigned long long)__double_as_longlong(mx), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(mine + C.m, (unsigned long long)__double_as_longlong(sum), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        int before = 0;
        if (l == 0) before = __hip_atomic_fetch_add(C.redo_count + group, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(before) != C.splits - 1) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        double pm[kSweepMerge];  // (requested together)
        mx = -kDblMax;
        sum = 0.0;
        for (int q0 = 0; q0 < C.splits; q0 += kSweepMerge) {
            double ps[kSweepMerge], nm = mx;
#pragma unroll
            for (int q = 0; q < kSweepMerge; ++q) {
                const double *part = C.redo + 2 * (int64_t)(q0 + q) * C.m + j;
                const bool on = redo && q0 + q < C.splits;
                pm[q] = on ? part[0] : -kDblMax;
                ps[q] = on ? part[C.m] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < kSweepMerge; ++q) nm = fmax(nm, pm[q]);
            sum *= exp_eta_any(mx - nm, C.ex);
            mx = nm;
#pragma unroll
            for (int q = 0; q < kSweepMerge; ++q) sum += ps[q] * exp_eta_any(pm[q] - mx, C.ex);
        }
    }
    const double bn = A.eta * log(bj) - (mx + A.eta * log(sum));
    if (redo) A.beta[j] = bn;
    // (one that is not -inf again -- no mass and no finite cost: NaN -- is for the maxima to pass on)
    if (NEAR && __ballot(redo && bn != -INFINITY) != 0 && l == 0) C.far[C.turn ^ 1] = 1;
}

}  // namespace regot
