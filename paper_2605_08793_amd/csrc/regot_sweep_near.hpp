// The sweeps of a call behind its first one (see regot_sweep.hpp, which this is part of).
//
// After a sweep, alpha and beta are such that the plan entries of the next one are of known size: T_ij <= c_j before the update of
// beta_j and T_ij b_j / c_j <= b_j after it, so that a row sums up to something between a_i min_j b_j / c_j and the sum of b.
// Relative to the old alpha, the terms of a row are plan entries e_ij = exp((alpha_i + beta_j - M_ij) / eta), S_i = sum_j e_ij,
// and the new alpha_i is alpha_i + eta (log a_i - log S_i), the plan entry at it e_ij a_i / S_i: there is no maximum to be found
// before the exponentials, no other one than the row's own to bring a wave's sum to, and one number to publish instead of two.
// sweep_finalize_kernel checks what that takes: no column redone, infinite or NaN, masses and b_j / c_j far from the limits of a double
// (kNear*), so that sums of a row lie between 1e-162 and 1e112 and their factors below 1e12 (as a term's underflow has to be
// small in a column's sum: kSweepTiny), and duals whose rounding errors are small against eta.  Where it finds otherwise, the sweep
// finds its rows' maxima as the first one does (`far`).
//
// Per entry that is 21 vector instructions instead of 32 (no maximum, one reduction over the wave for four rows instead of four for two pairs).
// With the loads taken out a sweep of 20000 x 20000 went from 447 to 375 us, so it no longer competes with the memory (470 for a kernel that only reads).
// Also, a row of exponentials goes to LDS one row before the costs that take its registers are requested: requested right behind the store they
// wait for it, and the whole compute unit's requests with them (550 -> 532).  Passes alone, us, before and after: 20000 x 20000 600 -> 532,
// 10000 x 10000 143 -> 134, 20000 x 3840 106 -> 102, 7001 x 4999 66 -> 60, 3000 x 3000 27.5 -> 25.8.  What bounds it now: the memory at what this
// pattern of rows gets (505 without waiting for the other members' numbers, whatever the arithmetic), and that waiting.
// Blocks of two batches (1600 x 1200: 8 rows) gain nothing in the pass and lose 0.6 us a sweep around it, hence the line at 8 rows
// (SweepPlan::later): 1600 x 1200 138 us by maxima against 144 for ten sweeps, 1400 x 3000 181 / 184; 2300 x 1200, 9 rows, 179 / 177; 3000 x 3000 267 / 256;
// 600 x 20000, 14 rows in six members, 192 / 182 for six.
#pragma once

namespace regot {

// R: rows of a batch.  LAG: a batch's factors are used LAG + 1 batches later, the exponentials of kSets batches being kept until
// then, the older half of them in LDS; the costs of kSets / 2 batches are requested ahead.
template <int NU, int R, int LAG>
struct SweepNear {
    static_assert(R == 4 && (LAG == 1 || LAG == 3) && NU * R * (LAG + 1) <= 16, "registers and LDS of a lane");
    static constexpr int kSets = LAG + 1;
    static constexpr int kSlots = kSets / 2;
    dbl2 prev[kSlots][R][NU][kSweepLanes];   // a lane's exponentials; read back by the same lane
    dbl2 beta[NU][kSweepLanes];              // a lane's beta; likewise
    double sums[2][R][kSweepWaves];          // per row and wave, by parity of the batch
    double fac[kSets][R];                    // what the exponentials of a row are to be multiplied by
    double minus_alpha[2][R];                // what the costs of a row are relative to
};

// What the costs of row i are relative to: -alpha_i, as long as that is finite (a row without mass has terms of exactly 0 then,
// and near_factors sees from its alpha what it is).
__device__ __forceinline__ double near_minus_alpha(const SweepArgs &A, int row) { return -fmax(A.alpha[row], A.floor); }

template <int NU, int R, int LAG, bool STREAM, bool MASKED>
__device__ __forceinline__ void near_wave(const SweepArgs &A, SweepNear<NU, R, LAG> &L, int cluster, const SweepRows &rows,
                                          int c0, int ncol, int w, int lane)
{
    typedef double dbl2u __attribute__((ext_vector_type(2), aligned(8)));  // 16 bytes wherever a double may lie
    constexpr int kStride = 2 * kLanes * kSweepWaves, kSets = LAG + 1, kSlots = kSets / 2;
    const int first = 2 * kLanes * w + 2 * lane;
    int nu = 0;
    unsigned off[NU];
    bool cv[NU][2], last[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int c = first + u * kStride;
        if (2 * kLanes * (u * kSweepWaves + w) < ncol) nu = u + 1;
        cv[u][0] = !MASKED || c < ncol;
        cv[u][1] = !MASKED || c + 1 < ncol;
        last[u] = MASKED && c == ncol - 1;
        off[u] = (unsigned)(MASKED ? min(c, ncol - 2) : c) * (unsigned)sizeof(double);
    }
    nu = MASKED ? __builtin_amdgcn_readfirstlane(nu) : NU;
    double csum[NU][2];
    bool massless = false;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        csum[u][0] = csum[u][1] = 0.0;
        const double *src = A.beta + c0 + first + u * kStride;
        const dbl2 bet{cv[u][0] ? src[0] : 0.0, cv[u][1] ? src[1] : 0.0};
        L.beta[u][threadIdx.x] = bet;
        massless = massless || bet.x == -INFINITY || bet.y == -INFINITY;
    }
    int floor_on = __ballot(massless) != 0 ? 1 : 0;
    double floor = -INFINITY;

    const double *M0 = A.M + (int64_t)rows.first * A.ldM + c0;
    const int64_t ld = rows.step * A.ldM;
    const double *next = M0;     // the row to be requested next
    int behind = rows.count - 1; // rows that follow it
    auto load_row = [&](double (&v)[NU][2]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const dbl2u *src = reinterpret_cast<const dbl2u *>(reinterpret_cast<const char *>(next) + off[u]);
            const dbl2u x = STREAM ? __builtin_nontemporal_load(src) : *src;
            v[u][0] = x.x;
            v[u][1] = x.y;
        }
        next += behind > 0 ? ld : 0;
        --behind;
    };
    auto exponentials = [&](double (&v)[NU][2], double ref, int row) -> double {
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            if (MASKED && u >= nu) continue;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                double t = exp_eta(v[u][e] - ref, A.ex);
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
                        t = exp_eta_any((bet[e] - prow[u * kStride + e]) - ref, A.ex);
                        acc += t;
                    }
                    v[u][e] = t;
                }
            }
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0), as in sweep_wave
        }
        return acc;
    };
    auto accumulate = [&](const dbl2 (&x)[NU], double f) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            csum[u][0] = __builtin_fma(f, x[u].x, csum[u][0]);
            csum[u][1] = __builtin_fma(f, x[u].y, csum[u][1]);
            asm volatile("" : "+v"(csum[u][0]), "+v"(csum[u][1]));
        }
    };

    double v[kSets][R][NU][2];
    dbl2 x[NU];  // exponentials whose row's factor is known: those of batch b - LAG - 1, on their way from LDS to the column sums
    auto turn = [&](dbl2 (&lds)[NU][kSweepLanes], const double (&old)[NU][2]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            x[u] = lds[u][threadIdx.x];
            lds[u][threadIdx.x] = dbl2{old[u][0], old[u][1]};
        }
    };
#pragma unroll
    for (int u = 0; u < NU; ++u) x[u] = dbl2{0.0, 0.0};
    // Batch b, b % kSets == SET: its costs are in set SET.  Row by row: the column sums of batch b - kSets, whose exponentials are in
    // LDS; in their place those of batch b - kSets / 2; in the place of these the costs of batch b + kSets / 2 requested.
    auto batch = [&](auto floor_tag, auto set_tag, int b) {
        constexpr bool FLOOR = decltype(floor_tag)::value;
        constexpr int SET = decltype(set_tag)::value, SLOT = SET % kSlots;
        double(&cur)[R][NU][2] = v[SET];
        double(&old)[R][NU][2] = v[(SET + kSlots) % kSets];
        double lsum[R], fac[R], ref[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            fac[r] = L.fac[SET][r];
            ref[r] = L.minus_alpha[b & 1][r];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            load_row(old[r]);
            __builtin_amdgcn_sched_barrier(0);  // (in this order: what is waited for is counted from the youngest load)
            accumulate(x, fac[r]);
            // the next row's turn in LDS, which makes room for the next request
            if (r + 1 < R) turn(L.prev[SLOT][r + 1], old[r + 1]);
            else turn(L.prev[(SET + 1) % kSlots][0], v[(SET + 1 + kSlots) % kSets][0]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (MASKED && u >= nu) continue;
                const dbl2 bet = L.beta[u][threadIdx.x];
                double(&c)[2] = cur[r][u];
                // (the subtraction stays here: moved to where the costs are requested it would have to wait for them)
                asm volatile("" : "+v"(c[0]), "+v"(c[1]));
                if (MASKED && last[u]) c[0] = c[1];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    c[e] = bet[e] - c[e];
                    if constexpr (FLOOR) c[e] = c[e] < floor ? floor : c[e];
                }
            }
            lsum[r] = exponentials(cur[r], ref[r], b * R + r);
        }
        const double sm = wave_reduce4<OpSum>(lsum[0], lsum[1], lsum[2], lsum[3]);
        if ((lane & 15) == 0) L.sums[b & 1][quad_row(lane)][w] = sm;
        __syncthreads();
    };
    const int nb = near_batches<R, LAG>(rows.count);
#pragma unroll
    for (int k = 0; k < kSets; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                if (k < kSlots) L.prev[k][r][u][threadIdx.x] = dbl2{0.0, 0.0};
                if (k >= kSlots) v[k][r][u][0] = v[k][r][u][1] = 0.0;
            }
    {
        const SweepArgs C = sweep_args_here();
        floor = C.floor;
        if (lane < kSets * R) (&L.fac[0][0])[lane] = 0.0;  // (the same in all waves, as what follows)
        if (lane < 2 * R) (&L.minus_alpha[0][0])[lane] = near_minus_alpha(C, rows.at(lane));
    }
#pragma unroll
    for (int k = 0; k < kSlots; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) load_row(v[k][r]);
    __builtin_amdgcn_sched_barrier(0);
    auto round = [&](auto floor_tag, int b) {
        batch(floor_tag, std::integral_constant<int, 0>{}, b);
        batch(floor_tag, std::integral_constant<int, 1>{}, b + 1);
        if constexpr (kSets == 4) {
            batch(floor_tag, std::integral_constant<int, 2>{}, b + 2);
            batch(floor_tag, std::integral_constant<int, 3>{}, b + 3);
        }
    };
    int b = 0;
    for (; b + kSets <= nb && floor_on == 0; b += kSets) round(std::false_type{}, b);
    for (; b + kSets <= nb; b += kSets) round(std::true_type{}, b);
    double held[kSlots][R][NU][2];  // the exponentials of the last batches
    const auto hold = [&](auto rest_tag) {
#pragma unroll
        for (int k = 0; k < kSlots; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    constexpr int REST = decltype(rest_tag)::value;
                    held[k][r][u][0] = v[(REST + kSlots + k) % kSets][r][u][0];
                    held[k][r][u][1] = v[(REST + kSlots + k) % kSets][r][u][1];
                }
    };
    const int rest = nb - b;
    if (kSets == 4 && rest > 0) {
        batch(std::true_type{}, std::integral_constant<int, 0>{}, b);
        if (rest > 1) batch(std::true_type{}, std::integral_constant<int, 1>{}, b + 1);
        if (rest > 2) batch(std::true_type{}, std::integral_constant<int, 2>{}, b + 2);
        if (rest == 1) hold(std::integral_constant<int, 1>{});
        else if (rest == 2) hold(std::integral_constant<int, 2>{});
        else hold(std::integral_constant<int, 3>{});
    } else {
        hold(std::integral_constant<int, 0>{});
    }
    // the batches that are left: the older ones in LDS, the others in registers
#pragma unroll
    for (int k = 0; k <= LAG; ++k) {
        const int at = (nb + k) % kSets;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                // (the first row of the batch in turn is on its way already, the one that takes its place in LDS)
                if (k == 0 && r == 0) continue;
                if (k < kSlots) x[u] = L.prev[at % kSlots][r][u][threadIdx.x];
                else x[u] = dbl2{held[k - kSlots][r][u][0], held[k - kSlots][r][u][1]};
            }
            accumulate(x, L.fac[at][r]);
        }
        if (k < LAG) __syncthreads();
    }
    double *out = A.colpart + (int64_t)cluster * A.m + c0 + first;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        if (cv[u][0]) out[u * kStride] = csum[u][0];
        if (cv[u][1]) out[u * kStride + 1] = csum[u][1];
    }
}

// What a member publishes for a row, operation by operation, by one wave.  For a member that is not there in time.
template <int NU>
__device__ __forceinline__ double near_member_sum(const SweepArgs &A, int row, int member, int lane)
{
    const int c0 = member * A.width, ncol = min(A.width, A.m - c0);
    const double *src = A.M + (int64_t)row * A.ldM + c0, *beta = A.beta + c0;
    const double ref = near_minus_alpha(A, row);
    double mine = 0.0;
#pragma unroll 1
    for (int w = 0; w < kSweepWaves; ++w) {
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int c = 2 * kLanes * (u * kSweepWaves + w) + 2 * lane + e;
                if (c < ncol) acc += exp_eta_any((beta[c] - src[c]) - ref, A.ex);
            }
        const double sum = wave_reduce4<OpSum>(acc, acc, acc, acc);
        if ((lane & 15) == w) mine = sum;
    }
    return row16_reduce<OpSum>(mine);
}

// The factors, by one wave: lanes 16 r + j work on row r of a batch, j being a wave of the workgroup or a member of the cluster.
// In turn t a member publishes its sums of batch t and finds the factors of batch t - (LAG - 1), whose sums the other members have
// published in the meantime.
template <int NU, int R, int LAG>
__device__ __forceinline__ void near_factors(const SweepArgs &A, SweepNear<NU, R, LAG> &L, int member, const SweepRows &rows, int lane)
{
    constexpr int D = LAG - 1;
    static_assert(R == 4, "16 lanes a row");
    const int r16 = lane >> 4, j16 = lane & 15;
    const int nb = near_batches<R, LAG>(rows.count);
    unsigned long long *exch = reinterpret_cast<unsigned long long *>(A.exch);
    int patience = A.looks;
    const auto row_of = [&](int b) { return rows.at(max(b * R + r16, 0)); };
    const auto is_live = [&](int b) { return b >= 0 && b < nb && b * R + r16 < rows.count; };
    const auto word_of = [&](int b, int k) { return exch + (int64_t)row_of(b) * A.K * 2 + k; };
    double ai_before = 0.0, old_before = 0.0, sum_before = 0.0;
    // the new alpha of the rows of batch b, by one member
    const auto write_alpha = [&](int b) {
        if (b < 0 || b >= nb || b % A.K != member) return;
        const bool empty = ai_before == 0.0 && old_before == -INFINITY;
        const double value = empty ? -INFINITY : old_before + A.eta * (log(ai_before) - log(sum_before));
        if (j16 == 0 && is_live(b)) A.alpha_out[row_of(b)] = value;
    };
    __builtin_amdgcn_s_setprio(3);
    double own[D + 1] = {};          // the member's sums of batches t, t - 1, ..
    unsigned long long x = 0;        // of batch t - D, by member j16
    double ai = A.a[row_of(-D)], old = A.alpha[row_of(-D)], later = A.alpha[row_of(2)];
    for (int t = 0; t < nb + D; ++t) {
        const int k = t - D;
        __syncthreads();  // the workers' sums of batch t are there
#pragma unroll
        for (int d = D; d > 0; --d) own[d] = own[d - 1];
        if (t < nb) {
            own[0] = row16_reduce<OpSum>(j16 < kSweepWaves ? L.sums[t & 1][r16][j16] : 0.0);
            if (A.K > 1) {
                unsigned long long word = (unsigned long long)__double_as_longlong(own[0]);
                if (word == kUnpublished) word = 0x7ff8000000000000ull;
                if (j16 == 0 && is_live(t)) __hip_atomic_store(word_of(t, member), word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (D == 0) write_alpha(k - 1);
        double sum = own[D];
        if (k >= 0) {
            if (A.K > 1) {
                const bool wanted = is_live(k) && j16 < A.K;
                if (D == 0 && wanted) x = __hip_atomic_load(word_of(k, j16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                bool late = __ballot(wanted && x == kUnpublished) != 0;
                for (int left = patience; late && left > 0; --left) {  // (see sweep_factors)
                    if (wanted) x = __hip_atomic_load(word_of(k, j16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    late = __ballot(wanted && x == kUnpublished) != 0;
                }
                patience = late ? 0 : A.looks;
                if (late) {
                    unsigned long long open = __ballot(wanted && x == kUnpublished);
                    while (open != 0) {
                        const int at = __builtin_ctzll(open);
                        open &= open - 1;
                        const double part = near_member_sum<NU>(A, rows.at(k * R + (at >> 4)), at & 15, lane);
                        if (lane == at) x = (unsigned long long)__double_as_longlong(part);
                    }
                }
                sum = row16_reduce<OpSum>(wanted ? __longlong_as_double((long long)x) : 0.0);
            }
            const bool empty = ai == 0.0 && old == -INFINITY;
            if (j16 == 0) L.fac[k % (LAG + 1)][r16] = !is_live(k) || empty ? 0.0 : ai / sum;
        }
        if (j16 == 0) L.minus_alpha[t & 1][r16] = -fmax(later, A.floor);  // of batch t + 2
        if (D > 0) write_alpha(k - 1);
        ai_before = ai;
        old_before = old;
        sum_before = sum;
        // for the next turn
        if (D > 0 && A.K > 1 && is_live(k + 1) && j16 < A.K) x = __hip_atomic_load(word_of(k + 1, j16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ai = A.a[row_of(k + 1)];
        old = A.alpha[row_of(k + 1)];
        later = A.alpha[row_of(t + 3)];
    }
    write_alpha(nb - 1);
    __syncthreads();
}

}  // namespace regot
