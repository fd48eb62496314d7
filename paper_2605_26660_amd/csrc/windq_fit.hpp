// The last step of fit+score for a unit, shared by the kernel that takes it alone (fit_score.hip) and the ones
// that take it beside the unit features' own last step (unit_features.hip).
#pragma once

#include "windq_common.hpp"
#include "windq_ws.hpp"

namespace windq {

struct FitFinalMat {
    double* partial;       // [n_tiles][5K+12]
    uint32_t* redo_count;  // number of units listed for the exact 8-bit pass
    uint32_t* redo_list;   // [U] their indices, in no particular order
    float* err;
    uint8_t* clip_idx;
    float* ref_energy;
    int64_t tiles_per_unit;
    const float* colsel;   // the chunks' records, or null: no unit is scored by a plan
    int32_t chunk_w;
    int32_t n_chunks;
};
struct FitFinalBatch {
    int32_t n;
    int32_t K;
    int32_t shares;        // sweeps the clip grid is dealt to: ratio k belongs to sweep (k - K) mod shares
    int32_t plans;         // nonzero: some matrix may have units that are scored by a plan
    int64_t unit_start[WINDQ_MAX_BATCH + 1];
    FitFinalMat m[WINDQ_MAX_BATCH];
};

// The 16 sums a unit's tiles are added in: sum p takes tiles p, p + 16, p + 32, ... in order; the sums are then added
// in order.  Fixed whatever the workgroup's size, so that every kernel that adds tiles up gives the same bits.
constexpr int FIN_PHASES = 16;

constexpr int FS_KB = 5;         // clip ratios of a sweep

#ifdef __HIPCC__

// The short 8-bit route's rounding noise that sends a unit to the exact pass, and the margin by which the bound of a
// left-out candidate has to exceed the chosen error (both derived in fit_score.hip).
constexpr double NOISE_MAX = 3e-6;
constexpr double NOISE_C1 = 4.0 * 3.552713678800501e-15 / (NOISE_MAX * NOISE_MAX);   // 4 * 2^-48 / NOISE_MAX^2
constexpr double BOUND_SLACK = 1e-4;


// NP phases (first, first + step, ...) of one candidate side by side: a unit is added up by one workgroup, a chain of loads that
// is as long as few of them are in flight.  (A sum that holds a lower bound, marked by its sign, is one itself and keeps the mark.)
// SHARED: the tiles' sums may have been stored by other workgroups of this launch (past the L2s).
template <int NP, bool SHARED>
__device__ __forceinline__ void fit_phase_sums(const double* __restrict__ base, int64_t tiles_per_unit, int32_t ncand, int32_t cand, int first, int step,
                                               double (&sum)[NP]) {
    bool bound[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        sum[p] = 0.0;
        bound[p] = false;
    }
    const auto add = [&](int64_t t, int p) {
        const double* at = base + (size_t)t * ncand + cand;
        const double v = SHARED ? __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *at;
        bound[p] |= v < 0.0;
        sum[p] += fabs(v);
    };
    int64_t t = 0;
#pragma unroll 4
    for (; t + FIN_PHASES <= tiles_per_unit; t += FIN_PHASES) {
#pragma unroll
        for (int p = 0; p < NP; ++p) add(t + first + p * step, p);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        if (t + first + p * step < tiles_per_unit) add(t + first + p * step, p);
        sum[p] = bound[p] ? -sum[p] : sum[p];
    }
}

// The phases of one candidate, in order, from [FIN_PHASES][stride].
__device__ __forceinline__ double fit_phases_total(const double* lds, int32_t stride, int32_t cand) {
    double acc = 0.0;
    bool bound = false;
#pragma unroll
    for (int p = 0; p < FIN_PHASES; ++p) {
        const double v = lds[p * stride + cand];
        bound |= v < 0.0;
        acc += fabs(v);
    }
    return bound ? -acc : acc;
}

// Index of the least of E[0..K-1], ties to the largest index; entries below zero are bounds: skipped, the least of
// their magnitudes to *bound_out.  (The last entry is never a bound.)
__device__ __forceinline__ int fit_least(const double* E, int32_t K, double* best_out, double* bound_out) {
    double best = 0.0, bound = INFINITY;
    int bk = -1;
    for (int k = 0; k < K; ++k) {
        const double e = E[k];
        if (e < 0.0) bound = fmin(bound, -e);
        else if (bk < 0 || e <= best) {
            best = e;
            bk = k;
        }
    }
    *best_out = best;
    *bound_out = bound;
    return bk;
}

// How many tiles of a listed unit have been scored again, and which sweeps they take (a bit each): two words in the unit's own
// partials (the first noise slot of its first tile, which nothing reads once the unit is listed).
__device__ __forceinline__ uint32_t* fit_redo_done(double* unit_partial, int32_t K) {
    return reinterpret_cast<uint32_t*>(unit_partial + fit_score_noise_slot(K));
}
__device__ __forceinline__ uint32_t* fit_redo_sweeps(double* unit_partial, int32_t K) { return fit_redo_done(unit_partial, K) + 1; }

// The sweep that ratio k belongs to.
__device__ __forceinline__ uint32_t fit_sweep_of(int32_t K, int32_t shares, int32_t k) { return (uint32_t)(k + FS_KB * shares - K) % (uint32_t)shares; }

// What is left to score of a unit whose heavy columns have been scored (windq_plan.hpp): a list of candidates, each with the number of
// columns it goes on to.  In the noise slots of the unit's first tile, behind the two words above (such units have no noise).
constexpr int PLAN_STEPS = 8;
struct FitPlan {
    uint32_t done, sweeps;                          // (sweeps: of the units that have no plan)
    uint8_t low[PLAN_STEPS], high[PLAN_STEPS];      // candidates that go on to plan_columns(chunk_w, step) columns: 4, 3 and 2 bits; 8 bits
    uint64_t scored[4];                             // those that take all (8, 4, 3, 2 bits): a bit per ratio
    uint8_t list[4 * WINDQ_MAX_CLIP];               // (bit-width << 6) | ratio: the low ones, most columns first, then the 8-bit ones (4 K at most)
};
static_assert(sizeof(FitPlan) - 4 * WINDQ_MAX_CLIP + 4 * FS_PLAN_MIN_K <= 8 * FS_PLAN_MIN_K, "fits the noise slots");
// In the noise slots of the unit's second tile: the shares of the chunk's columns (where the unit is the chunk's first, see windq_plan.hpp),
// then, once the unit is listed, the least error of each bit-width so far and its ratio.
struct FitListed {
    float shares[PLAN_STEPS + 2];
    double best[4];
    int32_t at[4];
};
static_assert(sizeof(FitListed) <= 8 * FS_PLAN_MIN_K, "fits the noise slots");
__device__ __forceinline__ FitListed* fit_listed(double* unit_partial, int32_t K) {
    return reinterpret_cast<FitListed*>(unit_partial + fit_score_ncand(K) + fit_score_noise_slot(K));
}
__device__ __forceinline__ FitPlan* fit_plan(double* unit_partial, int32_t K) {
    return reinterpret_cast<FitPlan*>(unit_partial + fit_score_noise_slot(K));
}
// A sum that is a bound: below zero, whatever it is.
__device__ __forceinline__ double plan_bound(double v) { return -fmax(fabs(v), 1e-300); }
// Columns (a multiple of 8) of a step: sixteenths of the chunk, the last one all of it.  (workload.py reads plans and records out of workspaces
// for the benchmark and the tests; tests/test_fit_workspace_layout.py holds it to these structures.)
__host__ __device__ __forceinline__ int32_t plan_columns(int32_t chunk_w, int step) {
    const int32_t n = (chunk_w * (int32_t)((0xFB754321u >> (4 * step)) & 15u) + (step == PLAN_STEPS - 1 ? chunk_w : 0)) >> 4;      // 1 2 3 4 5 7 11 16
    return n < 8 ? 8 : n & ~7;
}
// The list, by a workgroup of at least 4 K threads (called by all of them), thread i with the step of candidate i (b * K + k), or a number below zero.
// lds: PLAN_LIST_WORDS.
constexpr int PLAN_LIST_WORDS = 2 * PLAN_STEPS * 4 + 2 * PLAN_STEPS;
__device__ __forceinline__ void fit_plan_list(FitPlan* __restrict__ plan, uint64_t* __restrict__ lds, int step, int32_t K, int tid) {
    const int wave = tid >> 6, lane = tid & 63;
    const bool on = tid < 4 * K && step >= 0, high = tid < K;
    uint64_t* __restrict__ total = lds + 2 * PLAN_STEPS * 4;
    if (wave < 4) {
#pragma unroll
        for (int s = 0; s < PLAN_STEPS; ++s) {
            const uint64_t lo = __builtin_amdgcn_ballot_w64(on && !high && step == s), hi = __builtin_amdgcn_ballot_w64(on && high && step == s);
            if (lane == 0) {
                lds[s * 4 + wave] = lo;
                lds[(PLAN_STEPS + s) * 4 + wave] = hi;
            }
        }
    }
    __syncthreads();
    if (tid < 2 * PLAN_STEPS) {
        int n = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) n += __builtin_popcountll(lds[tid * 4 + w]);
        total[tid] = (uint64_t)n;
        (tid < PLAN_STEPS ? plan->low : plan->high)[tid & (PLAN_STEPS - 1)] = (uint8_t)n;
    }
    __syncthreads();
    if (on) {
        int at = __builtin_popcountll(lds[((high ? PLAN_STEPS : 0) + step) * 4 + wave] & ((1ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) at += __builtin_popcountll(lds[((high ? PLAN_STEPS : 0) + step) * 4 + w]);
#pragma unroll
        for (int s = 0; s < PLAN_STEPS; ++s) {
            if (high) at += (int)total[s];
            if (s > step) at += (int)total[(high ? PLAN_STEPS : 0) + s];
        }
        const int b = tid / K;
        plan->list[at] = (uint8_t)((b << 6) | (tid - b * K));
    }
    if (tid < 4) {          // bit-width tid: candidates tid K .. tid K + K - 1, out of the wavefronts' sets
        uint64_t all = 0u;
        const int s = PLAN_STEPS - 1, first = tid * K;
        for (int w = 0; w < 4; ++w) {
            const uint64_t set = lds[s * 4 + w] | lds[(PLAN_STEPS + s) * 4 + w];
            const int shift = first - 64 * w;
            all |= shift >= 64 || shift <= -64 ? 0ull : (shift >= 0 ? set >> shift : set << -shift);
        }
        all &= K < 64 ? (1ull << K) - 1ull : ~0ull;
        plan->scored[tid] = all;
    }
}

// Dynamic LDS of a workgroup that finalizes: [FIN_PHASES][ncand] phase sums, [ncand] totals.
constexpr size_t fit_finalize_lds_bytes(int32_t K) { return (size_t)(FIN_PHASES + 1) * (size_t)fit_score_ncand(K) * sizeof(double); }

// Per unit: add the tiles' partial errors in a fixed order, pick the clip index with the
// least error for each uniform bit-width (ties to the largest index), emit fp32.  A unit whose 8-bit
// error may hold too much of the short route's rounding noise, or one of whose left-out candidates is not
// proved to be worse, is put on the list.  Called by all NT threads of a workgroup.  PLANS: a launch that may have units scored by a plan.
template <int NT, bool PLANS>
__device__ __forceinline__ void fit_finalize_unit(const FitFinalBatch& B, int64_t block, double* __restrict__ lds) {
    const int mi = batch_index(B.unit_start, B.n, block);
    const FitFinalMat& A = B.m[mi];
    const int64_t u = block - B.unit_start[mi];
    const int32_t K = B.K;
    const int64_t tiles_per_unit = A.tiles_per_unit;
    const int32_t ncand = fit_score_ncand(K);
    double* __restrict__ E = lds + FIN_PHASES * ncand;
    double* base = A.partial + (size_t)u * (size_t)tiles_per_unit * (size_t)ncand;
    // (read ahead of the sums, which they wait for together; words of any kind where the unit is not planned)
    const int tid = threadIdx.x;
    static_assert(NT >= 4 * WINDQ_MAX_CLIP, "a candidate a thread");
    const bool planned = PLANS && A.colsel != nullptr &&
                         heavy_columns(__float_as_int(A.colsel[(size_t)((uint32_t)u % (uint32_t)A.n_chunks) * (size_t)colsel_words(A.chunk_w) + A.chunk_w + FS_HMAX])) != 0;
    const uint64_t scored = PLANS && A.colsel != nullptr ? fit_plan(base, K)->scored[tid < 4 * K ? tid / K : 0] : 0u;
    constexpr int WAVES = NT / 64, NP = FIN_PHASES / WAVES;
    static_assert(NP * WAVES == FIN_PHASES, "a wavefront's phases");
    for (int32_t cand = threadIdx.x & 63; cand < ncand; cand += 64) {
        const int first = threadIdx.x >> 6;
        double sum[NP];
        fit_phase_sums<NP, false>(base, tiles_per_unit, ncand, cand, first, WAVES, sum);
#pragma unroll
        for (int p = 0; p < NP; ++p) lds[(first + p * WAVES) * ncand + cand] = sum[p];
    }
    __syncthreads();
    for (int32_t cand = threadIdx.x; cand < ncand; cand += NT) E[cand] = fit_phases_total(lds, ncand, cand);
    __syncthreads();
    if (planned) {           // what has not taken every column is a bound
        if (tid < 4 * K && ((scored >> (tid % K)) & 1u) == 0u) E[tid] = plan_bound(E[tid]);
        __syncthreads();
    }
    bool open = false;           // (a planned unit) a candidate is not proved to be worse
    if (tid < 4) {
        double best, bound;
        const int bk = fit_least(E + tid * K, K, &best, &bound);
        A.err[u * WINDQ_N_ERR + tid] = (float)best;
        A.clip_idx[u * 4 + tid] = (uint8_t)bk;
        // (tid 0: 8 bits) listed: too much noise, then every sweep is taken again; or a candidate that was left out is not
        // proved to be worse, then the sweeps of such candidates
        open = planned && !(bound * (1.0 - BOUND_SLACK) > best) && bound < INFINITY;
        const bool noisy = tid == 0 && !planned && E[fit_score_noise_slot(K) + bk] * NOISE_C1 > best * best;
        if (tid == 0 && !planned && (noisy || bound * (1.0 - BOUND_SLACK) <= best)) {
            uint32_t sweeps = 0u;
            for (int k = 0; k < K; ++k) {
                const uint32_t v = fit_sweep_of(K, B.shares, k);
                if (noisy || (E[k] < 0.0 && -E[k] * (1.0 - BOUND_SLACK) <= best)) sweeps |= 1u << v;
            }
            *fit_redo_done(base, K) = 0u;
            *fit_redo_sweeps(base, K) = sweeps;
            const uint32_t pos = atomicAdd(A.redo_count, 1u);
            A.redo_list[pos] = (uint32_t)u;
        }
    } else if (tid < 7) {
        // ternary, binary, reference energy: the four column quarters, in order
        const int j = tid - 4;
        const double e = ((E[4 * K + j] + E[4 * K + 3 + j]) + E[4 * K + 6 + j]) + E[4 * K + 9 + j];
        if (j < 2) A.err[u * WINDQ_N_ERR + 4 + j] = (float)e;
        else if (A.ref_energy != nullptr) A.ref_energy[u] = (float)e;
    }
    if (!planned || __syncthreads_or(open ? 1 : 0) == 0) return;           // (the same for the whole workgroup)
    // listed: the open candidates are scored on all columns
    int step = -1;
    if (tid < 4 * K) {
        double best, bound;
        fit_least(E + (tid / K) * K, K, &best, &bound);
        if (E[tid] < 0.0 && !(-E[tid] * (1.0 - BOUND_SLACK) > best)) step = PLAN_STEPS - 1;
    }
    FitPlan* __restrict__ plan = fit_plan(base, K);
    uint64_t* __restrict__ lists = reinterpret_cast<uint64_t*>(lds);         // (the phases' sums are done with)
    fit_plan_list(plan, lists, step, K, tid);
    if (tid < 4) {
        double best, bound;
        fit_listed(base, K)->at[tid] = fit_least(E + tid * K, K, &best, &bound);
        fit_listed(base, K)->best[tid] = best;
    }
    if (tid == 0) {
        plan->done = 0u;
        const uint32_t pos = atomicAdd(A.redo_count, 1u);
        A.redo_list[pos] = (uint32_t)u;
    }
}

#endif  // __HIPCC__

}  // namespace windq
