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
};
struct FitFinalBatch {
    int32_t n;
    int32_t K;
    int32_t shares;        // sweeps the clip grid is dealt to: ratio k belongs to sweep (k - K) mod shares
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

// Dynamic LDS of a workgroup that finalizes: [FIN_PHASES][ncand] phase sums, [ncand] totals.
constexpr size_t fit_finalize_lds_bytes(int32_t K) { return (size_t)(FIN_PHASES + 1) * (size_t)fit_score_ncand(K) * sizeof(double); }

// Per unit: add the tiles' partial errors in a fixed order, pick the clip index with the
// least error for each uniform bit-width (ties to the largest index), emit fp32.  A unit whose 8-bit
// error may hold too much of the short route's rounding noise, or one of whose left-out candidates is not
// proved to be worse, is put on the list.  Called by all NT threads of a workgroup.
template <int NT>
__device__ __forceinline__ void fit_finalize_unit(const FitFinalBatch& B, int64_t block, double* __restrict__ lds) {
    const int mi = batch_index(B.unit_start, B.n, block);
    const FitFinalMat& A = B.m[mi];
    const int64_t u = block - B.unit_start[mi];
    const int32_t K = B.K;
    const int64_t tiles_per_unit = A.tiles_per_unit;
    const int32_t ncand = fit_score_ncand(K);
    double* __restrict__ E = lds + FIN_PHASES * ncand;
    double* base = A.partial + (size_t)u * (size_t)tiles_per_unit * (size_t)ncand;
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
    const int tid = threadIdx.x;
    if (tid < 4) {
        double best, bound;
        const int bk = fit_least(E + tid * K, K, &best, &bound);
        A.err[u * WINDQ_N_ERR + tid] = (float)best;
        A.clip_idx[u * 4 + tid] = (uint8_t)bk;
        // (tid 0: 8 bits) listed: too much noise, then every sweep is taken again; or a candidate that was left out is not
        // proved to be worse, then the sweeps of such candidates
        const bool noisy = tid == 0 && E[fit_score_noise_slot(K) + bk] * NOISE_C1 > best * best;
        if (tid == 0 && (noisy || bound * (1.0 - BOUND_SLACK) <= best)) {
            uint32_t sweeps = 0u;
            for (int k = 0; k < K; ++k) {
                const uint32_t v = (uint32_t)(k + FS_KB * B.shares - K) % (uint32_t)B.shares;
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
}

#endif  // __HIPCC__

}  // namespace windq
