// The order in which a launch comes to the units of a plan, where a unit's cost depends on its action: dear ones first, so
// that what the last workgroups of the launch do is short.
#pragma once

#include "windq_common.hpp"

namespace windq {

constexpr int64_t ORDER_MAX_UNITS = 512;     // of a matrix; one with more keeps its own order (its units are small)

#ifdef __HIPCC__

// The unit that comes at place `place` when a matrix's U (<= ORDER_MAX_UNITS) units are sorted by class, each class in its own
// order; classes holds the class (0: dearest, to 3) of action a in bits 2a and 2a + 1, of an action outside the plan's in those
// of WINDQ_N_ACTIONS.  From the actions themselves, by every wavefront that calls it (all lanes): a byte load and three
// ballots per 64 units.
__device__ __forceinline__ int64_t unit_by_cost(const uint8_t* __restrict__ action, int32_t U, int32_t place, uint32_t classes) {
    const int lane = threadIdx.x & 63;
    constexpr int ROUNDS = (int)(ORDER_MAX_UNITS / 64);
    uint32_t cls[ROUNDS];                   // 4: no unit
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        cls[k] = WINDQ_N_ACTIONS;
        if (64 * k + lane < U) cls[k] = action[64 * k + lane];
    }
    uint64_t is[ROUNDS][4];
    int32_t n[4] = {0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        const uint32_t a = cls[k] < WINDQ_N_ACTIONS ? cls[k] : WINDQ_N_ACTIONS;
        const uint32_t c = 64 * k + lane < U ? (classes >> (2u * a)) & 3u : 4u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            is[k][q] = __ballot(c == (uint32_t)q);
            n[q] += __builtin_popcountll(is[k][q]);
        }
    }
    int32_t left = place;
    int want = 0;
    while (want < 3 && left >= n[want]) left -= n[want++];
    int32_t u = 0;
    bool found = false;
#pragma unroll
    for (int k = 0; k < ROUNDS; ++k) {
        const uint64_t m = want == 0 ? is[k][0] : (want == 1 ? is[k][1] : (want == 2 ? is[k][2] : is[k][3]));
        const int32_t here = __builtin_popcountll(m);
        if (!found && left < here) {
            const uint64_t at = __ballot((m >> lane & 1ull) != 0ull && (int32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull)) == left);
            u = 64 * k + __builtin_ctzll(at);
            found = true;
        }
        if (!found) left -= here;
    }
    return u;
}

#endif  // __HIPCC__

}  // namespace windq
