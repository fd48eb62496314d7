// The order in which a launch comes to the units of a plan, where a unit's cost depends on its action: dear ones first, so
// that what the last workgroups of the launch do is short.
#pragma once

#include "windq_common.hpp"

namespace windq {

constexpr int64_t ORDER_MAX_UNITS = 512;     // of a matrix; one with more keeps its own order (its units are small)

#ifdef __HIPCC__

// Work item `item` of a matrix's U (<= ORDER_MAX_UNITS) units of `per` items each, sorted by class; inside a class the items
// with the same number in their units come one after the other, so that neighbours in a launch read neighbouring columns.
// Returns the unit, its item and its class; of a unit of the last class only the first per_last items are work.  classes
// holds the class (0: dearest, to 3) of action a in bits 2a and 2a + 1, of an action outside the plan's in those of
// WINDQ_N_ACTIONS.  From the actions themselves, by every wavefront that calls it (all lanes): a byte load and four ballots per
// 64 units.  A workgroup waits for it before its first load, so it is kept short: with the rounds unrolled and every ballot
// held, a product at a plan of 2-bit units only took 27.4 us, 24.5 so.  (A unit's items one after the other: 8-bit units only
// 55 us, 47.5 so.)
struct OrderedItem {
    int32_t unit;           // -1: nothing to do
    int32_t item;
    int32_t cls;
};
// FEW_LAST: launches of many rounds' units with work to leave out (refinement).  Without it per_last is not looked at, and a round asks for
// its actions when it comes to them: asking ahead costs the product of a 7B-shaped block 0.1 us of 35.5.
template <bool FEW_LAST>
__device__ __forceinline__ OrderedItem item_by_cost(const uint8_t* __restrict__ action, int32_t U, int32_t per, int32_t per_last, int32_t item,
                                                    uint32_t classes) {
    const int lane = threadIdx.x & 63;
    int32_t n[4] = {0, 0, 0, 0};
    uint32_t mine = 0;                      // 4 bits a round: class of this lane's unit, 4: no unit
    uint32_t next = 0u;
    if (FEW_LAST) next = lane < U ? action[lane] : 0u;
    for (int32_t u0 = 0, k = 0; u0 < U; u0 += 64, ++k) {
        uint32_t c = 4u;
        if (FEW_LAST) {
            const uint32_t a = next;
            if (u0 + 64 < U) next = u0 + 64 + lane < U ? action[u0 + 64 + lane] : 0u;      // (rounds wait for memory once)
            c = (classes >> (2u * (a < WINDQ_N_ACTIONS ? a : WINDQ_N_ACTIONS))) & 3u;
            if (u0 + lane >= U) c = 4u;
        } else if (u0 + lane < U) {
            const uint32_t a = action[u0 + lane];
            c = (classes >> (2u * (a < WINDQ_N_ACTIONS ? a : WINDQ_N_ACTIONS))) & 3u;
        }
        mine |= c << (4 * k);
#pragma unroll
        for (int q = 0; q < 4; ++q) n[q] += __builtin_popcountll(__ballot(c == (uint32_t)q));
    }
    int32_t left = item;
    int want = 0;
    while (want < 3 && left >= n[want] * per) left -= n[want++] * per;
    const int32_t of = want == 0 ? n[0] : (want == 1 ? n[1] : (want == 2 ? n[2] : n[3]));
    OrderedItem r;
    r.cls = want;
    r.unit = -1;
    r.item = 0;
    if (FEW_LAST && want == 3 && left >= n[3] * per_last) return r;
    r.item = (int32_t)((uint32_t)left / (uint32_t)of);
    left -= r.item * of;
    if (of == U) {
        r.unit = left;
        return r;
    }
    int32_t u0 = 0;
    uint64_t m = __ballot((mine & 15u) == (uint32_t)want);
    while (left >= (int32_t)__builtin_popcountll(m)) {
        left -= (int32_t)__builtin_popcountll(m);
        u0 += 64;
        mine >>= 4;
        m = __ballot((mine & 15u) == (uint32_t)want);
    }
    const uint64_t at = __ballot((m >> lane & 1ull) != 0ull && (int32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull)) == left);
    r.unit = u0 + (int32_t)__builtin_ctzll(at);
    return r;
}

#endif  // __HIPCC__

}  // namespace windq
