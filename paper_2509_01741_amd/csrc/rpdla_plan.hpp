// rpdla_plan.hpp -- how the groups of an ordered push are dealt to the waves:
// plain integer arithmetic, shared by the plan kernels, the push kernels and the
// host that sizes their scratch, and compiled for the host by its test.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "rpdla_fastmath.hpp"

namespace rpdla {

constexpr int kPlanLaunches = 32;         // slice launches

// Groups of 64 slots; no sum that could pass 2^32 on the way.
RPDLA_HD inline uint32_t groups_of(uint32_t slots)
{
    return slots / 64u + (slots % 64u != 0u ? 1u : 0u);
}

// `waves` waves, a whole number per SIMD, take `whole` groups in rounds (a
// multiple of waves) and the `rest` in `slices` time slices each, which fit
// kPlanLaunches launches of `waves` turns.
struct PlanSplit {
    uint32_t waves, whole, rest, slices;
};

RPDLA_HD inline PlanSplit plan_split(uint32_t groups, uint32_t simds, uint32_t max_waves)
{
    PlanSplit s;
    const uint32_t per_simd = groups / simds < max_waves ? groups / simds : max_waves;
    s.waves = simds * (per_simd > 0 ? per_simd : 1);
    s.whole = groups / s.waves >= 2 ? (groups / s.waves - 1) * s.waves : 0;
    s.rest = groups - s.whole;
    s.slices = s.rest <= s.waves ? 1u : (uint32_t)((uint64_t)kPlanLaunches * s.waves / s.rest);
    return s;
}

// Most groups that can be left for slices, and so need room in memory between
// them, of at most `groups`: none up to a group per SIMD (one slice), else
// fewer than two rounds of waves.
RPDLA_HD inline int64_t plan_rest_bound(int64_t groups, int64_t simds, int64_t max_waves)
{
    const int64_t two = 2 * simds * max_waves;
    return groups <= simds ? 0 : (groups < two ? groups : two);
}

// What wave `wave` does in slice launch `launch`: turn `turn` of group
// whole + `index`, or nothing.  Turns of a group are `rest` places apart in the
// sequence, and a launch has `waves` places: with more than one slice rest is
// larger, so that two turns of a group are never in one launch.
struct PlanTurn {
    bool any;
    uint32_t index, turn;
};

RPDLA_HD inline PlanTurn plan_turn(uint32_t launch, uint32_t wave, uint32_t waves, uint32_t rest,
                                   uint32_t slices)
{
    const uint64_t p = (uint64_t)launch * waves + wave;
    if (rest == 0 || p >= (uint64_t)rest * slices) return PlanTurn{false, 0, 0};
    const uint32_t turn = (uint32_t)(p / rest);
    return PlanTurn{true, (uint32_t)(p - (uint64_t)turn * rest), turn};
}

// Steps of one slice, where the longest electron of the rest has `most`.
RPDLA_HD inline uint32_t plan_slice_steps(double most, uint32_t slices)
{
    return (uint32_t)(most / (double)slices) + 1u;
}

}  // namespace rpdla
