// rpdla_plan.hpp -- which pushes are ordered, and how their groups are dealt to
// the waves: plain arithmetic, shared by the plan kernels, the push kernels and
// the host that sizes their scratch, and compiled for the host by its test.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "rpdla_fastmath.hpp"

namespace rpdla {

constexpr int kPlanLaunches = 32;         // slice launches

// Pushes of so few steps that putting the slots in order costs more than the
// order gains.  `steps` is the window's length in steps, the bound of every
// electron's.  The order costs two passes over the births, scattered loads and
// stores and, beyond one wave per SIMD (2^16 slots on 256 CUs), some 35 launches:
// 0.15 ms for 1.3e5 slots, 0.3 for 1e6, 0.8 for 4e6 and 3.4 for 1e7, where the
// queue takes 0.02, 0.07, 0.09 and 0.19 ms a step.  Queue / ordered, in
// microseconds, double precision (the other forms cross at the same steps): 1.3e5
// slots of 2 steps 69 / 154, of 4 123 / 154; 2.6e5 of 2 116 / 185, of 3 175 / 159;
// 1e6 of 2 158 / 286, of 4 292 / 272 (mixed 441 / 516); 4e6 of 4 535 / 813, of 8 950 / 850; 1e7 of 4
// 984 / 3476, of 16 3255 / 3491, of 24 4496 / 4013.
inline bool push_by_queue(int64_t n_slots, double steps)
{
    if (n_slots <= 1 << 16) return false;
    const double most = n_slots < 200000 ? 4.0 : 3.0 + 1.2 * (double)n_slots / (double)(1 << 20);
    return steps <= (most < 16.0 ? most : 16.0);
}

// The same for a chunk of a sweep, `slots` of all its configurations together:
// the plan of 64 configurations takes 0.14 ms, its launches 0.1 ms, and their
// queues waste less than the single one.  A chunk's time with the queue over that
// in order, double precision: 16 configurations of 20,480 slots 0.77 at 8 steps,
// 0.87 at 64, 1.03 at 192; 64 of 5,120 0.69, 0.80, 0.98; 64 of 10,240 0.85, 0.92,
// 1.05; 4 of 640 0.84 at 8, 1.09 at 64; with more slots in all (16 of 40,960, 64
// of 20,480) 1.0 and more from the start.  Mixed precision, whose steps are
// shorter, crosses at about twice the steps.
inline bool sweep_by_queue(int n_cfg, int64_t slots, double steps, bool mixed)
{
    const int64_t many = 10240ll * n_cfg > (1 << 19) ? 10240ll * n_cfg : 1 << 19;
    if (slots > many) return false;
    const double most = mixed ? 64.0 + (double)slots / 1536.0 : 32.0 + (double)slots / 2560.0;
    const double cap = mixed ? 256.0 : 128.0;
    return steps <= (most < cap ? most : cap);
}

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
