// rpdla_plan.hpp -- which pushes are ordered, and how their groups are dealt to
// the waves: plain arithmetic, shared by the plan kernels, the push kernels and
// the host that sizes their scratch, and compiled for the host by its test.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "rpdla_fastmath.hpp"

namespace rpdla {

constexpr int kPlanLaunches = 32;         // slice launches

// Form of an ionization of n atoms (of one launch) and K states over `panels`
// panels: a wave per atom, a wave per 64 (or fewer) atoms that asks the rate bound
// lane by lane and takes the few atoms left open one by one, or a lane per atom in
// the order of the work.  `reach` bounds the integral of the first state's rate for
// the atom in the strongest field, so an atom has that state open with at most the
// chance 1 - exp(-2 reach); infinite for a field constant in time (`uniform`).
//
// A wave per atom costs 2 to 4 us whatever the atom does, 12 us and more a birth;
// it balances atoms of unequal work and has the shortest chain.  Milliseconds, wave
// / few / lane (order 5, 30 fs and ten states unless said otherwise):
//   reach 1e-5 (7e14 W/cm^2)  16384 atoms 0.082 / 0.036 / 0.055, 1e6 4.2 / 0.09 / 0.32
//   reach 0.06 (2e15)         2e5 1.67 / 0.72 / 8.4,  1e6 7.6 / 1.5 / 8.6
//   reach 2.2 (4e15)          2e5 7.2 / 6.1 / 9.4,    1e6 34.7 / 21 / 21
//   reach 11 (6e15)           65536 3.8 / 4.2 / 10.3, 1e6 54 / 37 / 33
//   reach 54 (1e16)           2e5 12.4 / 12.7 / 15.8, 1e6 61 / 48 / 51
//   reach 137, one state      2e5 8.3 / 7.4 / 9.1,    1e6 40 / 27 / 28
//   reach 317, linear focus   2e5 9.8 / 9.4 / 15,     1e6 47 / 37 / 39
//   reach 1.2e4 (1e21)        2e5 24 / 31 / 31,       1e6 119 / 120 / 119, 3e6 358 / 337 / 340
//     in a target of 8 waists 2e5 7.1 / 7.4 / 19,     1e6 34 / 23 / 30 (the host sees no atoms)
//     linear focus            2e5 24 / 34 / 39,       1e6 117 / 133 / 125, 3e6 349 / 377 / 353
//   2 fs at 1e21, 2249 panels 2e5 6.4 / 8.5 / 5.5, one state 1.18 / 1.56 / 1.27;
//                             1e6 32 / 34 / 20,    one state 5.9 / 6.2 / 4.4
//   5 fs at 1e21, 5622 panels 1e6 42 / 43 / 36,    at 1e18 31 / 32 / 32,
//                             one state 8.0 / 8.4 / 6.7
//   10 steps a period, 1687   2e5 6.9 / 9.2 / 5.6,    1e6 34 / 37 / 19
//   uniform field, 1000       2e5 2.0 / 2.9 / 0.83,   1e6 10 / 11 / 2.5
enum IonizeForm { kIonizeWave, kIonizeFew, kIonizeLane };

inline IonizeForm ionize_form(int64_t n, int K, double panels, double reach, bool uniform)
{
    if (n < 16384) return kIonizeWave;
    if (uniform) return n >= 100000 ? kIonizeLane : kIonizeWave;
    if (reach <= (n < 65536 ? 0.01 : 0.5)) return kIonizeFew;
    if (panels <= (K <= 2 ? 12000.0 : 5000.0) && (double)n >= 3.0e4 + 1.0e4 * K + 75.0 * panels)
        return kIonizeLane;
    if (reach <= 60.0 && n >= (reach <= 30.0 ? 200000 : 500000)) return kIonizeFew;
    return reach <= (K <= 2 ? 2.0e4 : 1.0e3) && n >= 1000000 ? kIonizeFew : kIonizeWave;
}

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
