"""How an ordered push deals its groups to the waves (csrc/rpdla_plan.hpp),
compiled for the host: the group count up to the largest slot count the ordered
push takes, and, for group counts around whole rounds of waves, that the rounds
and slice launches together give every group each of its turns once, a later
turn always in a later launch, within the scratch the host allots."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_01741_amd", "csrc")

HARNESS = r'''
#include "rpdla_plan.hpp"
using namespace rpdla;
extern "C" {
unsigned t_groups(unsigned n) { return groups_of(n); }
void t_split(unsigned g, unsigned simds, unsigned waves, unsigned* o)
{
    const PlanSplit s = plan_split(g, simds, waves);
    o[0] = s.waves; o[1] = s.whole; o[2] = s.rest; o[3] = s.slices;
}
long long t_bound(long long g, long long simds, long long waves) { return plan_rest_bound(g, simds, waves); }
int t_turn(unsigned l, unsigned w, unsigned W, unsigned rest, unsigned slices, unsigned* o)
{
    const PlanTurn t = plan_turn(l, w, W, rest, slices);
    o[0] = t.index; o[1] = t.turn;
    return t.any;
}
unsigned t_steps(double most, unsigned slices) { return plan_slice_steps(most, slices); }
int t_queue(long long n, double steps) { return push_by_queue(n, steps); }
int t_sweep(int c, long long n, double steps, int mixed) { return sweep_by_queue(c, n, steps, mixed); }
int t_form(long long n, int K, double panels, double reach, int uniform)
{ return ionize_form(n, K, panels, reach, uniform); }
int t_launches() { return kPlanLaunches; }
}
'''


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "h.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + CSRC, "-o",
                    str(d / "libplan.so"), str(d / "h.cpp")], check=True)
    lib = C.CDLL(str(d / "libplan.so"))
    lib.t_groups.restype = C.c_uint
    lib.t_bound.restype = C.c_longlong
    lib.t_bound.argtypes = [C.c_longlong] * 3
    lib.t_form.argtypes = [C.c_longlong, C.c_int, C.c_double, C.c_double, C.c_int]
    lib.t_queue.argtypes = [C.c_longlong, C.c_double]
    lib.t_sweep.argtypes = [C.c_int, C.c_longlong, C.c_double, C.c_int]
    lib.t_steps.restype = C.c_uint
    lib.t_steps.argtypes = [C.c_double, C.c_uint]
    return lib


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 128, 2**31, 2**32 - 129, 2**32 - 65, 2**32 - 64,
                               2**32 - 63, 2**32 - 2])
def test_group_count(plan, n):
    assert plan.t_groups(C.c_uint(n)) == (n + 63) // 64


@pytest.mark.parametrize("simds,waves", [(1, 1), (4, 4), (12, 7)])
def test_every_group_gets_its_turns(plan, simds, waves):
    u = C.c_uint
    most = simds * waves
    counts = {0, 1, simds - 1, simds, simds + 1, 2 * simds - 1, 2 * simds, 2 * simds + 1, 3 * most}
    counts |= {k * most + d for k in (1, 2, 3) for d in (-1, 0, 1)} | set(range(0, 2 * most, 3))
    launches = plan.t_launches()
    for g in sorted(c for c in counts if c >= 0):
        o = (u * 4)()
        plan.t_split(u(g), u(simds), u(waves), o)
        W, whole, rest, slices = o
        assert W % simds == 0 and simds <= W <= most and whole % W == 0 and whole + rest == g
        assert slices >= 1 and rest * slices <= launches * W
        # room for the electrons that rest between slices
        if slices > 1:
            assert rest <= plan.t_bound(g, simds, waves)
        turns = [[] for _ in range(rest)]
        for launch in range(launches):
            for w in range(W):
                t = (u * 2)()
                if plan.t_turn(u(launch), u(w), u(W), u(rest), u(slices), t):
                    turns[t[0]].append((launch, t[1]))
        for seen in turns:
            assert [t for _, t in seen] == list(range(slices))
            assert all(a < b for (a, _), (b, _) in zip(seen, seen[1:]))
        # up to a group per SIMD the host makes one slice launch
        if g <= simds:
            assert all(seen == [(0, 0)] for seen in turns)
        for steps in (0.0, 1.0, 31.0, 22500.0, 2.0e9):
            assert plan.t_steps(steps, slices) * slices >= steps


def test_which_pushes_are_ordered(plan):
    """Few steps go to the queue, more of them with more slots; all others, the
    default window at any size among them, are ordered."""
    for n in (1, 64, 2**16):
        assert not any(plan.t_queue(n, float(s)) for s in (1, 2, 4, 22500))
    for n, steps in ((2**16 + 1, 4), (199999, 4), (200000, 3), (2**18, 3), (2**20, 4), (2**22, 7),
                     (10**7, 14), (2**32, 16), (2**40, 16)):
        assert plan.t_queue(n, float(steps)) and not plan.t_queue(n, steps + 1.0)
    assert not any(plan.t_queue(n, 22500.0) for n in (1, 2**20, 2**32, 2**40))
    for c, n, fp64, mixed in ((1, 10, 32, 64), (4, 40960, 48, 90), (64, 655360, 128, 256),
                              (16, 2**19, 128, 256)):
        assert plan.t_sweep(c, n, float(fp64), 0) and not plan.t_sweep(c, n, fp64 + 1.0, 0)
        assert plan.t_sweep(c, n, float(mixed), 1) and not plan.t_sweep(c, n, mixed + 1.0, 1)
    for c, n in ((1, 2**19 + 1), (51, 2**19 + 1), (64, 655361), (64, 2**33)):
        assert not plan.t_sweep(c, n, 1.0, 0) and not plan.t_sweep(c, n, 1.0, 1)
    assert not any(plan.t_sweep(c, 640 * c, 30000.0, m) for c in (1, 64) for m in (0, 1))


def test_ionization_forms(plan):
    """Few atoms always take a wave each, so do many on the default window at the
    intensities of the ensembles; the other forms begin where the rule says."""
    wave, few, lane = 0, 1, 2
    for n in (1, 1024, 16383):
        for reach in (0.0, 0.1, 1e9, float("inf")):
            assert plan.t_form(n, 10, 22500.0, reach, 0) == wave
    for n in (16384, 200_000, 1_000_000, 2**25):
        assert plan.t_form(n, 10, 33727.0, 1.2e4, 0) == wave
        assert plan.t_form(n, 1, 59584.0, float("inf"), 0) == wave
        assert plan.t_form(n, 10, 33727.0, 1e-3, 0) == few
    assert plan.t_form(65535, 10, 33727.0, 0.1, 0) == wave
    assert plan.t_form(65536, 10, 33727.0, 0.5, 0) == few
    for K, panels, n in ((10, 256.0, 149200), (1, 256.0, 59200), (10, 5000.0, 505000), (2, 12000.0, 950000)):
        assert plan.t_form(n, K, panels, 1e3, 0) == lane
        assert plan.t_form(n - 1, K, panels, 1e9, 0) == wave
    assert plan.t_form(2**25, 10, 5001.0, float("inf"), 0) == wave
    assert plan.t_form(200_000, 10, 33727.0, 30.0, 0) == few
    assert plan.t_form(500_000, 10, 33727.0, 60.0, 0) == few
    assert plan.t_form(1_000_000, 2, 33727.0, 2e4, 0) == few
    assert plan.t_form(1_000_000, 10, 33727.0, 1e3, 0) == few
    assert plan.t_form(999_999, 10, 33727.0, 61.0, 0) == wave
    assert plan.t_form(99_999, 10, 1000.0, float("inf"), 1) == wave
    assert plan.t_form(100_000, 10, 1000.0, float("inf"), 1) == lane
