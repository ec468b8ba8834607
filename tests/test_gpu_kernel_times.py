"""Per-kernel times of a timed step: the radix passes an iteration makes, and no others;
passes that keep up with a list that grows within a call."""
import pytest

from gpu_helpers import gpu_context, say
from paper_1811_11679_amd import fciqmc as F
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu


# one pass for a hundred records, two for 6e5
@pytest.mark.parametrize("walkers,passes", [(2e2, 1), (1e6, 2)])
def test_passes_that_are_not_made_take_no_time(walkers, passes):
    w = workloads.HUBBARD8
    say(f"[case] ring of eight, {walkers:g} walkers")
    ctx = gpu_context([w["system"]], [dict(w["qmc"], init_pop=walkers, target_population=walkers)],
                      main_capacity=1 << 14, spawn_capacity=1 << 20)
    ctx.step(20)
    ctx.set_timing(True)
    ctx.step(10)
    times, n = ctx.kernel_times()
    assert n == 10
    made = [p for p in range(8) if times[f"sort_pass{p}"] > 0.0]
    assert made == list(range(passes)), (times, ctx.estimators()["n_spawned"])
    assert len(times) == len(F.KERNEL_SLOTS) and times["spawn"] > 0.0
    ctx.close()


def test_passes_follow_growth_within_a_call():
    """Few records at first and more than a million nine iterations later, between two
    shift updates: the last ones need more passes than the first."""
    w = workloads.UEG14
    say("[case] electron gas of 123 plane waves from 2000 walkers with a large time step")
    ctx = gpu_context([dict(w["system"], ecut_n2=9)], [dict(w["qmc"], tau=0.02, init_pop=2e3, target_population=1e12,
                                                            initiator=0)], main_capacity=1 << 22, spawn_capacity=1 << 22)
    ctx.set_timing(True)
    ctx.step(9)
    spawned = [e["n_spawned"] for e in ctx.history()]
    assert len(spawned) == 9 and spawned[0] < 8192 / 1.5 and spawned[-1] > 64 * 8192, spawned
    assert ctx.kernel_times()[0]["sort_pass1"] > 0.0
    ctx.close()
