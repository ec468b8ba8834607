"""Per-kernel times of a timed step: the radix passes an iteration makes, and no others."""
import pytest

from gpu_helpers import gpu_context, say
from paper_1811_11679_amd import fciqmc as F
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu


# one pass up to 32 records a digit (8192 with half as many again to spare), two up to 2^21
@pytest.mark.parametrize("walkers,passes", [(5e3, 1), (1e6, 2)])
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
