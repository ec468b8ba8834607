"""The segmented reduction where its groups are larger than the plan expects, by
key width: the sorting network, ranges picked out of a group, several
determinants on one sort key inside a window and beyond one. (Keys of four and
eight words are read again where shorter ones are held.) Truncated sort keys and
lists that grow within one block of iterations make such groups; every result
must equal the oracle's."""
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu


# cutoff (9: four words, 14: eight), electrons, hash bits in the sort key, walkers on D_0, time step
@pytest.mark.parametrize("ecut,electrons,bits,walkers,tau", [
    (9, 14, 14, 2e3, 0.002),    # groups of some 2 to 4 records on one sort key
    (9, 14, 8, 2e3, 0.002),     # up to 18 determinants on one sort key
    (9, 4, 7, 3e4, 0.002),      # hundreds of records on one sort key
    (9, 2, 5, 2e5, 0.002),      # more than a window on one sort key
    (14, 14, 14, 2e3, 0.002),
    (14, 14, 8, 2e3, 0.002),
    (14, 4, 7, 3e4, 0.002),
    (14, 2, 5, 2e5, 0.002),
])
def test_long_keys_on_truncated_sort_keys(ecut, electrons, bits, walkers, tau):
    sysd = dict(kind="ueg", rs=1.0, ecut_n2=ecut, n_alpha=electrons // 2, n_beta=electrons // 2)
    q = dict(workloads.UEG14["qmc"], tau=tau, init_pop=walkers, target_population=2 * walkers, initiator=0)
    ctx = gpu_context([sysd, sysd], [q, q], replicas=[0, 1], main_capacity=1 << 18, spawn_capacity=1 << 21)
    ctx.set_sort_key_bits(bits)
    runs = [O.Run(oracle_system(sysd), oracle_qmc(sysd, q, replica=r)) for r in (0, 1)]
    for it in range(4):
        ctx.step(1)
        for r, run in enumerate(runs):
            run.step(1)
            where = f"cutoff {ecut}, {electrons} electrons, {bits} bits, instance {r}, iteration {it}"
            assert_same_lists(ctx, run, instance=r, where=where)
            assert_same_estimators(ctx.estimators(r), run.estimators(), where=where)
    e = ctx.estimators(0)
    say(f"[case] {ctx.W} words, {bits} bits: {e['n_spawned']} records on {e['n_spawn_events']} determinants")
    ctx.close()


# One pass orders 256 groups; the list grows from a handful of records within the
# block that was planned for it: groups of 128 to 1024 mixed records go through the
# network, larger ones are picked apart. With 20 hash bits, in two instances,
# determinants share sort keys in both.
@pytest.mark.parametrize("ecut,tau,walkers", [(5, 0.02, 2e3), (5, 0.02, 2e4), (9, 0.02, 2e2), (9, 0.02, 2e3),
                                              (14, 0.01, 3e2), (14, 0.01, 2e3)])
@pytest.mark.parametrize("bits", [64, 20])
def test_growth_beyond_the_plan(ecut, tau, walkers, bits):
    n = 1 if bits == 64 else 2
    if n > 1:
        walkers = min(walkers, 4e3)
    sysd = dict(kind="ueg", rs=1.0, ecut_n2=ecut, n_alpha=7, n_beta=7)
    q = dict(workloads.UEG14["qmc"], tau=tau, init_pop=walkers, target_population=1e12, initiator=0)
    ctx = gpu_context([sysd] * n, [q] * n, replicas=list(range(n)), main_capacity=1 << 23, spawn_capacity=1 << 22)
    if bits < 64:
        ctx.set_sort_key_bits(bits)
    ctx.step(9)
    for r in range(n):
        run = O.Run(oracle_system(sysd), oracle_qmc(sysd, q, replica=r))
        run.step(9)
        where = f"cutoff {ecut}, {walkers:g} walkers, {bits} bits, instance {r}"
        assert_same_lists(ctx, run, instance=r, where=where)
        for got in ctx.history(r)[-1:]:
            assert_same_estimators(got, run.estimators(), where=where)
    records = ctx.estimators(0)["n_spawned"]
    say(f"[case] {ctx.W} words, {bits} bits: {records * n} records in 256 groups")
    assert records * n / 256 > 128
    ctx.close()
