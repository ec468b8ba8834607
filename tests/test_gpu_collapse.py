"""Segmented reduction of the spawned list at the sizes where it changes path.

The radix passes order the list by its top digits; the reduction orders each
group of equal digits: groups of one sort key, small mixed groups (counting),
large mixed groups (sorting network), groups larger than a tile's window of
1024 records (of one determinant, of several determinants on different sort
keys, and of several on one sort key). Truncated sort keys make such groups on
small systems. Every result must equal the oracle's bit for bit.
"""
import numpy as np
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu

RING = dict(kind="hubbard", periodic=1, t=1.0, U=4.0)
QMC = dict(workloads.HUBBARD8["qmc"], initial_shift=0.0)


def _same(ctx, runs, where):
    for r, run in enumerate(runs):
        kg, pg = ctx.export(r)
        ko, po = run.export()
        assert np.array_equal(kg, ko) and np.array_equal(pg, po), f"{where} instance {r}: lists differ"
        assert_same_estimators(ctx.estimators(r), run.estimators(), where=f"{where} instance {r}")


# sort-key bits, sites, walkers: groups of a few hundred mixed records (the
# network), of thousands on a few sort keys (ranges picked out of a group), and
# of thousands on one sort key with up to 64 determinants
@pytest.mark.parametrize("bits,sites,walkers,iters", [(7, 6, 2e3, 30), (7, 6, 2e4, 30), (5, 6, 6e4, 20), (3, 5, 8e4, 20),
                                                      (64, 4, 8e4, 20)])
def test_group_sizes_match_oracle(bits, sites, walkers, iters):
    sysd = dict(RING, n_sites=sites, n_alpha=sites // 2, n_beta=sites // 2)
    q = dict(QMC, init_pop=walkers, target_population=4 * walkers)
    say(f"[case] ring of {sites}, {walkers:g} walkers on D_0, {bits} hash bits in the sort key, two instances")
    ctx = gpu_context([sysd, sysd], [q, q], replicas=[0, 1], main_capacity=1 << 16, spawn_capacity=1 << 20)
    if bits < 64:
        ctx.set_sort_key_bits(bits)
    runs = [O.Run(oracle_system(sysd), oracle_qmc(sysd, q, replica=r)) for r in (0, 1)]
    for blk in range(iters // 10):
        ctx.step(10)
        for run in runs:
            run.step(10)
        _same(ctx, runs, f"{bits} bits, {sites} sites, block {blk}")
    most = max(e["n_spawned"] for e in ctx.history(0))
    say(f"[case] up to {most} spawned records an iteration")
    ctx.close()


@pytest.mark.parametrize("graph", [False, True])
def test_plan_follows_the_spawn_count(graph):
    """Spawn counts from a handful to tens of thousands and back: the number of
    radix passes changes between blocks (and the captured graphs with it)."""
    sysd, w = workloads.UEG14["system"], workloads.UEG14["qmc"]
    q = dict(w, init_pop=50.0, target_population=200.0, shift_damping=1.0)
    say(f"[case] electron gas, growing and shrinking list, graph={graph}")
    ctx = gpu_context([sysd], [q], main_capacity=1 << 19, spawn_capacity=1 << 19, graph=graph)
    run = O.Run(oracle_system(sysd), oracle_qmc(sysd, q))
    seen = []
    for pops in (None, 4e4, 30.0):
        if pops is not None:
            t = int(ctx.estimators()["iteration"])
            keys = np.array([run.export()[0][0]], np.uint64)
            units = np.array([int(pops * 256)], np.int32)
            ctx.import_walkers(keys, units, iteration=t)
            run.import_walkers(keys, units, iteration=t)
        for blk in range(3):
            ctx.step(10)
            run.step(10)
            assert_same_lists(ctx, run, where=f"population {pops} block {blk}")
            assert_same_estimators(ctx.estimators(), run.estimators(), where=f"population {pops} block {blk}")
            seen.append(ctx.estimators()["n_spawned"])
    say(f"[case] spawned records: {seen}")
    assert max(seen) > 12000 and min(seen) < 1000
    ctx.close()
