"""The exact deterministic projection on both sides of the size of its terms from
which FP64 sums of two whole-number parts give way to limbs: |K_ij n_j| 2^20 times
the terms of a lane beyond 2^53."""
import itertools

import numpy as np
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu


def _rows_by_limbs(system, dkeys, keys, pops):
    """per row of K_DD: do its terms go beyond the FP64 sums"""
    cur = {tuple(int(x) for x in k): int(p) for k, p in zip(keys, pops)}
    dets = [np.array(k, np.uint64) for k in dkeys]
    c = np.array([cur.get(tuple(int(x) for x in k), 0) for k in dkeys], float)
    h00 = system.H00
    K = np.array([[system.diag(a) - h00 if i == j else system.hij(a, b) for j, b in enumerate(dets)]
                  for i, a in enumerate(dets)])
    return np.abs(K * c).max(axis=1) * 2.0 ** 20 * (len(dets) // 64 + 1) >= 2.0 ** 53


# deterministic space, hopping, largest population, share of the rows expected to go by
# limbs (a row that couples to nothing in the space never does)
@pytest.mark.parametrize("size,t,most,share", [(7, 1.0, 2 ** 28, (0, 0)), (7, 16.0, 2 ** 30, (0.1, 0.5)),
                                               (7, 64.0, 2 ** 30, (0.8, 1)), (130, 1.0, 2 ** 28, (0, 0)),
                                               (130, 4.0, 2 ** 30, (0.2, 0.8)), (130, 64.0, 2 ** 30, (0.9, 1))])
def test_projection_at_the_switch_to_limbs(size, t, most, share):
    sysd = dict(kind="hubbard", n_sites=6, periodic=1, t=t, U=0.25 * t, n_alpha=3, n_beta=3)
    q = dict(workloads.HUBBARD8["qmc"], tau=1e-6 / t, init_pop=1.0, target_population=1e12, fixed_point_bits=20,
             spawn_cutoff=0.01)
    ss = dict(size=size, start_iteration=1)
    rng = np.random.default_rng(size)
    system = oracle_system(sysd)
    bits = [sum(1 << 2 * int(b) for b in up) for up in itertools.combinations(range(6), 3)]
    dets = np.array(sorted(u | d << 1 for u in bits for d in bits), np.uint64)[:, None]
    size_of = np.exp(rng.uniform(np.log(most / 64), np.log(most), len(dets)))
    pops = (rng.choice([-1, 1], len(dets)) * size_of).astype(np.int32)
    ctx = gpu_context([sysd], [q], ss=ss, main_capacity=1 << 14, spawn_capacity=1 << 21)
    run = O.Run(system, oracle_qmc(sysd, q, ss=ss))
    ctx.import_walkers(dets, pops, iteration=1)
    run.import_walkers(dets, pops, iteration=1)
    for it in range(3):
        before = run.export()
        ctx.step(1)
        run.step(1)
        dkeys, y = ctx.detspace()
        assert np.array_equal(dkeys, run.detspace())
        limbs = _rows_by_limbs(system, dkeys, *before)
        say(f"[case] space of {size}, hopping {t:g}: {limbs.sum()} rows by limbs")
        assert share[0] <= limbs.mean() <= share[1]
        assert np.array_equal(y, run.last_projection())
        assert_same_lists(ctx, run, where=f"iteration {it}")
        assert_same_estimators(ctx.estimators(), run.estimators(), where=f"iteration {it}")
    ctx.close()
