"""Coupled cluster lists a program imports, where the sampler of the composite
clusters takes its general paths."""
import numpy as np
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import fciqmc as F

pytestmark = pytest.mark.gpu

FIELDS = ("n_walkers_units", "n_occupied", "ref_pop_units", "n_spawned", "n_cluster_spawns", "spawn_sum")


def _bits(det):
    return [b for b in range(64) if det >> b & 1]


def test_excitors_that_add_electrons():
    """An imported excitor may hold another number of electrons than D_0. It then
    adds no level to a cluster, so bounds on the level of what is still to be
    drawn do not hold. The expected numbers are those of evaluating every
    selection in full."""
    sysd = dict(kind="ueg", rs=1.0, ecut_n2=2, n_alpha=3, n_beta=3)
    q = dict(tau=0.01, rng_seed=5, init_pop=1.0, target_population=1e9, fixed_point_bits=8, spawn_cutoff=0.01)
    say("[case] CCSD on 6 electrons in 19 plane waves, excitors with one electron more")
    ctx = gpu_context([sysd], [dict(q, method=F.CCMC, ccmc_truncation=2)], main_capacity=1 << 14,
                      spawn_capacity=1 << 18)
    ref = int(ctx.export()[0][0, 0])
    empty = [b for b in range(ctx.n_so) if not ref >> b & 1]
    singles = [ref & ~(1 << h) | 1 << p for h in _bits(ref) for p in empty[:12] if (h - p) % 2 == 0]
    keys = [ref] + [ref | 1 << p for p in empty[:6]] + singles[:20]
    pops = [-20000] + [(-1) ** i * (9000 + 37 * i) for i in range(1, len(keys))]
    ctx.import_walkers(np.array(keys, np.uint64)[:, None], np.array(pops, np.int32))
    for expected in ((418807, 286, -20000, 562, 401, 7519), (624971, 440, -20019, 510, 322, 5677),
                     (792588, 570, -20019, 439, 251, -104287)):
        ctx.step(1)
        e = ctx.estimators()
        assert tuple(e[f] for f in FIELDS) == expected
    ctx.close()


# amplitudes of the list: the prefix staged in LDS with bucket bounds (up to 4095), and in global memory
@pytest.mark.parametrize("amplitudes", [4094, 4095, 4096, 20000])
def test_prefix_at_the_end_of_its_staging(amplitudes):
    """The composite clusters of lists on both sides of the largest prefix a block stages."""
    sysd = dict(kind="ueg", rs=1.0, ecut_n2=9, n_alpha=7, n_beta=7)
    q = dict(tau=0.001, rng_seed=13, init_pop=1.0, target_population=1e9, fixed_point_bits=8, spawn_cutoff=0.1)
    ctx = gpu_context([sysd], [dict(q, method=F.CCMC, ccmc_truncation=2)], main_capacity=1 << 16,
                      spawn_capacity=1 << 20)
    oq = oracle_qmc(sysd, q)
    oq.method, oq.ccmc_truncation = O.CCMC, 2
    run = O.Run(oracle_system(sysd), oq)
    ref = sum(int(x) << 64 * i for i, x in enumerate(ctx.export()[0][0]))
    held = [b for b in range(ctx.n_so) if ref >> b & 1]
    empty = [b for b in range(ctx.n_so) if not ref >> b & 1]
    rng = np.random.default_rng(amplitudes)
    dets = {ref: 256 * 4000}
    while len(dets) < amplitudes:
        n = int(rng.integers(1, 3))
        holes, parts = rng.choice(held, n, replace=False), rng.choice(empty, n, replace=False)
        det = ref ^ sum(1 << int(b) for b in (*holes, *parts))
        if sum(int(b) & 1 for b in holes) == sum(int(b) & 1 for b in parts):
            dets.setdefault(det, int(rng.integers(1, 600)) * int(rng.choice([-1, 1])))
    keys = np.array([[d >> 64 * w & (1 << 64) - 1 for w in range(ctx.W)] for d in dets], np.uint64)
    pops = np.array(list(dets.values()), np.int32)
    say(f"[case] CCSD on the 14-electron gas in 123 plane waves, {amplitudes} amplitudes")
    for x in (ctx, run):
        x.import_walkers(keys, pops)
    for it in range(3):
        ctx.step(1)
        run.step(1)
        assert_same_lists(ctx, run, where=f"{amplitudes} amplitudes, iteration {it}")
        assert_same_estimators(ctx.estimators(), run.estimators(), where=f"{amplitudes} amplitudes, iteration {it}")
        assert ctx.estimators()["n_cluster_spawns"] > 0
    ctx.close()
