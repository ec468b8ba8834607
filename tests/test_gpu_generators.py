"""Excitation generators at the sizes where their code paths change.

The heat-bath pair weights are summed in registers for up to 16 electrons on a
table staged in LDS, and by the general loop beyond that (or with several
different systems, which stage no table). Every list must equal the oracle's
bit for bit.
"""
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import synth, workloads

pytestmark = pytest.mark.gpu


# the smallest and largest numbers of electrons of the unrolled sums, one more,
# odd numbers, and keys of two words (more than 32 orbitals)
@pytest.mark.parametrize("orbitals,up,down", [(4, 1, 1), (6, 2, 1), (10, 3, 4), (12, 8, 7), (12, 8, 8), (12, 9, 8),
                                              (34, 2, 2), (36, 8, 8)])
def test_heat_bath_electrons(orbitals, up, down):
    ints = synth.molecular_integrals(orbitals)
    sysd = dict(kind="molecular", n_alpha=up, n_beta=down)
    q = dict(workloads.MOL30["qmc"], tau=0.01, init_pop=2e3, target_population=1e4, shift_damping=0.2)
    say(f"[case] molecular, {orbitals} orbitals, {up}+{down} electrons")
    ctx = gpu_context([sysd], [q], ints=ints, main_capacity=1 << 19, spawn_capacity=1 << 19)
    run = O.Run(oracle_system(sysd, ints), oracle_qmc(sysd, q))
    for blk in range(3):
        ctx.step(10)
        run.step(10)
        assert_same_lists(ctx, run, where=f"{orbitals} orbitals block {blk}")
        assert_same_estimators(ctx.estimators(), run.estimators(), where=f"{orbitals} orbitals block {blk}")
    say(f"[case] {ctx.estimators()['n_occupied']} determinants, {ctx.estimators()['n_spawned']} spawned")
    ctx.close()
