"""The heat-bath spawn with pair weights summed from registers and by the general
loops: electron numbers and tables on both sides of where one gives way to the other."""
import pytest

from gpu_helpers import assert_same_estimators, assert_same_lists, gpu_context, oracle_qmc, oracle_system, say
from oracle import oracle as O
from paper_1811_11679_amd import synth, workloads

pytestmark = pytest.mark.gpu


# 10 orbitals: a table of 1.5 KB; 33: 17 KB, beyond 16; 46: none in LDS
@pytest.mark.parametrize("orbitals", [10, 33, 46])
@pytest.mark.parametrize("electrons", [2, 7, 8, 9, 10, 15, 16, 17])
@pytest.mark.parametrize("instances", [1, 2])
def test_electron_numbers(orbitals, electrons, instances):
    ints = synth.molecular_integrals(orbitals, n_chol=8)
    sysd = dict(kind="molecular", n_alpha=(electrons + 1) // 2, n_beta=electrons // 2)
    q = dict(workloads.MOL30["qmc"], tau=0.001, init_pop=1e4, target_population=3e4)
    say(f"[case] {electrons} electrons in {orbitals} orbitals, {instances} instances")
    ctx = gpu_context([sysd] * instances, [q] * instances, ints=ints, replicas=list(range(instances)),
                      main_capacity=1 << 17, spawn_capacity=1 << 17)
    ctx.step(10)
    for r in range(instances):
        run = O.Run(oracle_system(sysd, ints), oracle_qmc(sysd, q, replica=r))
        run.step(10)
        assert_same_lists(ctx, run, instance=r, where=f"instance {r}")
        assert_same_estimators(ctx.estimators(r), run.estimators(), where=f"instance {r}")
        assert run.estimators()["n_spawned"] > 20
    ctx.close()
