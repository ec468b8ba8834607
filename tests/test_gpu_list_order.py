"""Lists read back and imported around the sizes from which they are sorted by
several threads: export in key order, import in any order, other instances kept,
duplicates refused."""
import numpy as np
import pytest

from gpu_helpers import gpu_context, say
from paper_1811_11679_amd import fciqmc as F
from paper_1811_11679_amd import workloads

pytestmark = pytest.mark.gpu


def _keys(rng, n, bits, words, electrons):
    """n different determinants, half the electrons of each spin"""
    rows = set()
    half = electrons // 2
    while len(rows) < n:
        up = rng.choice(bits // 2, half, replace=False)
        down = rng.choice(bits // 2, half, replace=False)
        rows.add(sum(1 << 2 * int(p) for p in up) + sum(1 << 2 * int(p) + 1 for p in down))
    ints = list(rows)
    mask = (1 << 64) - 1
    return np.array([[k >> 64 * w & mask for w in range(words)] for k in ints], np.uint64)


def _ordered(keys, pops):
    order = np.lexsort(tuple(keys[:, w] for w in range(keys.shape[1])))
    return keys[order], pops[order]


@pytest.mark.parametrize("n", [1, 4095, 16383, 16384, 32768, 70001])
@pytest.mark.parametrize("ecut,bits,words", [(3, 54, 1), (5, 114, 2), (9, 246, 4)])
def test_import_then_export(n, ecut, bits, words):
    rng = np.random.default_rng(n + words)
    sysd = dict(kind="ueg", rs=1.0, ecut_n2=ecut, n_alpha=7, n_beta=7)
    q = dict(workloads.UEG14["qmc"], init_pop=100.0, target_population=1e4)
    say(f"[case] {n} determinants of {words} key words, two instances")
    ctx = gpu_context([sysd, sysd], [q, q], replicas=[0, 1], main_capacity=1 << 18, spawn_capacity=1 << 18)
    held = ctx.export(0)
    keys = _keys(rng, n, bits, words, 14)
    pops = rng.integers(1, 1000, n).astype(np.int32) * rng.choice([-1, 1], n).astype(np.int32)
    ctx.import_walkers(keys, pops, instance=1)
    for got, want in zip(ctx.export(1) + ctx.export(0), _ordered(keys, pops) + held):
        assert np.array_equal(got, want)
    assert ctx.estimators(1)["n_occupied"] == n
    if n > 1:
        keys[n // 2] = keys[n - 1]
        with pytest.raises(F.FqError):
            ctx.import_walkers(keys, pops, instance=1)
    ctx.close()
