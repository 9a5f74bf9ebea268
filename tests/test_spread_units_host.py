"""Block tables of batch launches (hmc_test_spread_units, no GPU needed): every workgroup of every unit once,
and through the XCD remap an eighth of each unit's workgroups, in order and give or take one, on every XCD."""
import random

import pytest

from paper_2204_14241_amd import hmc


@pytest.mark.parametrize("seed", range(12))
def test_spread_units(seed):
    rng = random.Random(seed)
    lattices, nrhs = rng.choice([1, 2, 5, 12, 64]), rng.choice([1, 2, 4])
    vols = [rng.choice([64, 144 * 40, 576 * 80, 2304 * 80]) for _ in range(lattices)]
    counts = [rng.choice([1, 2, 7, 8, 9, 40, 333]) for _ in range(lattices * nrhs)]
    table = hmc.test_spread_units(vols, counts, nrhs)
    assert sorted(table) == [(u, w) for u, n in enumerate(counts) for w in range(n)]
    on = [[[] for _ in counts] for _ in range(8)]
    for bid in range(len(table)):
        u, w = table[hmc.test_xcd_remap(bid, len(table))]
        on[bid % 8][u].append(w)
    for u, n in enumerate(counts):
        for xcd in range(8):
            mine = on[xcd][u]
            assert n // 8 <= len(mine) <= n // 8 + 1
            assert mine == list(range(mine[0], mine[0] + len(mine))) if mine else n < 8


def test_spread_units_rejects_bad_arguments():
    assert hmc.test_spread_units([64], [1, 2], 3) is None
    assert hmc.test_spread_units([64, 64], [0, 0], 1) == []
