"""The march cut that a solve takes by itself (hmc_test_auto_cut, no GPU needed) on lattices whose cuts were
timed: it is one of those within 8% of the fastest.  Where workgroups of five to eight wavefronts share a
CU the estimate has to know that a SIMD holds three wavefronts, not a CU twelve."""
import pytest

from paper_2204_14241_amd import hmc

# (precision, two-site hops, L, L_tau, right-hand sides): {bands: slices per segment} timed on an MI355X at
# most 1.08 times the fastest cut of some hundred
GOOD = {
    ("mixed", True, 36, 50, 16): {2: (8, 10), 3: (10, 12), 4: (6, 8), 5: (6, 8, 10), 6: (6, 8, 10), 8: (8, 10), 9: (8, 10), 12: (8, 10)},
    ("mixed", True, 60, 80, 3): {5: (6,), 6: (6, 8), 8: (8,), 9: (10,), 10: (10,), 15: (3, 6, 8), 20: (10,), 30: (8,)},
    ("mixed", True, 64, 50, 4): {6: (6,), 7: (6, 8), 8: (8,), 16: (6, 8), 32: (8,)},
    ("mixed", True, 32, 64, 16): {2: (8, 10), 3: (4, 6), 4: (4, 6, 8, 10), 6: (8,), 7: (8,), 8: (8,)},
    ("mixed", True, 64, 100, 2): {6: (6,), 7: (6, 8), 8: (8,), 11: (10,), 16: (8,), 22: (6,)},
    ("mixed", False, 32, 64, 16): {2: (8, 10), 3: (4, 6, 8), 4: (4, 6, 8, 10), 5: (6, 8, 10, 12), 6: (6, 8, 10), 7: (6, 8, 10), 8: (6, 8), 11: (8, 10, 12), 16: (6, 8, 10)},
    ("fp64", True, 24, 40, 16): {2: (6,), 3: (8,), 4: (4, 6, 10), 6: (8,)},
    ("fp64", True, 32, 128, 2): {3: (4,), 4: (4,), 8: (4,)},
    ("fp64", True, 32, 32, 8): {3: (4,), 4: (4, 6), 5: (6,), 8: (4, 8)},
    ("fp64", True, 32, 32, 16): {3: (8,), 4: (8, 10), 8: (6, 8, 10)},
    ("mixed", False, 40, 100, 1): {2: (1,), 4: (1, 2), 5: (1, 2), 8: (2,), 10: (2,)},
    ("fp64", False, 40, 100, 2): {4: (4, 6), 5: (2, 4, 6), 6: (6,), 7: (3, 6), 8: (8,), 10: (2, 3, 4), 14: (3, 4, 6), 20: (4, 6)},
    ("fp64", False, 60, 160, 1): {10: (4, 8, 10), 12: (4, 8, 10, 12), 15: (6, 10, 12), 20: (8,), 30: (10, 12), 60: (10,)},
}


@pytest.mark.parametrize("case", GOOD, ids=str)
def test_chosen_cut_is_fast(case):
    precision, nn2, L, Lt, n = case
    rows, slices = hmc.test_auto_cut(L, Lt, n, precision, nn2)
    assert slices in GOOD[case].get((L + rows - 1) // rows, ())


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nn2", [False, True])
def test_cut_bounds(precision, nn2):
    for L in (4, 6, 14, 22, 60, 100, 128, 170, 172, 204, 256):
        for Lt in (2, 3, 7, 40, 200):
            if L * L * Lt >= 2**26:
                continue
            for n in (1, 3, 16):
                rows, slices = hmc.test_auto_cut(L, Lt, n, precision, nn2)
                assert 1 <= rows <= L and 1 <= slices <= 12
