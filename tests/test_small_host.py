"""The decision of the one-kernel solve after a true residual (small.h), run on the host: every solve
ends, whatever its tolerance, at most 128 iterations past the cap."""
import pytest

from paper_2204_14241_amd import hmc

ON, DONE, STOPPED, FAILED = 0, 3, 4, 5


@pytest.mark.parametrize("maxit", [1, 50, 2**31 - 1])
def test_small_solve_ends(maxit):
    # the iterated residual passes at every iteration and the true one never does
    last = min(maxit + 128, 2**31 - 1)
    assert hmc.test_small_next(2.0, 1.0, False, maxit - 1, maxit) == ON
    if last < 2**31 - 1:
        assert hmc.test_small_next(2.0, 1.0, False, last - 1, maxit) == ON
        assert hmc.test_small_next(2.0, 1.0, False, last, maxit) == STOPPED
    assert hmc.test_small_next(2.0, 1.0, True, maxit, maxit) == STOPPED


@pytest.mark.parametrize("capped", [False, True])
def test_small_solve_outcomes(capped):
    assert hmc.test_small_next(1.0, 1.0, capped, 7, 50) == DONE
    assert hmc.test_small_next(0.0, 0.0, capped, 7, 50) == DONE
    assert hmc.test_small_next(float("nan"), 1.0, capped, 7, 50) == FAILED
    assert hmc.test_small_next(float("inf"), 1.0, capped, 7, 50) == FAILED
