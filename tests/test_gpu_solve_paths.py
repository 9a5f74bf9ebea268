"""Which kernels a solve runs (include/hmc_testing.h, hmc_test_solve_path), at both sides of each rule:
what the comparisons of the one-kernel solve and of the joined steps with the separate kernels compare."""
import pytest

pytestmark = pytest.mark.gpu

SMALL, A, B = {"one_kernel"}, {"join_a"}, {"join_b"}


# every size of the one-kernel comparison, the largest lattices of the rule and the next
@pytest.mark.parametrize("L,Lt,n", [(4, 2, 1), (4, 8, 3), (6, 5, 2), (10, 5, 1), (6, 14, 2), (8, 8, 16), (4, 32, 1)])
def test_one_kernel(hip, L, Lt, n):
    h = hip.HMC(L, Lt, n_pf=n)
    assert h.solve_path(n) == SMALL
    h.set_params(precision="mixed")
    assert "one_kernel" not in h.solve_path(n)
    h.set_params(precision="fp64", precond="fourier")
    assert "one_kernel" not in h.solve_path(n)
    ref = hip.HMC(L, Lt, n_pf=n)
    ref.set_cg_march(*ref.cg_march("fp64"), "fp64")
    assert "one_kernel" not in ref.solve_path(n)


@pytest.mark.parametrize("L,Lt", [(6, 15), (8, 9), (4, 33)])
def test_above_one_kernel(hip, L, Lt):
    assert "one_kernel" not in hip.HMC(L, Lt).solve_path(1)


# both steps or step B alone by the slice's size (FP32 L <= 24, FP64 L <= 16) or 160 slices; neither
# where two workgroups do not fit a CU and more than 256 would run, or one does not fit
@pytest.mark.parametrize("precision,L,Lt,n,joined", [
    ("mixed", 4, 2, 1, A | B), ("mixed", 16, 10, 4, A | B), ("mixed", 24, 4, 1, A | B), ("mixed", 28, 5, 1, B),
    ("mixed", 28, 50, 3, B), ("mixed", 28, 54, 3, A | B), ("mixed", 32, 4, 1, B), ("mixed", 32, 70, 4, A | B),
    ("mixed", 36, 64, 4, A | B), ("mixed", 36, 70, 4, set()), ("mixed", 48, 4, 1, B), ("mixed", 50, 4, 1, set()),
    ("fp64", 4, 9, 3, A | B), ("fp64", 16, 10, 4, A | B), ("fp64", 18, 4, 1, B), ("fp64", 20, 7, 2, B),
    ("fp64", 28, 5, 1, B), ("fp64", 28, 54, 3, A | B), ("fp64", 28, 64, 4, A | B), ("fp64", 28, 90, 3, set()),
    ("fp64", 32, 4, 1, B), ("fp64", 36, 4, 1, set()), ("fp64", 48, 4, 1, set())])
def test_joined(hip, precision, L, Lt, n, joined):
    h = hip.HMC(L, Lt, n_pf=n, precision=precision, precond="fourier")
    assert h.solve_path(n) & (A | B) == joined
    h.set_kernel_timing(True)
    assert not h.solve_path(n) & (A | B)
    h.set_kernel_timing(False)
    assert h.solve_path(n) & (A | B) == joined
    h.set_params(precond=None)
    assert not h.solve_path(n) & (A | B)
    h.set_params(precond="fourier")
    h.set_cg_march(*h.cg_march(precision), precision)
    assert not h.solve_path(n) & (A | B)
