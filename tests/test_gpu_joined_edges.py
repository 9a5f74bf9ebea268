"""Edges of the joined steps and of the cut by the number of right-hand sides: non-finite input ends with
HMC_ERR_NONFINITE as with the separate kernels and leaves the context usable; a solve repeated with the same
arguments and settings gives the same bits; a vector solved with others, with kernel times sampled or at a
set shape, agrees to the solver's tolerance (include/hmc.h, hmc_set_cg_march)."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(a).cuda()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,Lt,n", [(6, 5, 2), (16, 20, 3), (28, 5, 2)])
@pytest.mark.parametrize("bad", ["b_nan", "b_inf", "phi_nan", "phi_inf"])
def test_non_finite_input(hip, precision, L, Lt, n, bad):
    import torch
    print(f"non-finite {bad} {L}x{L}x{Lt} n={n} {precision}", flush=True)
    g = S.rng(23 * L + Lt)
    phi, b = dev(S.draw_phi(g, L, Lt, 0.5)), dev(S.draw_spinor(g, L, Lt, n))
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precision=precision, precond="fourier")
    ref = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precision=precision, precond="fourier")
    ref.set_cg_march(*ref.cg_march(precision), precision)
    assert "join_b" in h.solve_path(n) and not ref.solve_path(n) & {"join_a", "join_b"}
    x, st = h.cg_solve(phi, b)
    bad_phi, bad_b = phi.clone(), b.clone()
    v = float("nan") if bad.endswith("nan") else float("inf")
    if bad.startswith("b"):
        bad_b.view(n, -1)[n - 1, 2 * L * L * Lt - L] = v
    else:
        bad_phi[1, Lt - 1, 0, L - 1] = v
    for ctx in (h, ref):
        with pytest.raises(RuntimeError, match="non-finite|-3"):
            ctx.cg_solve(bad_phi, bad_b)
    again, at = h.cg_solve(phi, b)
    assert torch.equal(x, again) and list(at.iterations) == list(st.iterations)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,Lt,n,precond", [(4, 8, 4, None), (16, 40, 4, "fourier"), (28, 54, 3, "fourier"),
                                            (20, 60, 4, None), (36, 20, 3, None)])
def test_bits_and_agreement(hip, precision, L, Lt, n, precond):
    import torch
    print(f"agreement {L}x{L}x{Lt} n={n} {precond} {precision}", flush=True)
    m = O.Model(L=L, Lt=Lt)
    g = S.rng(29 * L + Lt)
    phi, b = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    d_phi, d_b = dev(phi), dev(b)
    kw = dict(cg_tol=1e-10, precision=precision, precond=precond)
    h = hip.HMC(L, Lt, n_pf=n, **kw)
    x, st = h.cg_solve(d_phi, d_b)
    again, _ = h.cg_solve(d_phi, d_b)
    other, _ = hip.HMC(L, Lt, n_pf=n, **kw).cg_solve(d_phi, d_b)
    assert torch.equal(x, again) and torch.equal(x, other)
    one, ot = h.cg_solve(d_phi, d_b[:1].contiguous())
    h.set_kernel_timing(True)
    timed, tt = h.cg_solve(d_phi, d_b)
    h.set_kernel_timing(False)
    back, _ = h.cg_solve(d_phi, d_b)
    assert torch.equal(x, back)
    for y, s, k in [(one, ot, 1), (timed, tt, n)]:
        for j in range(k):
            r = np.linalg.norm(b[j] - O.apply_MdagM(m, phi, y[j].cpu().numpy())) / np.linalg.norm(b[j])
            assert r <= 1e-10 * (1 + 1e-6)
            assert precision == "mixed" or abs(s.iterations[j] - st.iterations[j]) <= 1
