"""The one-kernel solve of small lattices (FP64, no preconditioner, at most 512 sites) against the
oracle's operator (true residual <= tol, Eq. 22) and against the chunked kernels on the same inputs:
the iteration counts agree within one (another order of summation), an iteration cap stops both at the
same iterate (the first iterations differ by rounding: 1e-12 relative), a zero right-hand side returns
zero."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu

V1 = dict(t=((1.0, 0.0), (0.0, 1.0)), tn=((0.0, 0.45), (-0.45, 0.0)), mu=(-0.47, 0.47))


@pytest.fixture(scope="module")
def hip():
    import torch
    assert torch.cuda.is_available()
    from paper_2204_14241_amd import hmc
    return hmc


# one wavefront and less, counts that are no multiple of 64, the largest lattices of the rule
@pytest.mark.parametrize("nnn", [False, True])
@pytest.mark.parametrize("L,Lt,n", [(4, 2, 1), (4, 8, 3), (6, 5, 2), (10, 5, 1), (6, 14, 2), (8, 8, 16)])
def test_small_solve(hip, L, Lt, n, nnn):
    import torch
    print(f"one-kernel solve {L}x{L}x{Lt} n={n} nnn={nnn}", flush=True)
    model = V1 if nnn else {}
    m = O.Model(L=L, Lt=Lt, **model)
    g = S.rng(7 * L + Lt + n)
    phi, b = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    if n > 1:
        b[n - 1] = 0.0
    d_phi, d_b = torch.from_numpy(phi).cuda(), torch.from_numpy(b).cuda()
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-11, model=model)
    ref = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-11, model=model)
    ref.set_cg_march(*ref.cg_march("fp64"), "fp64")          # a launch shape: the chunked kernels
    (x, st), (y, rt) = h.cg_solve(d_phi, d_b), ref.cg_solve(d_phi, d_b)
    assert st.status == 0 and rt.status == 0
    for k in range(n):
        xk, bn = x[k].cpu().numpy(), np.linalg.norm(b[k])
        assert np.linalg.norm(b[k] - O.apply_MdagM(m, phi, xk)) <= 1e-11 * bn
        assert abs(st.iterations[k] - rt.iterations[k]) <= 1 and st.reliable_updates[k] == rt.reliable_updates[k]
        if bn == 0.0:
            assert np.count_nonzero(xk) == 0 and st.iterations[k] == 0 and st.true_resid[k] == 0.0
    for hh in (h, ref):
        hh.set_params(cg_maxit=3)
    (x, st), (y, rt) = h.cg_solve(d_phi, d_b), ref.cg_solve(d_phi, d_b)
    assert st.status == rt.status != 0 and st.iterations == rt.iterations
    assert float((x - y).norm()) <= 1e-12 * float(y.norm())
    assert np.allclose(st.true_resid, rt.true_resid, rtol=1e-10)
