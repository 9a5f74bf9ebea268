"""One-kernel solves whose tolerance FP64 cannot reach end near the iteration cap, with a status that
agrees with their true residuals (include/hmc.h: HMC_ERR_NOT_CONVERGED, x and stats still written)."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu


# M^dagger M a multiple of the identity: every iteration brings the iterated residual below any
# tolerance, while the true one stays at the rounding of x
@pytest.mark.parametrize("maxit", [1, 40])
@pytest.mark.parametrize("tol", [1e-16, 1e-20])
def test_unreachable_tolerance_ends(hip, tol, maxit):
    import torch
    print(f"one-kernel solve, tol {tol}, cap {maxit}", flush=True)
    L, Lt, n = 4, 2, 3
    g = S.rng(5)
    phi, b = (torch.from_numpy(v).cuda() for v in (S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)))
    model = dict(t=((0.0, 0.0), (0.0, 0.0)), mu=(2.3, 2.3), lam=0.0)
    m = O.Model(L=L, Lt=Lt, **model)
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=tol, cg_maxit=maxit, model=model)
    x, st = h.cg_solve(phi, b)
    assert all(1 <= i <= maxit + 128 for i in st.iterations)
    met = [r <= tol for r in st.true_resid]
    assert st.status == (0 if all(met) else -2)
    # the reported residuals are the solution's (evaluated to some tens of roundings of |b|)
    for k in range(n):
        bk = b[k].cpu().numpy()
        r = np.linalg.norm(bk - O.apply_MdagM(m, phi.cpu().numpy(), x[k].cpu().numpy())) / np.linalg.norm(bk)
        assert abs(r - st.true_resid[k]) <= 1e-14
