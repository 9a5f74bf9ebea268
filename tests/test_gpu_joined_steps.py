"""The preconditioned solve of a small lattice with steps A and B joined to the slice transforms
beside them (three launches an iteration) against the oracle's operator (true residual, Eq. 22) and
against the separate kernels on the same inputs.  Converged: FP64 iteration counts agree within one,
mixed ones end after the same reliable updates.  Stopped after three iterations: the iterates differ by
rounding only, FP64 1e-12 relative; FP32 about 30 roundings of 6e-8 a value and iteration, through an
operator of norm about 10: 2e-5 relative."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu

V1 = dict(t=((1.0, 0.0), (0.0, 1.0)), tn=((0.0, 0.45), (-0.45, 0.0)), mu=(-0.47, 0.47))


# the least lattice, one transform stage and several, odd counts of slices, the widest radices, step B
# joined alone (28, 32), step A too for the number of slices (28 x 28 x 54), the largest slices of
# either precision
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nnn", [False, True])
@pytest.mark.parametrize("L,Lt,n", [(4, 2, 1), (4, 9, 3), (6, 5, 2), (10, 7, 1), (14, 4, 2), (16, 10, 4), (20, 7, 2),
                                    (28, 5, 1), (32, 4, 1), (28, 54, 3), (48, 4, 1)])
def test_joined_steps(hip, L, Lt, n, nnn, precision):
    import torch
    print(f"joined steps {L}x{L}x{Lt} n={n} nnn={nnn} {precision}", flush=True)
    model = V1 if nnn else {}
    m = O.Model(L=L, Lt=Lt, **model)
    g = S.rng(11 * L + Lt + n)
    phi, b = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    if n > 1:
        b[n - 1] = 0.0
    d_phi, d_b = torch.from_numpy(phi).cuda(), torch.from_numpy(b).cuda()
    hs = [hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precision=precision, model=model, precond="fourier") for _ in range(2)]
    hs[1].set_cg_march(*hs[1].cg_march(precision), precision)      # a launch shape: the separate kernels
    (x, st), (y, rt) = [h.cg_solve(d_phi, d_b) for h in hs]
    assert st.status == 0 and rt.status == 0
    for k in range(n):
        xk, bn = x[k].cpu().numpy(), np.linalg.norm(b[k])
        assert np.linalg.norm(b[k] - O.apply_MdagM(m, phi, xk)) <= 1e-10 * bn * (1 + 1e-6)
        assert st.reliable_updates[k] == rt.reliable_updates[k]
        if precision == "fp64":
            assert abs(st.iterations[k] - rt.iterations[k]) <= 1
        if bn == 0.0:
            assert np.count_nonzero(xk) == 0 and st.iterations[k] == 0
    for h in hs:
        h.set_params(cg_maxit=3)
    (x, st), (y, rt) = [h.cg_solve(d_phi, d_b) for h in hs]
    assert st.status == rt.status and list(st.iterations) == list(rt.iterations)
    bar = 1e-12 if precision == "fp64" else 2e-5
    assert float((x - y).norm()) <= bar * float(y.norm())


# counts of iterations over one status chunk: step A joined, step B alone
@pytest.mark.parametrize("L,Lt,n", [(16, 80, 2), (28, 54, 3), (28, 60, 1)])
def test_joined_steps_do_not_depend_on_earlier_solves_or_graphs(hip, L, Lt, n):
    import torch
    print(f"joined steps repeated {L}x{L}x{Lt} n={n}", flush=True)
    g = S.rng(13 * L + Lt)
    phi, soft = (torch.from_numpy(S.draw_phi(g, L, Lt, v)).cuda() for v in (0.5, 0.05))
    b = torch.from_numpy(S.draw_spinor(g, L, Lt, n)).cuda()
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precond="fourier")
    x, st = h.cg_solve(phi, b)
    again, _ = h.cg_solve(phi, b)
    short = h.cg_solve(soft, b)[1]
    after, at = h.cg_solve(phi, b)
    assert max(st.iterations) > 40 > max(short.iterations)
    h.set_graphs(True)
    graph, gt = h.cg_solve(phi, b)
    for y in (again, after, graph):
        assert torch.equal(x, y)
    assert list(at.iterations) == list(gt.iterations) == list(st.iterations)
