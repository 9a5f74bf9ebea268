"""FP64 solves whose status chunks are cut to an estimate (from the records and the context's last solve):
solutions and iteration counts are bit for bit those of the same solve after itself, after a shorter
solve, after a longer one and from graphs of whole chunks, with the marches, the tile kernels and the
preconditioner's separate passes."""
import pytest

import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Lt,n,precond,shape", [
    (12, 40, 2, None, None), (12, 40, 2, None, (4, 8)), (12, 40, 1, None, (0, 0)), (6, 20, 3, None, None),
    (36, 24, 1, "fourier", None), (12, 40, 2, "fourier", (4, 8)), (12, 40, 2, "fourier", (0, 0)), (20, 40, 1, "fourier", None)])
def test_solutions_do_not_depend_on_earlier_solves(hip, L, Lt, n, precond, shape):
    import torch
    print(f"chunk lengths {L}x{L}x{Lt} n={n} {precond} {shape}", flush=True)
    g = S.rng(19 * L + Lt)
    phi, soft = (torch.from_numpy(S.draw_phi(g, L, Lt, v)).cuda() for v in (0.5, 0.05))
    b = torch.from_numpy(S.draw_spinor(g, L, Lt, n)).cuda()
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precond=precond)
    if shape is not None:
        h.set_cg_march(*shape, "fp64")
    assert not h.solve_path(n) & {"one_kernel", "join_a"}
    x, st = h.cg_solve(phi, b)
    assert st.status == 0 and max(st.iterations) > 8
    again, at = h.cg_solve(phi, b)
    h.cg_solve(soft, b)
    after, ft = h.cg_solve(phi, b)
    h.set_params(cg_tol=1e-13)
    h.cg_solve(phi, b)
    h.set_params(cg_tol=1e-10)
    shorter, lt = h.cg_solve(phi, b)
    h.set_graphs(True)
    graph, gt = h.cg_solve(phi, b)
    for y in (again, after, shorter, graph):
        assert torch.equal(x, y)
    for s in (at, ft, lt, gt):
        assert list(s.iterations) == list(st.iterations) and list(s.true_resid) == list(st.true_resid)
