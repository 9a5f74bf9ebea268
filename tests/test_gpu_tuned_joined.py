"""Preconditioned solves of small lattices keep their joined steps (hmc_test_solve_path) whatever shape the
autotuner chose for the separate kernels, tile kernels and a tile step B among them: against the oracle's
operator (true residual, Eq. 22) and against a context without a tuned shape, whose iterations agree
within one (another order of the partial sums of each chunk's first step A)."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu

V1 = dict(t=((1.0, 0.0), (0.0, 1.0)), tn=((0.0, 0.45), (-0.45, 0.0)), mu=(-0.47, 0.47))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nnn", [False, True])
@pytest.mark.parametrize("L,Lt,n,joined", [(12, 40, 2, {"join_a", "join_b"}), (28, 10, 1, {"join_b"})])
def test_tuned_shape_keeps_joined_steps(hip, tmp_path, monkeypatch, L, Lt, n, joined, nnn, precision):
    import torch
    print(f"tuned joined steps {L}x{L}x{Lt} n={n} nnn={nnn} {precision}", flush=True)
    model = V1 if nnn else {}
    kw = dict(n_pf=n, cg_tol=1e-10, precision=precision, model=model, precond="fourier")
    plain = hip.HMC(L, Lt, **kw)
    assert plain.solve_path(n) == joined | {"march"}
    # a line of the tuning cache as the autotuner writes it, its choice replaced
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("HMC_TUNE_CACHE", str(cache))
    t = hip.HMC(4, 6, **kw)
    g = S.rng(17 * L + Lt)
    b4 = torch.from_numpy(S.draw_spinor(g, 4, 6, n)).cuda()
    t.autotune(torch.from_numpy(S.draw_phi(g, 4, 6, 0.5)).cuda(), b4)
    line, = [v for v in cache.read_text().splitlines() if v.startswith(f"one 4 6 {n} ")]
    key = line.split()[:-8]
    key[1:3] = [str(L), str(Lt)]
    cache.write_text(" ".join(key + "512 512 0 0 0 0 0 0".split()) + "\n")
    h = hip.HMC(L, Lt, **kw)
    assert h.cg_march(precision) == (0, 0) and not h.cg_march_step_b(precision)
    assert h.solve_path(n) == joined
    m = O.Model(L=L, Lt=Lt, **model)
    phi, b = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    d_phi, d_b = torch.from_numpy(phi).cuda(), torch.from_numpy(b).cuda()
    (x, st), (y, rt) = h.cg_solve(d_phi, d_b), plain.cg_solve(d_phi, d_b)
    assert st.status == 0 and rt.status == 0
    for k in range(n):
        r = np.linalg.norm(b[k] - O.apply_MdagM(m, phi, x[k].cpu().numpy()))
        assert r <= 1e-10 * np.linalg.norm(b[k]) * (1 + 1e-6)
        assert st.reliable_updates[k] == rt.reliable_updates[k]
        assert precision == "mixed" or abs(st.iterations[k] - rt.iterations[k]) <= 1
    h.set_graphs(True)
    z, gt = h.cg_solve(d_phi, d_b)
    assert torch.equal(x, z) and list(gt.iterations) == list(st.iterations)
    # a shape that the caller sets is still what runs
    h.set_cg_march(0, 0, precision)
    assert h.solve_path(n) == set()
