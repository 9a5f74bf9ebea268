"""The march cut a context chooses by itself: solves on lattices at the edges of the rule (two time
slices, segments of one slice, bands that do not divide L, several right-hand sides, the two-site
hops, a lattice no FP64 band fits), FP64 true residual by the oracle's operator <= the solver's
1e-10 (Eq. 22)."""
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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,Lt,n,nnn", [(4, 2, 1, False), (6, 3, 3, True), (22, 5, 2, False), (26, 31, 1, True),
                                        (34, 7, 1, False), (256, 2, 1, False)])
def test_default_cut_solves(hip, precision, L, Lt, n, nnn):
    import torch
    print(f"default cut {precision} {L}x{L}x{Lt} n={n} nnn={nnn}", flush=True)
    model = V1 if nnn else {}
    m = O.Model(L=L, Lt=Lt, **model)
    g = S.rng(61 * L + Lt)
    phi, b = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    h = hip.HMC(L, Lt, n_pf=n, cg_tol=1e-10, precision=precision, model=model)
    rows, slices = h.cg_march(precision)
    assert 1 <= rows <= L and slices >= 1
    x, st = h.cg_solve(torch.from_numpy(phi).cuda(), torch.from_numpy(b).cuda())
    assert st.status == 0
    x = x.cpu().numpy()
    for k in range(n):
        assert np.linalg.norm(b[k] - O.apply_MdagM(m, phi, x[k])) <= 1e-10 * np.linalg.norm(b[k])


def test_small_batch_cut(hip):
    """A batch that cannot fill the chip takes shorter segments; the reported cuts are the ones in use."""
    bt = hip.Batch([(12, 40, 0.1), (24, 80, 0.0)], n_pf=1, precision="mixed")
    assert [bt.cg_march(i, "mixed")[0] for i in range(2)] == [(8, 1), (8, 1)]
    bt.set_cg_march(8, 8)
    assert [bt.cg_march(i, "mixed")[0] for i in range(2)] == [(8, 8), (8, 8)]


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,Lt,n", [(4, 2, 1), (6, 3, 3), (14, 11, 2), (34, 9, 1), (60, 13, 1), (128, 2, 1)])
def test_default_one_pass_shape(hip, precision, L, Lt, n):
    """M^dagger M at the shape chosen by itself (Eq. 22) against the oracle: 1e-14 (FP64) and 2e-6 (FP32, on
    the rounded inputs) of the largest entry, the bars of the one-pass kernels at set shapes."""
    import torch
    m = O.Model(L=L, Lt=Lt)
    g = S.rng(5 * L + Lt)
    phi, psi = S.draw_phi(g, L, Lt, 0.5), S.draw_spinor(g, L, Lt, n)
    h = hip.HMC(L, Lt, max_rhs=n)
    print(f"one pass {precision} {L}x{L}x{Lt} n={n} shape {h.mdm_shape(precision, n)}", flush=True)
    if precision == "mixed":
        phi, psi = phi.astype(np.float32), psi.astype(np.complex64)
    f = h.apply_MdagM_f32 if precision == "mixed" else h.apply_MdagM
    got = f(torch.from_numpy(phi).cuda(), torch.from_numpy(psi).cuda()).cpu().numpy().astype(np.complex128)
    want = np.stack([O.apply_MdagM(m, phi.astype(np.float64), psi[k].astype(np.complex128)) for k in range(n)])
    assert np.abs(got.reshape(want.shape) - want).max() <= (2e-6 if precision == "mixed" else 1e-14) * np.abs(want).max()
