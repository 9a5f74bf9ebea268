"""Contexts of different sizes side by side in one process: the preconditioner and the metric at slices
that need more than 64 KB of LDS work whether the context asked for them at its creation or later, and
after a small lattice's context has been made and used in between.  Against the oracle's operator (true
residual, Eq. 22) and metric."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S
from oracle import metric as Me

pytestmark = pytest.mark.gpu


def resid(m, phi, b, x):
    return np.linalg.norm(b - O.apply_MdagM(m, phi, x)) / np.linalg.norm(b)


def solve(h, L, Lt, seed):
    import torch
    g = S.rng(seed)
    phi, b = S.draw_phi(g, L, Lt, 0.3), S.draw_spinor(g, L, Lt, 1)
    x, st = h.cg_solve(torch.from_numpy(phi).cuda(), torch.from_numpy(b).cuda())
    assert st.status == 0
    assert resid(O.Model(L=L, Lt=Lt), phi, b[0], x[0].cpu().numpy()) <= h._p.cg_tol * (1 + 1e-6)


# FP64: 130 KB a slice at L = 90 (wide radices at 98); FP32: 66 KB at 90
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,Lt", [(90, 4), (98, 4)])
def test_preconditioner_asked_for_later(hip, L, Lt, precision):
    print(f"precond later {L}x{L}x{Lt} {precision}", flush=True)
    big = hip.HMC(L, Lt, cg_tol=1e-9)
    small = hip.HMC(6, 4, cg_tol=1e-9, precond="fourier", precision=precision)
    solve(small, 6, 4, 1)
    big.set_params(precision=precision, precond="fourier")
    solve(big, L, Lt, 2)
    small2 = hip.HMC(8, 6, cg_tol=1e-9, precond="fourier", precision=precision)
    solve(small2, 8, 6, 3)
    solve(big, L, Lt, 4)
    big.set_graphs(True)
    solve(big, L, Lt, 5)


def test_batch_preconditioner_asked_for_later(hip):
    import torch
    chains = [(90, 4), (6, 6)]
    bt = hip.Batch([(L, Lt, 0.5) for L, Lt in chains], cg_tol=1e-9)
    solve(hip.HMC(6, 4, cg_tol=1e-9, precond="fourier"), 6, 4, 1)
    bt.set_params(precond="fourier")
    g = S.rng(9)
    phi = [S.draw_phi(g, L, Lt, 0.3) for L, Lt in chains]
    b = [S.draw_spinor(g, L, Lt, 1) for L, Lt in chains]
    x, st = bt.cg_solve(bt.pack_phi([torch.from_numpy(v).cuda() for v in phi]),
                        bt.pack_spinors([torch.from_numpy(v).cuda() for v in b]))
    assert st["status"] == 0
    for (L, Lt), p, v, y in zip(chains, phi, b, bt.unpack_spinors(x)):
        assert resid(O.Model(L=L, Lt=Lt), p, v[0], y[0].cpu().numpy()) <= 1e-9 * (1 + 1e-6)


# L = 100 takes 162,400 of the 163,840 bytes of a CU's LDS; odd and even N_tau; 98 = 7 x 14.  Two
# transforms in FP64: a few units of 1e-16 per stage, eight stages each way: 1e-13 of the largest value.
@pytest.mark.parametrize("L,Lt", [(100, 3), (100, 4), (98, 5), (96, 2), (80, 7), (56, 3)])
def test_metric_of_large_slices(hip, L, Lt):
    import torch
    print(f"metric {L}x{L}x{Lt}", flush=True)
    g = S.rng(31 * L + Lt)
    sigma = g.uniform(0.5, 2.0, (3, Lt, L, L))
    xi = g.standard_normal((3, Lt, L, L))
    h = hip.HMC(L, Lt)
    h.set_metric(torch.from_numpy(sigma).cuda())
    hip.HMC(6, 4).set_metric(torch.ones(3, 4, 6, 6, dtype=torch.float64, device="cuda"))
    pi = h.metric_momenta(torch.from_numpy(xi).cuda())
    ref = Me.momenta(sigma, xi)
    assert np.abs(pi.cpu().numpy() - ref).max() <= 1e-13 * np.abs(ref).max()
    d_ref = torch.from_numpy(np.ascontiguousarray(ref)).cuda()
    for got, want in ((h.metric_kinetic(d_ref), Me.kinetic(sigma, ref)), (h.metric_norm2(d_ref), Me.metric_norm2(sigma, ref))):
        assert abs(got - want) <= 1e-12 * want
