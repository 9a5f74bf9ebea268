"""The metric's transforms of real fields, two slices at a time and half the frequencies of a slice,
against the oracle with a table that is not even in the frequency (the two halves of a pair of
frequencies then count differently): 1e-12 of the largest entry, or relative for the sums, as for the
other metric tests.  Sizes: one pair of slices, odd counts (the last slice stands alone), a single transform
stage and the widest radices, a launch of small and of large workgroups in the tau pass."""
import numpy as np
import pytest

import synth_inputs as S
from oracle import metric as Me

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Lt", [(4, 2), (4, 3), (6, 2), (14, 25), (16, 7), (28, 9), (32, 128), (54, 12)])
def test_uneven_table(hip, L, Lt):
    import torch
    print(f"metric pairs {L}x{L}x{Lt}", flush=True)
    g = S.rng(900 + L + Lt)
    s = S.draw_metric_table(g, L, Lt, even=False)
    v, xi = S.draw_phi(g, L, Lt, 0.7), S.draw_momentum(g, L, Lt)
    d = {k: torch.from_numpy(np.ascontiguousarray(a)).cuda() for k, a in (("s", s), ("v", v), ("xi", xi))}
    h = hip.HMC(L, Lt)
    h.set_metric(d["s"])
    want = Me.momenta(s, xi)
    assert np.abs(h.metric_momenta(d["xi"]).cpu().numpy() - want).max() <= 1e-12 * np.abs(want).max()
    assert h.metric_kinetic(d["xi"]) == pytest.approx(Me.kinetic(s, xi), rel=1e-12)
    assert h.metric_norm2(d["v"]) == pytest.approx(Me.metric_norm2(s, v), rel=1e-12)
    acc = torch.zeros(3, Lt, L, L, dtype=torch.float64, device="cuda")
    h.metric_accumulate(d["v"], acc)
    h.metric_accumulate(d["xi"], acc)
    ref = Me.power_spectrum(v) + Me.power_spectrum(xi)
    assert np.abs(acc.cpu().numpy() - ref).max() <= 1e-12 * ref.max()
