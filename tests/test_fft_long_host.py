"""FFT plans of long time extents (L_tau of a lattice of 4 x 4 may be up to 2^22), run on the host: the
plan holds every frequency once and the transform agrees with NumPy's (FP64, 1e-12 relative as for
shorter lengths).  Each length in a process of its own: a fault in a plan ends the process."""
import subprocess
import sys

import pytest

from conftest import ROOT

CODE = """
import sys; sys.path.insert(0, {root!r})
import numpy as np
from paper_2204_14241_amd import hmc
n = {n}
perm = np.array([hmc.test_fft_freq(n, p) for p in range(0, n, {step})])
assert len(set(perm.tolist())) == len(perm) and perm.min() >= 0 and perm.max() < n
if n <= 2**17:
    x = np.random.default_rng(n).normal(size=n) + 0j
    y, ref = hmc.test_fft(x), np.fft.fft(x)
    assert np.abs(y[::{step}] - ref[perm]).max() <= 1e-12 * np.abs(ref).max()
"""


@pytest.mark.parametrize("n", [2**16, 3 * 5 * 7 * 2**10, 2**17, 2**18, 2**19, 2**20, 2**21, 2**18 * 7])
def test_long_plans(n):
    r = subprocess.run([sys.executable, "-c", CODE.format(root=ROOT, n=n, step=max(1, n // 4096))],
                       capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr[-500:])
