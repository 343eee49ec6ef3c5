"""Occupation numbers where one of field and momentum is eight orders smaller and its modes
lie apart: the large array holds shells |n| < 3, the small one white noise, and the shells
above see the small one alone.  Reference: numpy's transform of each array by itself.
A separate transform leaves 2e-16 of the large array's rows, which adds 4e-14 of the small
array's power in these shells (a numpy model of the packings, N = 32 and 64); with both arrays
in one complex line it is 1e-10 to 1e-9.  Bound: 1e-12 of each shell."""
import math

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [22, 32, 45, 64])
@pytest.mark.parametrize("small", ["pi", "phi"])
def test_small_array_beside_a_large_one(N, small):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    rng = np.random.default_rng(N)
    f = np.fft.fftfreq(N, d=1.0 / N)
    m = np.rint(f[:, None, None] ** 2 + f[None, :, None] ** 2 + f[None, None, :] ** 2).astype(int)
    big = np.fft.ifftn(np.fft.fftn(rng.standard_normal((N, N, N))) * (m < 9)).real
    host = dict(phi=big / big.std(), pi=1e-8 * rng.standard_normal((N, N, N)))
    if small == "phi":
        host = dict(phi=host["pi"], pi=host["phi"])
    d = {k: torch.tensor(v.reshape(-1)).cuda() for k, v in host.items()}
    say(f"N={N} small {small}")
    lat = Lattice([d["phi"]], [d["pi"]], N=N, dx=0.3, dt=0.005, integrator="vv2", potential="phi4")
    n = lat.occupation(0)["n"]
    lat.close()
    b = np.arange(5, N // 2)
    bins = lambda x: np.array([(np.abs(np.fft.fftn(x)) ** 2)[(m >= s * s) & (m < (s + 1) ** 2)].sum() for s in b])
    om = np.sqrt((2 * math.pi / (N * 0.3) * b) ** 2 + 3 * np.mean(host["phi"] ** 2))
    ref = (N * 0.3) ** 3 / (2.0 * N ** 6) * (om * bins(host["phi"]) + bins(host["pi"]) / om) / (4 * math.pi * b ** 2)
    assert np.max(np.abs(n[b] / ref - 1)) <= 1e-12
