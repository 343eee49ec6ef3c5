"""Spectra and occupation numbers of random fields over the transform sizes:
every radix (8, 4, 2, 3, 5, 7) alone and mixed, odd sizes (an odd number of rows
to pair), the smallest, primes above 7, a size left to the library transform, and
a number of bins below the mode range.  Reference: numpy's transform of the same
values in float64.  A length-n transform's error is a few ulp times log2 n, so
shell sums are held to 1e-13 of the largest shell."""
import math

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _shells(N):
    f = np.fft.fftfreq(N, d=1.0 / N).astype(int)
    m = f[:, None, None] ** 2 + f[None, :, None] ** 2 + f[None, None, :] ** 2
    b = np.floor(np.sqrt(m)).astype(int)
    b = np.where((b + 1) ** 2 <= m, b + 1, b)
    return np.where(b * b > m, b - 1, b).reshape(-1)


@pytest.mark.parametrize("N,prec", [(2, "f64"), (3, "f64"), (5, "f64"), (7, "f64"), (8, "f64"), (15, "f64"),
                                    (28, "f32"), (42, "f64"), (64, "f64"), (81, "f64"), (22, "f64"), (11, "f32"),
                                    (128, "f64")])
def test_sizes(N, prec):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    dt = torch.float64 if prec == "f64" else torch.float32
    rng = np.random.default_rng(N)
    host = [rng.standard_normal((N, N, N)) for _ in range(4)]
    dev = [torch.tensor(h.reshape(-1)).to(dt).cuda() for h in host]
    host = [t.double().cpu().numpy().reshape(N, N, N) for t in dev]
    H0 = 0.3
    lat = Lattice(dev[:2], dev[2:], N=N, dx=0.3, dt=0.005, integrator="vv2", expansion="fixed", H0=H0,
                  potential="phi4_chi2", q=10.0, precision=prec)
    shell = _shells(N)
    full = int(math.isqrt(3 * (N // 2) ** 2)) + 1
    for nb in {full, max(1, full // 2)}:
        say(f"N={N} {prec} nbins={nb}")
        cnt = np.bincount(shell, minlength=nb)[:nb]
        for field in (0, 1):
            ref = [np.bincount(shell, weights=(np.abs(np.fft.fftn(x)) ** 2).reshape(-1), minlength=nb)[:nb]
                   for x in (host[field], host[2 + field], host[2 + field] + H0 * host[field])]
            for arr, r in (("phi", ref[0]), ("pi", ref[1])):
                s = lat.spectrum(field, arr, nbins=nb)
                assert np.array_equal(s["count"], cnt)
                assert np.max(np.abs(s["sum"] - r)) <= 1e-13 * r.max()
            o = lat.occupation(field, nbins=nb)
            assert np.array_equal(o["count"], cnt)
            b = np.arange(1, nb)
            vpp = (3 * np.mean(host[0] ** 2) + 10.0 * np.mean(host[1] ** 2)) if field == 0 \
                else 10.0 * np.mean(host[0] ** 2)
            w = np.sqrt((2 * math.pi / (N * 0.3) * b) ** 2 + vpp)
            n = (N * 0.3) ** 3 / (2.0 * N ** 6) * (w * ref[0][1:] + ref[2][1:] / w) / (4 * math.pi * b ** 2)
            if nb > 1:
                assert np.max(np.abs(o["n"][1:] - n)) <= 1e-12 * n.max()
    lat.close()


def test_library_size():
    """257 times its largest prime, itself, lies beyond the line transforms' rule."""
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    N, nb = 257, 40
    rng = np.random.default_rng(N)
    phi = rng.standard_normal((N, N, N))
    dev = [torch.tensor(a.reshape(-1)).cuda() for a in (phi, np.zeros_like(phi))]
    say(f"N={N} library transform")
    lat = Lattice(dev[:1], dev[1:], N=N, dx=0.3, dt=0.005, potential="phi4")
    s = lat.spectrum(0, "phi", nbins=nb)
    lat.close()
    shell, w = _shells(N), (np.abs(np.fft.fftn(phi)) ** 2).reshape(-1)
    assert np.array_equal(s["count"], np.bincount(shell, minlength=nb)[:nb])
    ref = np.bincount(shell, weights=w, minlength=nb)[:nb]
    assert np.max(np.abs(s["sum"] - ref)) <= 1e-13 * ref.max()
