"""Line transforms whose stages have more butterflies than a block threads (two LDS buffers
in turn: 150, 216, 243 odd and even numbers of stages, 384 near the LDS limit) or two prime
factors above 7 (121, 143: the general sum over a stage's roots), spectra, occupation numbers
and the spectrum-bin gradient.  Reference: the library transform of the same values in
float64.  A length-n transform's error is a few ulp times log2 n, n for a prime: 1e-13 of the
largest shell; 1e-12 for the numbers and gradients formed from them."""
import math

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _shells(N):
    import torch
    f = torch.fft.fftfreq(N, d=1.0 / N, device="cuda", dtype=torch.float64).round().long()
    m = f[:, None, None] ** 2 + f[None, :, None] ** 2 + f[None, None, :] ** 2
    b = m.double().sqrt().floor().long()
    b = torch.where((b + 1) ** 2 <= m, b + 1, b)
    return torch.where(b * b > m, b - 1, b).reshape(-1)


@pytest.mark.parametrize("N,prec", [(121, "f64"), (143, "f32"), (150, "f64"), (216, "f64"), (243, "f64"), (384, "f64")])
def test_sizes(N, prec):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    dt = torch.float64 if prec == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N)
    f = [torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64).to(dt) for _ in range(2)]
    shell, nb, H0 = _shells(N), int(math.isqrt(3 * (N // 2) ** 2)) + 1, 0.3
    say(f"N={N} {prec}")
    lat = Lattice(f[:1], f[1:], N=N, dx=0.3, dt=0.005, integrator="vv2", expansion="fixed", H0=H0, potential="phi4",
                  precision=prec)
    power = lambda x: torch.bincount(shell, minlength=nb, weights=torch.fft.fftn(
        x.double().reshape(N, N, N)).abs().square().reshape(-1)).cpu().numpy()
    cnt = torch.bincount(shell, minlength=nb).cpu().numpy()
    ref = [power(f[0]), power(f[1]), power(f[1].double() + H0 * f[0].double())]
    for arr, r in (("phi", ref[0]), ("pi", ref[1])):
        s = lat.spectrum(0, arr)
        assert np.array_equal(s["count"], cnt)
        assert np.max(np.abs(s["sum"] - r)) <= 1e-13 * r.max()
    o = lat.occupation(0)
    b = np.arange(1, nb)
    w = np.sqrt((2 * math.pi / (N * 0.3) * b) ** 2 + 3 * float(f[0].double().square().mean()))
    n = (N * 0.3) ** 3 / (2.0 * float(N) ** 6) * (w * ref[0][1:] + ref[2][1:] / w) / (4 * math.pi * b ** 2)
    assert np.array_equal(o["count"], cnt)
    assert np.max(np.abs(o["n"][1:] - n)) <= 1e-12 * n.max()
    lat.close()


@pytest.mark.parametrize("N", [121, 143, 150])
def test_shell_gradient(N):
    import torch

    from paper_2102_01031_amd import autograd
    from test_gpu_shell_gradient import DT, DX, LAM, Q, _observable
    rng = np.random.default_rng(N)
    host = [torch.tensor(s * rng.standard_normal((N, N, N))) for s in (0.5, 0.4, 0.3, 0.2)]
    top = int(math.isqrt(3 * (N // 2) ** 2))
    for b in (1, top // 2, top):
        say(f"N={N} bin={b}")
        ref_in = [h.clone().requires_grad_() for h in host] + [torch.tensor(Q, dtype=torch.float64, requires_grad=True)]
        ref = _observable(*ref_in, N, 0, b)
        rg = torch.autograd.grad(ref, ref_in, allow_unused=True)
        ins = [h.cuda().requires_grad_() for h in host] + [torch.tensor(Q, dtype=torch.float64, requires_grad=True)]
        O = autograd.spectrum_bin(*ins, field=0, bin=b, N=N, dx=DX, dt=DT, nsteps=1, lam=LAM)
        got = torch.autograd.grad(O, ins)
        assert abs(O.item() - ref.item()) <= 1e-12 * abs(ref.item())
        for x, r in zip(got, rg):
            r = torch.zeros_like(x.cpu()) if r is None else r
            assert (x.cpu() - r).abs().max() <= 1e-12 * r.abs().max()
