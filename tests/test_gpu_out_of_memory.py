"""Calls that find no device memory: what torch's allocator holds unused goes back to the
driver and the call is made again, a gradient without its trajectory; the state is what
it was.  The want of memory is put in by a stand-in for the library that answers
LAT_ENOMEM, as the library does before it has launched anything."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


class Library:
    """The library, except that call number `at` (from 1) of `name` finds no memory."""

    def __init__(self, real, name, at=1):
        self.real, self.name, self.left = real, name, at

    def __getattr__(self, k):
        fn = getattr(self.real, k)
        if k != self.name:
            return fn

        def call(*args):
            self.left -= 1
            return -6 if self.left == 0 else fn(*args)
        return call


def _lattice(N=16, **kw):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    g = torch.Generator(device="cuda").manual_seed(5)
    f = [0.3 * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(4)]
    return Lattice(f[:2], f[2:], N=N, dx=0.3, dt=0.005, integrator="vv2", potential="phi4_chi2", q=1.0, **kw), f


def _batch():
    import torch

    from paper_2102_01031_amd.lattice import LatticeBatch
    f = [[torch.ones(512, dtype=torch.float64, device="cuda")] for _ in range(2)]
    return LatticeBatch(*f, [8], autotune=False, dx=0.5, dt=0.01, integrator="lf", potential="phi4"), f


@pytest.mark.parametrize("name,use", [
    ("lattice_init", lambda: _lattice()[0].energy()["rho"]),
    ("lattice_init_batch", lambda: _batch()[0].energy(0)["rho"]),
    ("lattice_spectrum", lambda: float(_lattice()[0].spectrum(0)["sum"][3])),
    ("lattice_occupation", lambda: float(_lattice()[0].occupation(0)["n"][3])),
    ("lattice_grad_in", lambda: _lattice()[0].grad(5, stride=2)["value"]),
])
def test_call_is_made_again(monkeypatch, name, use):
    import torch

    from paper_2102_01031_amd import lattice
    ref = use()
    torch.empty(256 << 20, dtype=torch.uint8, device="cuda")   # held by torch's allocator, unused
    held = torch.cuda.memory_reserved()
    real = lattice.lib()
    monkeypatch.setattr(lattice, "lib", lambda fake=Library(real, name): fake)
    say(name)
    got = use()
    assert abs(got / ref - 1) <= 1e-13   # (bin sums may differ in the last bits)
    assert torch.cuda.memory_reserved() <= held - (256 << 20)


@pytest.mark.parametrize("exp", ["none", "self"])
@pytest.mark.parametrize("obs,sel", [("energy_fraction", dict(field=0)), ("spectrum_bin", dict(field=1, bin=2))])
def test_gradient_without_its_trajectory(monkeypatch, exp, obs, sel):
    import torch

    from paper_2102_01031_amd import lattice
    kw = dict(expansion=exp, **(dict(kappa2=0.01) if exp == "self" else {}))
    ref = _lattice(**kw)[0].grad(7, stride=3, observable=obs, **sel)
    lat, f = _lattice(**kw)
    init = [x.clone() for x in f]
    real = lattice.lib()
    monkeypatch.setattr(lattice, "lib", lambda fake=Library(real, "lattice_grad_in"): fake)
    say(f"{exp} {obs}")
    r = lat.grad(7, observable=obs, **sel)
    assert all(torch.equal(a, b) for a, b in zip(f, init))
    # the same sweep over checkpoints, with another stride: rounding of seven steps
    for a, b in zip(r["dO_dphi"] + r["dO_dpi"], ref["dO_dphi"] + ref["dO_dpi"]):
        assert (a - b).abs().max() <= 1e-11 * b.abs().max()
    assert abs(r["value"] / ref["value"] - 1) <= 1e-12
