"""Gradients over a kept trajectory (stride 0) against those over checkpoints (strides 1
and 3), which are held to the oracle by their own tests: one step, an even and an odd
number, lattices that fill less than a block and leave a ragged last one, every
background, both observables, called twice, with the caller's arrays bitwise untouched and
the context fit to go on stepping.  The checkpoint path rebuilds the states backward, seven
steps of a few ulp each: 1e-11 of an array's largest entry, 1e-10 of a scalar."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,T", [(5, 1), (16, 7), (33, 2), (64, 7), (73, 3)])
@pytest.mark.parametrize("exp", ["none", "fixed", "self"])
@pytest.mark.parametrize("obs,sel", [("energy_fraction", dict(field=0)), ("spectrum_bin", dict(field=1, bin=2))])
def test_kept_trajectory_matches_checkpoints(N, T, exp, obs, sel):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    g = torch.Generator(device="cuda").manual_seed(N)
    init = [0.3 * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(4)]
    bg = dict(none={}, fixed=dict(H0=0.1, w_eos=1 / 3), self=dict(kappa2=0.01))[exp]
    res = []
    for stride in (0, 1, 3):
        say(f"N={N} T={T} {exp} {obs} stride={stride}")
        f = [x.clone() for x in init]
        lat = Lattice(f[:2], f[2:], N=N, dx=0.3, dt=0.005, integrator="vv2", potential="phi4_chi2", q=10.0,
                      expansion=exp, **bg)
        for _ in range(2):
            r = lat.grad(T, stride=stride, observable=obs, **sel)
            assert all(torch.equal(a, b) for a, b in zip(f, init))
        lat.step(2)
        res.append((r, lat.energy()["rho"]))
        lat.close()
    r0, rho0 = res[0]
    for r, rho in res[1:]:
        for k in ("dO_dphi", "dO_dpi"):
            for a, b in zip(r0[k], r[k]):
                assert (a - b).abs().max() <= 1e-11 * b.abs().max()
        for k in ("value", "dO_dq", "dO_da0", "dO_db0"):
            assert abs(r0[k] - r[k]) <= 1e-10 * abs(r[k]) + 1e-16, k
        assert abs(rho / rho0 - 1) < 1e-13
