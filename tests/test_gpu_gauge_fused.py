"""Self-consistent gauge steps whose drift takes the finish of the summing pass before it
(small lattices) against the same steps one call at a time, whose finishes run alone: the
sums are added in the same order and the update is the same, so the fields and the scale
factor agree to a few ulp (1e-13).  Sizes on both sides of the rule, lattices smaller than
a block and with a ragged last one, one to many records."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [3, 9, 24, 57])
@pytest.mark.parametrize("kind", ["u1", "su2"])
@pytest.mark.parametrize("integ,steps", [("lf", 4), ("vv2", 3), ("vv4", 1)])
def test_fused_finish_matches_single_calls(N, kind, integ, steps):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    g = torch.Generator(device="cuda").manual_seed(N)

    def rnd(n, s):
        return [s * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(n)]

    if kind == "u1":
        init = dict(phi=rnd(2, 0.3), pi=rnd(2, 0.2), A=rnd(3, 0.4), piA=rnd(3, 0.3))
        par = dict(potential="abelian_higgs", e=0.5, v=1.0, kappa_g=1.0)
    else:
        U = rnd(12, 1.0)
        for i in range(3):
            n = sum(u * u for u in U[4 * i:4 * i + 4]).sqrt()
            U[4 * i:4 * i + 4] = [u / n for u in U[4 * i:4 * i + 4]]
        init = dict(doublet=rnd(4, 0.3), pi_doublet=rnd(4, 0.2), U=U, E=rnd(9, 0.1))
        par = dict(potential="su2_higgs", g=0.5, v=1.0)
    res = []
    for calls in ([steps], [1] * steps):
        say(f"N={N} {kind} {integ} calls={calls}")
        f = {k: [x.clone() for x in v] for k, v in init.items()}
        if kind == "u1":
            lat = Lattice(f["phi"], f["pi"], A=f["A"], piA=f["piA"], N=N, dx=0.4, dt=0.02, integrator=integ,
                          expansion="self", kappa2=0.05, **par)
        else:
            lat = Lattice([], [], doublet=f["doublet"], pi_doublet=f["pi_doublet"], U=f["U"], E=f["E"], N=N, dx=0.4,
                          dt=0.02, integrator=integ, expansion="self", kappa2=0.05, **par)
        for n in calls:
            lat.step(n)
        e = lat.energy()
        res.append(([x.cpu().numpy() for v in f.values() for x in v], (e["a"], e["b"], e["rho"])))
        lat.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert np.max(np.abs(a - b)) <= 1e-13 * np.max(np.abs(b))
    assert np.allclose(res[0][1], res[1][1], rtol=1e-13, atol=0)
