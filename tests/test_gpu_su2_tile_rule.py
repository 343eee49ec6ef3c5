"""SU(2) tiles on both sides of the lines of their rule (whole rows against halves at 43 and
44, five rows of a whole-row tile up to 51) against tiles of 16 sites a row: the same site
terms, sums in another order (1e-13)."""
import math

import pytest

from gpu_util import say, tile_env, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [38, 43, 44, 51, 52])
@pytest.mark.parametrize("integ,exp", [("lf", "none"), ("vv2", "fixed"), ("lf", "self")])
def test_tile_rule(N, integ, exp):
    import torch

    from paper_2102_01031_amd import inputs
    from paper_2102_01031_amd.lattice import Lattice
    bg = dict(none={}, fixed=dict(H0=0.2, w_eos=1 / 3), self=dict(kappa2=1e-4))[exp]
    state = inputs.random_su2_state(N, N, e_amp=0.3)
    res = []
    for tile in (None, "16"):
        say(f"N={N} {integ} {exp} {tile}")
        d = [to_dev(v, torch.float64) for v in state]
        with tile_env(tile, "LATTICE_SU2_TILE"):
            lat = Lattice(doublet=d[0], pi_doublet=d[1], U=d[2], E=d[3], N=N, dx=0.4, dt=0.02, lam=1.0, v=1.0, g=0.5,
                          integrator=integ, expansion=exp, potential="su2_higgs", **bg)
        lat.step(2)
        res.append(([x for v in d for x in v], lat.energy()["rho"]))
        lat.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert (a - b).abs().max() <= 1e-13 * b.abs().max()
    assert math.isclose(res[0][1], res[1][1], rel_tol=1e-13)
