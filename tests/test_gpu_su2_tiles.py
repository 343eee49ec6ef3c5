"""SU(2) passes over the tile shapes: whole rows, halves and thirds of a row, a tile
of one row, tiles that leave part of their threads or of the XCD bands empty, and
odd sizes, against the oracle (float64 parity bound 1e-12 relative).  A drift angle
beyond the polynomial range of the link exponential is included."""
import math

import pytest

from gpu_util import rel_maxdiff, say, tile_env, to_dev
from paper_2102_01031_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,tile,e_amp", [(2, None, 0.3), (7, None, 0.3), (24, None, 0.3), (33, "17", 0.3), (40, None, 0.3),
                                          (50, "25", 0.3), (96, None, 0.3), (12, None, 400.0)])
@pytest.mark.parametrize("integ,exp,steps", [("lf", "none", 4), ("lf", "self", 2), ("vv2", "self", 1), ("vv2", "fixed", 1)])
def test_su2_tiles_parity(N, tile, e_amp, integ, exp, steps):
    import oracle
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    if N == 96 and exp != "self":
        steps = 1
    phi, pi, U, E = inputs.random_su2_state(N, 11 + N, e_amp=e_amp)
    kw = dict(dx=0.4, dt=0.02, lam=1.0, v=1.0, g=0.5)
    bg = dict(none={}, fixed=dict(H0=0.2, w_eos=1 / 3), self=dict(kappa2=1e-4))[exp]
    say(f"N={N} tile={tile} e_amp={e_amp} {integ} {exp}")
    m = oracle.SU2Model(N=N, expansion=dict(none=oracle.NONE, fixed=oracle.FIXED, self=oracle.SELF)[exp], **kw, **bg)
    st = oracle.SU2State(m, phi, pi, U, E)
    st = st.run(steps) if integ == "lf" else st.run_vv(steps, 2)
    d = [to_dev(v, torch.float64) for v in (phi, pi, U, E)]
    with tile_env(tile, "LATTICE_SU2_TILE"):
        lat = Lattice(doublet=d[0], pi_doublet=d[1], U=d[2], E=d[3], N=N, integrator=integ, expansion=exp,
                      potential="su2_higgs", **kw, **bg)
    lat.step(steps)
    for got, ref in zip(d, (st.phi, st.pi, st.U, st.E)):
        scale = max(abs(r).max() for r in ref)
        for g, r in zip(got, ref):
            assert abs(g.cpu().numpy() - r).max() <= 1e-12 * scale
    e, o = lat.energy(), st.energy()
    for k in ("rho", "a", "b"):
        assert math.isclose(e[k], o[k], rel_tol=1e-12, abs_tol=1e-300), (k, e[k], o[k])
    lat.close()
