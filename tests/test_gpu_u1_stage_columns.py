"""Summing passes of the U(1) kernel for any size in columns of z planes (one plane, columns
with a ragged last one, the whole height) against the oracle: the energies of a leapfrog
state (momenta kicked on the fly) and the self-consistent steps, whose kick-and-sums pass
is that energy pass and a kick."""
import math

import numpy as np
import pytest

from gpu_util import rel_maxdiff, say, tile_env, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [13, 20])
@pytest.mark.parametrize("zc", ["1", "5", "13"])
@pytest.mark.parametrize("exp", ["none", "self"])
def test_columns(N, zc, exp):
    import oracle
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    rng = np.random.default_rng(N)
    f = {k: [s * rng.standard_normal((N, N, N)) for _ in range(n)]
         for k, n, s in (("phi", 2, 0.3), ("pi", 2, 0.2), ("A", 3, 0.4), ("piA", 3, 0.3))}
    kw = dict(dx=0.4, dt=0.02, lam=1.0, v=1.0, e=0.5, kappa_g=1.0)
    bg = dict(none={}, self=dict(kappa2=0.05))[exp]
    say(f"N={N} zc={zc} {exp}")
    m = oracle.U1Model(N=N, expansion=oracle.NONE if exp == "none" else oracle.SELF, **kw, **bg)
    st = oracle.U1State(m, f["phi"], f["pi"], f["A"], f["piA"]).run(2)
    d = {k: to_dev(v, torch.float64) for k, v in f.items()}
    with tile_env("tile", "LATTICE_U1_TILE"), tile_env(zc, "LATTICE_U1_ENERGY_ZC"):
        lat = Lattice(d["phi"], d["pi"], A=d["A"], piA=d["piA"], N=N, integrator="lf", expansion=exp,
                      potential="abelian_higgs", **kw, **bg)
    lat.step(2)
    e, o = lat.energy(), st.energy()
    lat.close()
    for k, ref in (("phi", st.phi), ("pi", st.pi), ("A", st.A), ("piA", st.piA)):
        for x, r in zip(d[k], ref):
            assert rel_maxdiff(x.cpu().numpy(), r) <= 1e-12, k
    for k in ("rho", "a", "b", "EK_A", "EG_A", "gauss_max", "gauss_mean"):
        assert math.isclose(e[k], o[k], rel_tol=1e-12, abs_tol=1e-300), k
