"""The U(1) row-sharing kernel with one row per block, two halo cells per thread, by its own
choice and forced, with z chunks that do not divide N and more than one halo-row operation
per thread, in every mode, against the oracle (float64 parity bound 1e-12 relative); and at
the upper end of its range against the kernel that serves any size."""
import math

import numpy as np
import pytest

from gpu_util import rel_maxdiff, say, tile_env, to_dev

pytestmark = pytest.mark.gpu

KW = dict(dx=0.4, dt=0.02, lam=1.0, v=1.0, e=0.5, kappa_g=1.0)


@pytest.mark.parametrize("N,spec", [(33, None), (34, "1,34"), (35, None), (40, "1,7"), (63, "1,5"), (66, "1,66"),
                                    (90, "1,13"), (24, "2,5"), (47, "5,9"), (50, "10,3")])
@pytest.mark.parametrize("integ,exp,steps", [("lf", "none", 3), ("lf", "self", 2), ("vv2", "fixed", 1), ("vv4", "self", 1)])
def test_parity(N, spec, integ, exp, steps):
    import oracle
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    rng = np.random.default_rng(11 * N)
    f = {k: [s * rng.standard_normal((N, N, N)) for _ in range(n)]
         for k, n, s in (("phi", 2, 0.3), ("pi", 2, 0.2), ("A", 3, 0.4), ("piA", 3, 0.3))}
    bg = dict(none={}, fixed=dict(H0=0.2, w_eos=1 / 3), self=dict(kappa2=0.05))[exp]
    say(f"N={N} {spec} {integ} {exp}")
    E = dict(none=oracle.NONE, fixed=oracle.FIXED, self=oracle.SELF)[exp]
    st = oracle.U1State(oracle.U1Model(N=N, expansion=E, **KW, **bg), f["phi"], f["pi"], f["A"], f["piA"])
    st = st.run(steps) if integ == "lf" else st.run_vv(steps, {"vv2": 2, "vv4": 4}[integ])
    d = {k: to_dev(v, torch.float64) for k, v in f.items()}
    with tile_env(spec, "LATTICE_U1_TILE"):
        lat = Lattice(d["phi"], d["pi"], A=d["A"], piA=d["piA"], N=N, integrator=integ, expansion=exp,
                      potential="abelian_higgs", **KW, **bg)
    lat.step(steps)
    e, o = lat.energy(), st.energy()
    for k, ref in (("phi", st.phi), ("pi", st.pi), ("A", st.A), ("piA", st.piA)):
        for g, r in zip(d[k], ref):
            assert rel_maxdiff(g.cpu().numpy(), r) <= 1e-12, k
    for k in ("rho", "a", "b", "gauss_max", "gauss_mean"):
        assert math.isclose(e[k], o[k], rel_tol=1e-12, abs_tol=1e-300), (k, e[k], o[k])
    lat.sync()
    st.sync()
    for g, r in zip(d["pi"] + d["piA"], list(st.pi) + list(st.piA)):
        assert rel_maxdiff(g.cpu().numpy(), r) <= 1e-12
    lat.close()


@pytest.mark.parametrize("N", [257, 500])
def test_large(N):
    """One step and the energies; the sums of 1e8 terms in another order: 1e-12."""
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    res = []
    for spec in (None, "tile"):
        say(f"N={N} {spec}")
        g = torch.Generator(device="cuda").manual_seed(N)
        f = [0.3 * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(10)]
        with tile_env(spec, "LATTICE_U1_TILE"):
            lat = Lattice(f[:2], f[2:4], A=f[4:7], piA=f[7:], N=N, integrator="lf", potential="abelian_higgs", **KW)
        lat.step(1)
        e = lat.energy()
        lat.close()
        res.append((f, e))
    (f, e), (h, o) = res
    for a, b in zip(f, h):
        assert (a - b).abs().max() <= 1e-12 * b.abs().max()
    for k in ("rho", "EK_A", "EG_A", "gauss_max", "gauss_mean"):
        assert math.isclose(e[k], o[k], rel_tol=1e-12), k
