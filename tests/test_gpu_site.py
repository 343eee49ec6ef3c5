"""GPU parity of the one-site-per-thread scalar kernel: the smallest lattices, sizes off
every tile, a last block that is nearly empty, one and several sites per thread, and each
kind of pass (kick and drift, kicks alone, the self-consistent drift on load, energies),
against the oracle (float64 parity bound 1e-12 relative); then the sizes where the launch
rule changes kernels, against the marching kernel."""
import numpy as np
import pytest

from gpu_util import compare_energy, gpu_scalar, oracle_model, rel_maxdiff, say, scalar_kwargs, tile_env
from paper_2102_01031_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,spec", [(2, "site,1,1"), (3, "site,1,1"), (7, "site,1,1,1"), (17, "site,1,1"),
                                    (33, "site,1,1,50"), (40, None)])
@pytest.mark.parametrize("wl,over", [(workloads.PREHEAT_128, dict(integrator="vv2", expansion="self")),
                                     (workloads.PREHEAT_128, dict(integrator="lf", expansion="self")),
                                     (workloads.PREHEAT_128, dict(integrator="vv2", expansion="none")),
                                     (workloads.LPHI4_32, {}),
                                     (workloads.LPHI4_32, dict(integrator="vv4", expansion="self"))])
def test_site_parity(N, spec, wl, over):
    import oracle
    steps = 3
    kw = scalar_kwargs(wl, N=N, **over)
    phi, pi = wl.initial_fields(N=N)
    st = oracle.ScalarState(oracle_model(kw), phi, pi).run(steps)
    say(f"N={N} {kw['integrator']} {kw['expansion']} {kw['potential']} {spec}")
    with tile_env(spec), tile_env("0", "LATTICE_SLAB"):
        lat, tp, tq = gpu_scalar(kw, phi, pi, [steps])
    e = lat.energy()
    for s in range(wl.nfields):
        assert rel_maxdiff(tp[s].cpu().numpy(), st.phi[s]) < 1e-12
        assert rel_maxdiff(tq[s].cpu().numpy(), st.pi[s]) < 1e-12
    lat.close()
    compare_energy(e, st.energy(), 1e-12)


@pytest.mark.parametrize("N", [63, 72, 73, 96, 110])
@pytest.mark.parametrize("nf,prec,integ,exp", [(2, "f64", "vv2", "self"), (2, "f32", "vv2", "self"),
                                               (1, "f32", "lf", "fixed"), (1, "f64", "vv4", "fixed")])
def test_site_rule_matches_marching(N, nf, prec, integ, exp):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    dt = torch.float64 if prec == "f64" else torch.float32
    tol = 1e-12 if prec == "f64" else 2e-6
    g = torch.Generator().manual_seed(N)
    init = [torch.randn(N ** 3, generator=g, dtype=torch.float64) for _ in range(2 * nf)]
    bg = dict(H0=0.2) if exp == "fixed" else {}
    res = []
    for spec in (None, "plane"):   # the plane-run kernel is held to the oracle by its own tests
        say(f"N={N} nf={nf} {prec} {integ} {exp} {spec}")
        f = [(0.1 * t + (1.0 if i == 0 else 0.0)).to(dt).cuda() for i, t in enumerate(init)]
        with tile_env(spec):
            lat = Lattice(f[:nf], f[nf:], N=N, dx=0.3, dt=0.005, integrator=integ, expansion=exp, q=100.0,
                          potential="phi4" if nf == 1 else "phi4_chi2", precision=prec, **bg)
        lat.step(2)
        res.append(([t.double().cpu().numpy() for t in f], lat.energy()["rho"]))
        lat.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))
    assert abs(res[0][1] / res[1][1] - 1) < (1e-12 if prec == "f64" else 1e-7)
