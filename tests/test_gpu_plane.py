"""GPU parity of the plane-run scalar kernel (any N): odd and ragged sizes on
either side of its launch shapes' edges, and cuts of the lattice that leave
partial runs and z chunks, against the oracle.  The tolerance is the float64
parity bound of the scalar passes (1e-12 relative); float32 fields take the
bound of the float32 path's parity test at these step counts."""
import pytest

from gpu_util import compare_energy, gpu_scalar, oracle_model, rel_maxdiff, say, scalar_kwargs, tile_env
from paper_2102_01031_amd import workloads

pytestmark = pytest.mark.gpu


def _run(N, wl, spec, steps, **over):
    import oracle
    kw = scalar_kwargs(wl, N=N, **over)
    phi, pi = wl.initial_fields(N=N)
    st = oracle.ScalarState(oracle_model(kw), phi, pi).run(steps)
    say(f"N={N} {kw['integrator']} {kw['expansion']} {kw.get('precision', 'f64')} {spec}")
    with tile_env(spec), tile_env("0", "LATTICE_SLAB"):
        lat, tp, tq = gpu_scalar(kw, phi, pi, [steps])
    e = lat.energy()
    got = [[t.cpu().numpy() for t in ts] for ts in (tp, tq)]
    lat.close()
    return got, e, st


# one site per run's thread, whole plane in one run, N across the halo and
# threads-per-block edges (64 | 65, 128 | 129), a prime
@pytest.mark.parametrize("N,spec", [(2, None), (3, "plane,2,3"), (5, "plane,2,25"), (17, None), (33, "plane,5,7"),
                                    (63, None), (65, None), (97, "plane,40,19"), (129, None), (136, "plane,136,37")])
@pytest.mark.parametrize("wl,over", [(workloads.PREHEAT_128, dict(integrator="vv2", expansion="self")),
                                     (workloads.LPHI4_32, {}),
                                     (workloads.LPHI4_32, dict(integrator="vv4", expansion="none"))])
def test_plane_parity(N, spec, wl, over):
    steps = 3
    got, e, st = _run(N, wl, spec, steps, **over)
    for s in range(wl.nfields):
        assert rel_maxdiff(got[0][s], st.phi[s]) < 1e-12 and rel_maxdiff(got[1][s], st.pi[s]) < 1e-12
    compare_energy(e, st.energy(), 1e-12)


# wider halos: more than one halo site per thread, in both precisions
@pytest.mark.parametrize("N,prec", [(258, "f64"), (257, "f32"), (96, "f32")])
def test_plane_wide_halo(N, prec):
    import numpy as np
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    dt = torch.float64 if prec == "f64" else torch.float32
    tol = 1e-12 if prec == "f64" else 2e-6
    g = torch.Generator().manual_seed(11)
    init = [torch.randn(N ** 3, generator=g, dtype=torch.float64) for _ in range(4)]
    res = []
    for spec in (None, "16,16"):   # the tiled kernel is held to the oracle by its own tests
        say(f"N={N} {prec} {spec}")
        f = [(0.1 * t + (1.0 if i == 0 else 0.0)).to(dt).cuda() for i, t in enumerate(init)]
        with tile_env(spec):
            lat = Lattice(f[:2], f[2:], N=N, dx=0.3, dt=0.005, integrator="vv2", expansion="self",
                          potential="phi4_chi2", q=100.0, precision=prec)
        lat.step(2)
        res.append(([t.double().cpu().numpy() for t in f], lat.energy()["rho"]))
        lat.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))
    assert abs(res[0][1] / res[1][1] - 1) < (1e-12 if prec == "f64" else 1e-7)
