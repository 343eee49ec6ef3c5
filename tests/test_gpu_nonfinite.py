"""Infinities and NaN in a field or momentum come out where the site's stencil carries them:
the one-site-per-thread, plane-run and two-passes kernels against the tiled kernel, the U(1)
row-sharing kernel against the one for any size, the SU(2) passes against the oracle, and
the spectra's counts and sums.  The finite sites agree as they do without them."""
import numpy as np
import pytest

from gpu_util import say, tile_env, to_dev

pytestmark = pytest.mark.gpu

BAD = [float("nan"), float("inf"), -float("inf")]


def _same(a, b, tol):
    import torch
    for x, y in zip(a, b):
        assert torch.equal(torch.isnan(x), torch.isnan(y))
        assert torch.equal(torch.isinf(x), torch.isinf(y))
        k = torch.isfinite(y)
        assert torch.equal(x[~k & ~torch.isnan(y)], y[~k & ~torch.isnan(y)])
        if k.any():
            assert (x[k].double() - y[k].double()).abs().max() <= tol * y[k].double().abs().max()


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("where", ["field", "momentum"])
@pytest.mark.parametrize("nf,prec", [(1, "f64"), (2, "f64"), (2, "f32")])
@pytest.mark.parametrize("integ,exp", [("lf", "fixed"), ("vv2", "none"), ("vv2", "self")])
def test_scalar(bad, where, nf, prec, integ, exp):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    N = 18
    dt = torch.float64 if prec == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N)
    init = [torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64).mul(0.1).to(dt) for _ in range(2 * nf)]
    init[nf - 1 if where == "field" else nf][N ** 3 - 1 if nf == 2 else N * N * 7 + N * 3] = bad
    xs = {(1, "f64"): 6, (2, "f64"): 3, (2, "f32"): 6}[nf, prec]
    specs = [("8,8", None), ("site,1,1", None), ("plane", None)]
    if exp != "self":
        specs += [(None, str(xs))]
    res = []
    for tile, pair in specs:
        say(f"{bad} {where} nf={nf} {prec} {integ} {exp} {tile} {pair}")
        f = [x.clone() for x in init]
        with tile_env(tile), tile_env(pair, "LATTICE_PAIR"), tile_env("0", "LATTICE_SLAB"):
            lat = Lattice(f[:nf], f[nf:], N=N, dx=0.3, dt=0.005, integrator=integ, expansion=exp, q=10.0,
                          potential="phi4" if nf == 1 else "phi4_chi2", precision=prec,
                          **dict(fixed=dict(H0=0.2), none={}, self=dict(kappa2=0.01, b0=0.1))[exp])
        lat.step(3)
        res.append((f, lat.energy()["rho"]))
        lat.close()
    for f, rho in res[1:]:
        _same(f, res[0][0], 1e-14 if prec == "f64" else 1e-6)
        assert not np.isfinite(rho) and np.isnan(rho) == np.isnan(res[0][1])


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("name", ["phi", "A", "piA"])
def test_u1(bad, name):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    N = 17
    g = torch.Generator(device="cuda").manual_seed(N)
    init = {k: [0.3 * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(n)]
            for k, n in (("phi", 2), ("pi", 2), ("A", 3), ("piA", 3))}
    init[name][1][N ** 3 - N] = bad
    res = []
    for spec in ("tile", None, "1,5"):
        say(f"{bad} {name} {spec}")
        f = {k: [x.clone() for x in v] for k, v in init.items()}
        with tile_env(spec, "LATTICE_U1_TILE"):
            lat = Lattice(f["phi"], f["pi"], A=f["A"], piA=f["piA"], N=N, dx=0.4, dt=0.02, integrator="lf",
                          potential="abelian_higgs", e=0.5, v=1.0, kappa_g=1.0)
        lat.step(2)
        res.append(([x for v in f.values() for x in v], lat.energy()["rho"]))
        lat.close()
    for f, rho in res[1:]:
        _same(f, res[0][0], 1e-13)
        assert not np.isfinite(rho) and np.isnan(rho) == np.isnan(res[0][1])


@pytest.mark.parametrize("bad", BAD + [0.0])
@pytest.mark.parametrize("name", ["E", "U"])
def test_su2(bad, name):
    """(0.0: an electric field of zero, whose link exponential is the identity)"""
    import oracle
    import torch

    from paper_2102_01031_amd import inputs
    from paper_2102_01031_amd.lattice import Lattice
    N = 9
    phi, pi, U, E = inputs.random_su2_state(N, 3, e_amp=0.3)
    for k in range(3):
        (E if name == "E" else U)[3 + k].reshape(-1)[N ** 3 - 2] = bad
    kw = dict(dx=0.4, dt=0.02, lam=1.0, v=1.0, g=0.5)
    say(f"{bad} {name}")
    st = oracle.SU2State(oracle.SU2Model(N=N, expansion=oracle.NONE, **kw), phi, pi, U, E).run(1)
    d = [to_dev(v, torch.float64) for v in (phi, pi, U, E)]
    lat = Lattice(doublet=d[0], pi_doublet=d[1], U=d[2], E=d[3], N=N, integrator="lf", potential="su2_higgs", **kw)
    lat.step(1)
    lat.close()
    for got, ref in zip(d, (st.phi, st.pi, st.U, st.E)):
        for x, r in zip(got, ref):
            x, r = x.cpu().numpy(), np.asarray(r).reshape(-1)
            assert np.array_equal(np.isfinite(x), np.isfinite(r))
            k = np.isfinite(r)
            assert np.max(np.abs(x[k] - r[k])) <= 1e-12 * np.max(np.abs(r[k]))


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("N", [8, 15, 22])
def test_spectra(bad, N):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    f = [torch.ones(N ** 3, dtype=torch.float64, device="cuda") for _ in range(2)]
    say(f"{bad} N={N}")
    lat = Lattice(f[:1], f[1:], N=N, dx=0.3, dt=0.005, integrator="vv2", potential="phi4")
    good = lat.spectrum(0, "phi")["count"]
    f[0][N ** 3 - 3] = bad
    s, o = lat.spectrum(0, "phi"), lat.occupation(0)
    assert not np.isfinite(s["sum"]).any() and not np.isfinite(o["n"][1:]).any()
    assert np.array_equal(s["count"], good) and np.array_equal(o["count"], good)
    assert np.isfinite(lat.spectrum(0, "pi")["sum"]).all()
    lat.close()
