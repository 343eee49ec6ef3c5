"""Two passes per launch against single passes (which are held to the oracle by their own
tests), the same expressions per site: bitwise in the fields of a leapfrog, to a few ulp
where compilers may contract the second half kick differently (1e-14 of the largest entry
in float64, 1e-6 in float32).  Smallest lattices, a run that ends inside a row, a last run
and z chunk that are nearly empty, one z plane per block, more outer neighbours than
threads, every remainder of the passes modulo four, and each integrator's closing kick."""
import numpy as np
import pytest

from gpu_util import say, tile_env

pytestmark = pytest.mark.gpu

XS = {(1, "f64"): (6, 8), (1, "f32"): (8, 12), (2, "f64"): (3, 4), (2, "f32"): (6,)}


@pytest.mark.parametrize("N,cut", [(16, ""), (17, ",1,3"), (33, ",5,7"), (65, ",13,64"), (100, ""), (264, ",88,60")])
@pytest.mark.parametrize("nf,prec", [(1, "f64"), (2, "f64"), (1, "f32"), (2, "f32")])
def test_pair_matches_single_passes(N, cut, nf, prec):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    dt = torch.float64 if prec == "f64" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(N)
    init = [torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(2 * nf)]
    runs = [("lf", "fixed", n) for n in (3, 4, 6, 7, 9)] + [("vv2", "none", n) for n in (2, 3, 4, 5)] + [("vv4", "fixed", 1)]
    if N > 200:
        runs = [("lf", "fixed", 4), ("vv4", "fixed", 1)]
    for integ, exp, steps in runs:
        res = []
        for spec in ["0"] + [f"{xs}{cut}" for xs in XS[nf, prec]]:
            say(f"N={N} nf={nf} {prec} {integ} {exp} steps={steps} LATTICE_PAIR={spec}")
            f = [(0.1 * t + (1.0 if i == 0 else 0.0)).to(dt) for i, t in enumerate(init)]
            with tile_env(spec, "LATTICE_PAIR"), tile_env("0", "LATTICE_SLAB"):
                lat = Lattice(f[:nf], f[nf:], N=N, dx=0.3, dt=0.005, integrator=integ, expansion=exp, q=10.0,
                              potential="phi4" if nf == 1 else "phi4_chi2", precision=prec,
                              **(dict(H0=0.2) if exp == "fixed" else {}))
            for n in (steps, -steps):
                lat.step(n)
                lat.sync()
            res.append([t.double().cpu().numpy() for t in f])
            lat.close()
        tol = 1e-14 if prec == "f64" else 1e-6
        for r in res[1:]:
            for a, b in zip(r, res[0]):
                assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))
