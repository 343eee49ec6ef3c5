"""Calls of odd and even numbers of passes end in the caller's arrays, whichever
buffers the passes in between write: every schedule, with the whole-row, the
plane-run and the tiled kernel, against the oracle (float64 parity bound 1e-12),
and the copy back for arrays that are aligned to their element size only."""
import pytest

from gpu_util import compare_energy, compare_state, gpu_scalar, oracle_model, say, scalar_kwargs, tile_env
from paper_2102_01031_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,spec", [(64, None), (20, None), (20, "8,8")])
@pytest.mark.parametrize("integ,exp", [("lf", "self"), ("lf", "fixed"), ("vv2", "none"), ("vv2", "self"),
                                       ("vv4", "fixed"), ("vv4", "self")])
def test_odd_and_even_calls(N, spec, integ, exp):
    import oracle
    wl = workloads.PREHEAT_128
    kw = scalar_kwargs(wl, N=N, integrator=integ, expansion=exp)
    phi, pi = wl.initial_fields(N=N)
    for calls in ([1], [2, 1], [3, 2]):
        say(f"N={N} {spec} {integ} {exp} calls {calls}")
        st = oracle.ScalarState(oracle_model(kw), phi, pi)
        for n in calls:
            st.run(n)
        with tile_env(spec), tile_env("0", "LATTICE_SLAB"):
            lat, tp, tq = gpu_scalar(kw, phi, pi, calls)
        compare_state(tp, tq, st, 1e-12, f"{calls}")
        compare_energy(lat.energy(), st.energy(), 1e-12)
        lat.close()


@pytest.mark.parametrize("N,shift", [(5, 1), (16, 3), (16, 0)])
def test_copy_back_of_element_aligned_arrays(N, shift):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    g = torch.Generator().manual_seed(3)
    init = [torch.randn(N ** 3, generator=g, dtype=torch.float64).float() for _ in range(2)]
    out = []
    for s in (shift, 0):
        flat = [torch.zeros(N ** 3 + 8, dtype=torch.float32, device="cuda") for _ in range(2)]
        f = [t[s:s + N ** 3] for t in flat]
        for a, b in zip(f, init):
            a.copy_(b)
        lat = Lattice(f[:1], f[1:], N=N, dx=0.5, dt=0.01, integrator="lf", potential="phi4", precision="f32")
        lat.step(1)
        torch.cuda.synchronize()
        out.append([t.cpu().clone() for t in f])
        for t in flat:   # nothing beside the arrays is written
            assert float(t[:s].abs().sum() + t[s + N ** 3:].abs().sum()) == 0.0
        lat.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
