"""The work array of a gradient over a kept trajectory: none for contexts that lattice_grad
refuses."""
import ctypes as C

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _lattice(N, integrator="vv2", potential="phi4_chi2", precision="f64", seed=1, scale=0.3, **kw):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    nf = 1 if potential == "phi4" else 2
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if precision == "f32" else torch.float64
    f = [(scale * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64)).to(dt) for _ in range(2 * nf)]
    return Lattice(f[:nf], f[nf:], N=N, dx=0.3, dt=0.005, integrator=integrator, potential=potential, q=1.0,
                   precision=precision, **kw), f


@pytest.mark.parametrize("over,takes", [({}, True), (dict(integrator="lf"), False), (dict(integrator="vv4"), False),
                                        (dict(potential="phi4"), False), (dict(precision="f32"), False)])
def test_no_work_where_the_gradient_is_refused(over, takes):
    import torch

    from paper_2102_01031_amd.lattice import LAT_EUNSUPPORTED, LatGradSpec, LatticeError, lib
    say(f"{over}")
    lat, _ = _lattice(16, **over)
    need = lib().lattice_grad_work(lat._ctx, C.byref(LatGradSpec(0, 0, 7, 0, 0, 0)))
    assert need == (8 * (8 + 2 * 7) * 16 ** 3 if takes else 0)
    if not takes:
        held = torch.cuda.memory_reserved()
        with pytest.raises(LatticeError) as e:
            lat.grad(20000, want_phi=False, want_pi=False)
        assert e.value.code == LAT_EUNSUPPORTED
        assert torch.cuda.memory_reserved() == held
    lat.close()
