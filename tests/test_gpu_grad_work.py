"""The work array of a gradient over a kept trajectory: none for contexts that lattice_grad
refuses, and no other memory of the context that grows with it."""
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


def test_long_self_consistent_trajectory_keeps_its_tables_small():
    """A sweep of T steps runs in calls of at most 1024, so beside the trajectory (torch's) the
    context's memory grows by 16 bytes a step, the scale factors: 4 MB from 50000 to 300000
    steps, and as the driver hands memory out in 2 MB pieces at most one more for each of the
    four arrays that a gradient may enlarge; one call's coefficient table adds 24 MB."""
    import torch
    own = []
    for T in (8, 50000, 300000):   # the first for what a process allocates once
        say(f"N=2 T={T}")
        lat, _ = _lattice(2, expansion="self", kappa2=0.01, scale=0.05)
        torch.cuda.synchronize()
        free, held = torch.cuda.mem_get_info()[0], torch.cuda.memory_reserved()
        lat.grad(T)
        own.append(free - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - held))
        lat.close()
    assert own[2] - own[1] <= 4e6 + 4 * 2.1e6


@pytest.mark.parametrize("T", [1024, 1025, 2100])
def test_kept_trajectory_across_calls(T):
    """The calls' boundaries against the checkpointed sweep: rounding of a few ulp per step,
    2e-16 T, carried through up to ten units of time of weakly coupled fields (a factor of
    the order of 100): 1e-10 of an array's largest entry, 1e-9 of a scalar."""
    res = []
    for stride in (0, 50):
        say(f"T={T} stride={stride}")
        lat, _ = _lattice(6, expansion="self", kappa2=0.01, scale=0.05)
        res.append(lat.grad(T, stride=stride))
        lat.close()
    r0, r = res
    for k in ("dO_dphi", "dO_dpi"):
        for a, b in zip(r0[k], r[k]):
            assert (a - b).abs().max() <= 1e-10 * b.abs().max()
    for k in ("value", "dO_dq", "dO_da0", "dO_db0"):
        assert abs(r0[k] - r[k]) <= 1e-9 * abs(r[k]) + 1e-16, k
