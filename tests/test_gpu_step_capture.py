"""A caller's graph that holds lattice_step of a small lattice: the call keeps its coefficient
table there (calls of few launches pass them by value otherwise), and replays with eager
work and synchronisations between them equal the same eager steps bit for bit."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nf,integ,steps", [(16, 1, "lf", 3), (16, 1, "lf", 8), (24, 2, "vv2", 2), (40, 2, "lf", 5)])
def test_captured_step(N, nf, integ, steps):
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    g = torch.Generator(device="cuda").manual_seed(N)
    init = [0.1 * torch.randn(N ** 3, generator=g, device="cuda", dtype=torch.float64) for _ in range(2 * nf)]
    kw = dict(N=N, dx=0.3, dt=0.005, integrator=integ, potential="phi4" if nf == 1 else "phi4_chi2", q=10.0)
    f, h = [x.clone() for x in init], [x.clone() for x in init]
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    lat, ref = Lattice(f[:nf], f[nf:], stream=s, **kw), Lattice(h[:nf], h[nf:], **kw)
    lat.step(steps)
    ref.step(steps)
    torch.cuda.synchronize()
    say(f"N={N} nf={nf} {integ} steps={steps}")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        lat.step(steps)
    torch.cuda.synchronize()
    for k in range(4):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(steps)
        ref.energy()
        assert all(torch.equal(a, b) for a, b in zip(f, h)), k
    lat.close()
    ref.close()
