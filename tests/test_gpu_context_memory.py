"""Device memory of small contexts: the shadows or records and scratch of their own size.
The driver accounts it in 2 MB pieces, 21 KB of each of 100 contexts."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


def _per_context(n, make):
    import torch
    make()[0].close()   # what a process allocates once
    torch.cuda.synchronize()
    free, held = torch.cuda.mem_get_info()[0], torch.cuda.memory_reserved()
    made = [make() for _ in range(n)]
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - held)
    for lat, _ in made:
        lat.close()
    return used / n


@pytest.mark.parametrize("batch", [False, True])
def test_scalar(batch):
    """Two shadows of 4 KB (a batch: three) and a few small records, at most 4 KB each; block
    sums of 768 blocks took 97 KB."""
    import torch

    from paper_2102_01031_amd.lattice import Lattice, LatticeBatch
    kw = dict(dx=0.5, dt=0.01, integrator="lf", potential="phi4")
    zeros = lambda: torch.zeros(512, dtype=torch.float64, device="cuda")

    def one():
        f = [zeros(), zeros()]
        return Lattice(f[:1], f[1:], N=8, **kw), f

    def many():
        f = [[zeros() for _ in range(500)] for _ in range(2)]
        return LatticeBatch(*f, [8] * 500, autotune=False, **kw), f

    say(f"batch={batch}")
    used = _per_context(2, many) / 500 if batch else _per_context(500, one)
    assert used <= 64e3, used


def test_su2():
    """Two record buffers of 512 KB; block sums of thin tiles took 87 KB."""
    import torch

    from paper_2102_01031_amd.lattice import Lattice
    V = 16 ** 3
    ones, z = torch.ones(V, dtype=torch.float64, device="cuda"), torch.zeros(V, dtype=torch.float64, device="cuda")

    def one():
        f = dict(doublet=[z] * 4, pi_doublet=[z] * 4, U=[ones, z, z, z] * 3, E=[z] * 9)
        return Lattice(N=16, dx=0.4, dt=0.02, integrator="lf", potential="su2_higgs", g=0.5, **f), f

    say("su2")
    used = _per_context(100, one)
    assert used <= 2 ** 20 + 64e3, used
