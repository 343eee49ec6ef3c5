"""lattice_grad_in takes all its memory before its first pass, so that a call that finds
none leaves the state and the clock as they were (the text of the function: every
allocation stands before the forward sweep)."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2102_01031_amd", "csrc",
                   "lattice.hip")


def test_gradient_allocates_before_its_sweep():
    body = open(SRC).read()
    body = body[body.index('extern "C" lat_status lattice_grad_in('):]
    body = body[:body.index("\n}\n")]
    first = body.index("// ---- forward sweep")
    assert re.search(r"hipMalloc|ensure_lines|reserve_coef", body[:first])
    assert not re.search(r"hipMalloc|hipHostMalloc|ensure_\w+\(|reserve_coef\(|place_lam\(", body[first:])


@pytest.mark.parametrize("capturing", [False, True])
def test_a_captured_call_is_not_made_again(monkeypatch, capturing):
    """torch's cached memory is given back, and the call repeated, outside a capture only."""
    import torch

    from paper_2102_01031_amd import lattice
    seen = []
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: seen.append("cache"))

    def refused():
        seen.append("call")
        return lattice.LAT_ENOMEM

    assert lattice._call(refused) == lattice.LAT_ENOMEM
    assert seen == (["call"] if capturing else ["call", "cache", "call"])
