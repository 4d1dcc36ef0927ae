"""kappa of every source from pieces that start on any double (GPU).

The pieces of a walk may be a part of a larger buffer, aligned to eight bytes
only: the sums are those of an aligned copy, bit for bit.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nr,ns", [(1, 1), (257, 9)])
def test_pieces_at_an_odd_double(nr, ns, prec):
    import torch

    from paper_1601_02012_amd import api
    dt = torch.float32 if prec == "fp32" else torch.float64
    t = api.TidalTensor(api.Grid(torch.zeros((4, 4, 4), device="cuda", dtype=dt), 4.0), prec)
    g = torch.Generator(device="cuda").manual_seed(nr)
    mom = torch.randn((nr, 4 if prec == "fp32" else 2), generator=g, device="cuda", dtype=dt)
    flat = torch.randn(2 * nr * ns + 1, generator=g, device="cuda", dtype=torch.float64)
    src = [9.0 - 0.5 * j for j in range(ns)]
    part = flat[1:].view(nr, ns, 2)
    assert part.is_contiguous() and part.data_ptr() % 16 == 8
    out = [api.kappa_from_pieces(api.Plan(), t, src, api.SourcesOutput(mom, p, None))
           for p in (part, part.clone())]
    assert torch.equal(*out)
