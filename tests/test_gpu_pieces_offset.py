"""kappa of every source: pieces that start on any double, few sources (GPU).

The pieces of a walk may be a part of a larger buffer, aligned to eight bytes
only: the sums are those of an aligned copy, bit for bit.  Up to three sources
are summed in place, more through LDS: both do the same operations in the same
order as numpy does here, so the bits are equal.
"""
import numpy as np
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


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("ns", [2, 3, 4])
@pytest.mark.parametrize("nr", [1, 256, 513])
def test_few_sources(nr, ns, prec):
    import torch

    from paper_1601_02012_amd import api
    rng = np.random.default_rng(10 * nr + ns)
    ft = np.float32 if prec == "fp32" else np.float64
    grid = torch.zeros((4, 4, 4), device="cuda",
                       dtype=torch.float32 if prec == "fp32" else torch.float64)
    t = api.TidalTensor(api.Grid(grid, 4.0), prec)   # h0 = 1
    src = np.sort(rng.uniform(1.0, 9.0, ns))[::-1].copy()
    mom = rng.standard_normal((nr, 4 if prec == "fp32" else 2)).astype(ft)
    pcs = rng.standard_normal((nr, ns, 2))
    st = api.SourcesOutput(torch.as_tensor(mom).cuda(), torch.as_tensor(pcs).cuda(), None)
    got = api.kappa_from_pieces(api.Plan(), t, src, st).cpu().numpy()
    m = mom.astype(np.float64)
    a, b = (m[:, 0] - m[:, 1], m[:, 2] - m[:, 3]) if prec == "fp32" else (m[:, 0], m[:, 1])
    for j in range(ns - 1, -1, -1):
        assert np.array_equal(got[:, j], a - b / src[j])
        a, b = a + pcs[:, j, 0], b + pcs[:, j, 1]
