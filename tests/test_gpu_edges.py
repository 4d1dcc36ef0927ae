"""Grid builds and the per-source sums at the edges of their tiles (GPU).

Vertex tensors and cell-centre records on grids whose sides leave remainders
against every column shape (and reach each of them), vertex boxes of a few
vertices, kappa_from_pieces around its tiles of 8 sources and 256 rays.
Reference: the same stencils in FP64 torch.  Tolerances: FP64 1e-12 of the
field's largest component; FP32 6 roundings of values up to 8 (vertex: the sum
of 8 cells) times the largest component, 2^-24 * 6 * 8 < 3e-6.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


def _centres(p):
    import torch
    def r(dz=0, dy=0, dx=0):
        return torch.roll(p, (-dz, -dy, -dx), (0, 1, 2))
    def d2(**k):
        return (r(**k) - p) - (p - r(**{a: -v for a, v in k.items()}))
    def mixed(a, b):
        s = {(i, j): r(**{a: i, b: j}) for i in (1, -1) for j in (1, -1)}
        return 0.25 * ((s[1, 1] - s[1, -1]) - (s[-1, 1] - s[-1, -1]))
    return torch.stack([d2(dx=1), d2(dy=1), d2(dz=1), mixed("dx", "dy"), mixed("dx", "dz"),
                        mixed("dy", "dz")], -1)


def _vertices(p):
    import torch
    c = _centres(p)
    for a in (0, 1, 2):
        c = 0.5 * (c + torch.roll(c, 1, a))
    return c


def _field(n, prec):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    p = torch.randn((n, n, n), generator=g, device="cuda", dtype=torch.float64)
    return p.float() if prec == "fp32" else p


def _check(got, ref, prec):
    import torch
    nan = torch.isnan(ref)
    lim = (3e-6 if prec == "fp32" else 1e-12) * float(ref[~nan].abs().max())
    assert torch.equal(torch.isnan(got), nan)
    assert float((got.double() - ref)[~nan].abs().max()) <= lim


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [4, 63, 65, 100, 130, 161, 200, 257])
def test_builds_on_ragged_grids(api, n, prec):
    p = _field(n, prec)
    t = api.TidalTensor(api.Grid(p, 1.0), prec)
    ref = _vertices(p.double())
    _check(t.build().to_torch().view(n, n, n, 6), ref, prec)
    _check(t.build_centres().to_torch().view(n, n, n, 6), _centres(p.double()), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [6, 65, 130])
def test_centres_on_open_grids(api, n, prec):
    p = _field(n, prec)
    t = api.TidalTensor(api.Grid(p, 1.0, boundary="open"), prec)
    ref = _centres(p.double())
    for a in range(3):
        ref.select(a, 0).fill_(float("nan"))
        ref.select(a, n - 1).fill_(float("nan"))
    _check(t.build_centres().to_torch().view(n, n, n, 6), ref, prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("lo,size", [((0, 0, 0), (1, 1, 1)), ((-3, 60, 95), (65, 5, 9)),
                                     ((90, 90, 90), (70, 33, 40)), ((5, 0, 0), (100, 100, 3))])
def test_box_builds(api, lo, size, prec):
    import torch
    n = 100
    p = _field(n, prec)
    t = api.TidalTensor(api.Grid(p, 1.0), prec)
    t.build(api.Grid(torch.zeros_like(p), 1.0))
    got = t.build_box(lo, size, grid=api.Grid(p, 1.0)).to_torch().view(n, n, n, 6)
    ref = _vertices(p.double())
    inside = [torch.zeros(n, dtype=torch.bool, device="cuda") for _ in range(3)]
    for a in range(3):
        inside[a][torch.arange(lo[a], lo[a] + size[a]) % n] = True
    m = inside[2][:, None, None] & inside[1][None, :, None] & inside[0][None, None, :]
    _check(got, torch.where(m[..., None], ref, torch.zeros_like(ref)), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("ns", [1, 7, 8, 9, 17])
@pytest.mark.parametrize("nr", [1, 255, 257])
def test_kappa_from_pieces(api, nr, ns, prec):
    import torch
    rng = np.random.default_rng(ns * 1000 + nr)
    t = api.TidalTensor(api.Grid(_field(4, prec), 4.0), prec)   # h0 = 1
    src = np.sort(rng.uniform(1.0, 9.0, ns))[::-1].copy()
    mom = rng.standard_normal((nr, 4 if prec == "fp32" else 2))
    mom = mom.astype(np.float32 if prec == "fp32" else np.float64)
    pcs = rng.standard_normal((nr, ns, 2))
    st = api.SourcesOutput(torch.as_tensor(mom).cuda(), torch.as_tensor(pcs).cuda(), None)
    got = api.kappa_from_pieces(api.Plan(), t, src, st).cpu().numpy()
    m = mom.astype(np.float64)
    a, b = (m[:, 0] - m[:, 1], m[:, 2] - m[:, 3]) if prec == "fp32" else (m[:, 0], m[:, 1])
    for j in range(ns - 1, -1, -1):   # the same operations in the same order: equal bits
        assert np.array_equal(got[:, j], a - b / src[j])
        a, b = a + pcs[:, j, 0], b + pcs[:, j, 1]
