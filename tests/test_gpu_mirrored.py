"""Rays that march against each other in one quad of lanes (GPU).

A quad of lanes shares the records of a cell only while its four rays are in
the same cell and leave it through the same face.  Bundles of mirrored
directions keep to one column of cells and march it in opposite senses, so the
lanes can be equally many crossings along in different layers.  Every ray has
to get the bits of the march that shares nothing (debug outputs) and of a
bundle of that ray alone: pairs along and near each axis, side by side, one
above the other, in 2 x 2 blocks and spread over an 8 x 8 tile, from observers
on, next to and away from the lattice's origin.
"""
import numpy as np
import pytest

from tests.test_gpu_runs import _tensor

pytestmark = pytest.mark.gpu

N, BOX = 12, 12.0
# (a, b, c): the pair is (a, b, c) and (a, b, -c), then their cyclic permutations
SLOPES = [(0.0, 0.0), (0.02, -0.01), (0.3, 0.2)]
# observer offsets in cells, the same on every axis but for a shift that keeps
# the rays off the lattice planes
OBSERVERS = [0.0, 0.4, 3.7]
MAPS = [(2, 1, "pair"), (1, 2, "pair"), (2, 2, "pair"), (2, 2, "one"), (8, 8, "pair"),
        (8, 8, "one")]
HOW = {"kappa": {}, "gamma1": dict(quantity="gamma1"), "method_a": {},
       "scalar": dict(quantity="scalar")}


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


def _directions(axis, slope, nx, ny, layout):
    """(ny*nx, 3): every second ray mirrored, or only the last one."""
    v = np.array([slope[0], slope[1], np.sqrt(1.0 - slope[0] ** 2 - slope[1] ** 2)])
    d = np.tile(np.roll(v, axis + 1), (nx * ny, 1))   # axis 2: as written
    i = np.arange(nx * ny)
    back = (i % nx + i // nx) % 2 == 1 if layout == "pair" else i == nx * ny - 1
    d[back, axis] *= -1.0
    return d


@pytest.mark.parametrize("mode", ["kappa", "gamma1", "method_a", "scalar", "sources"])
@pytest.mark.parametrize("nx,ny,layout", MAPS)
def test_mirrored_rays_share_nothing(api, mode, nx, ny, layout):
    import torch
    t = _tensor(api, mode, N, BOX, "fp32")
    plan = api.Plan()
    src = [10.0, 7.3, 4.1, 0.9]
    for axis in range(3):
        for slope in SLOPES:
            for off in OBSERVERS:
                obs = [off + 0.3, off + 0.3, off + 0.3]
                obs[axis] = off
                d = torch.as_tensor(_directions(axis, slope, nx, ny, layout)).cuda()
                b = [api.RayBundle(d, nx, ny, 10.0, 10.0, 0.37)]
                alone = [api.RayBundle(d[i:i + 1].contiguous(), 1, 1, 10.0, 10.0, 0.37, i)
                         for i in range(nx * ny)]
                what = (axis, slope, off)
                if mode == "sources":
                    x = api.trace_sources(plan, t, b, obs, src, debug=True, persistent=0)
                    for y in (api.trace_sources(plan, t, bb, obs, src, persistent=p)
                              for bb, p in ((b, 0), (b, 1), (alone, 0))):
                        assert torch.equal(x.pieces, y.pieces), what
                        assert torch.equal(x.moments, y.moments), what
                        assert torch.equal(x.status, y.status), what
                    continue
                x = api.trace(plan, t, b, obs, debug=True, persistent=0, **HOW[mode])
                assert bool((x.status == 0).all()) and bool((x.count > 9).all())
                for bb, p in ((b, 0), (b, 1), (alone, 0)):
                    y = api.trace(plan, t, bb, obs, persistent=p, **HOW[mode])
                    assert torch.equal(x.kappa, y.kappa), what
                    assert torch.equal(x.kappa_comp, y.kappa_comp), what
                    assert torch.equal(x.status, y.status), what
                k, c = torch.zeros_like(x.kappa), torch.zeros_like(x.kappa_comp)
                api.trace_noalloc(t, b, obs, kappa=k, kappa_comp=c, **HOW[mode])
                assert torch.equal(x.kappa, k) and torch.equal(x.kappa_comp, c), what
