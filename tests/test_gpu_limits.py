"""Open grids and crossing limits on the uniform march (GPU).

Launches whose rays may end early, at the edge of an open grid or at a limit of
crossings, march without runs.  The path of every ray (crossing hash, count,
status) is the oracle's; direct, persistent and split launches without debug
outputs give the bits of the debug launch.  Observers stand inside the usable
cells (2 .. n - 3), on their border planes, in the two outer layers and beyond
the grid, so that rays leave through every face, some at once, some never, side
by side in one wavefront; limits from one crossing to the longest ray's own.
kappa against the oracle in FP64: 1e-11 of the largest value.
"""
import numpy as np
import pytest

from tests.test_gpu_runs import _tensor

pytestmark = pytest.mark.gpu

N = 16
VIEWS = [(0, 0, 1), (0, 0, -1), (1, 0, 0), (0, -1, 0), (0.6, -0.48, 0.64), (-1, 1, 1)]
OBSERVERS = [(8.3, 7.6, 8.1), (2.0, 8.0, 14.0), (1.4, 7.3, 8.2), (8.1, 14.6, 0.5),
             (-3.3, 7.7, 18.2)]
HOW = {"kappa": {}, "method_a": {}, "scalar": dict(quantity="scalar"), "ngp": dict(integral="ngp")}


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


def _open(api, mode, prec):
    """The periodic tensor's fields on an open grid."""
    import torch
    real = api.Grid

    class Open(real):
        def __init__(self, *a, **k):
            super().__init__(*a, boundary="open", **k)

    api.Grid = Open
    try:
        t = _tensor(api, mode, N, float(N), prec)
    finally:
        api.Grid = real
    torch.cuda.synchronize()
    return t


def _same(x, y, what):
    import torch
    assert torch.equal(x.status, y.status), what
    for a in ("kappa", "kappa_comp", "moments", "pieces"):
        if getattr(x, a, None) is not None:
            assert torch.equal(getattr(x, a), getattr(y, a)), (what, a)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", ["kappa", "method_a", "scalar", "ngp", "sources"])
def test_open_grids(api, oracle, mode, prec):
    import torch

    from paper_1601_02012_amd import inputs as I
    t = _open(api, mode, prec)
    plan = api.Plan()
    nx, ny = 19, 11
    f = np.radians(30.0)
    seen = set()
    for obs in OBSERVERS:
        for view in VIEWS:
            dirs = I.fov_directions(view, f, f, nx, ny)
            d = torch.as_tensor(dirs).cuda()
            b = [api.RayBundle(d, nx, ny, 12.0, 11.0, 0.0)]
            plan.set_shape(b, passes=5)
            ref = oracle.trace_uniform(N, float(N), obs, dirs, 12.0, 11.0, 0.0,
                                       phi=np.zeros((N, N, N)), open_boundary=True,
                                       ngp=mode == "ngp")
            if mode == "sources":
                src = [9.5, 6.0, 0.4]
                x = api.trace_sources(plan, t, b, obs, src, debug=True, persistent=0)
                same = [api.trace_sources(plan, t, b, obs, src, persistent=p) for p in (0, 1, -1)]
            else:
                x = api.trace(plan, t, b, obs, debug=True, persistent=0, **HOW[mode])
                same = [api.trace(plan, t, b, obs, persistent=p, **HOW[mode]) for p in (0, 1, -1)]
                assert np.array_equal(x.hash.cpu().numpy().view(np.uint64), ref.hash), (obs, view)
                assert np.array_equal(x.count.cpu().numpy(), ref.ncross), (obs, view)
            assert np.array_equal(x.status.cpu().numpy(), ref.status), (obs, view)
            for y in same:
                _same(x, y, (obs, view))
            seen |= set(np.unique(ref.status).tolist())
    assert len(seen) == 2   # rays that end inside and rays that leave


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", ["kappa", "method_a", "scalar", "ngp", "sources"])
def test_crossing_limits(api, oracle, mode, prec):
    import torch

    from paper_1601_02012_amd import inputs as I
    t = _tensor(api, mode, N, float(N), prec)
    plan = api.Plan()
    nx, ny = 11, 9
    f = np.radians(12.0)
    obs = (0.3, 1.7, -2.1)
    for view in VIEWS:
        dirs = I.fov_directions(view, f, f, nx, ny)
        d = torch.as_tensor(dirs).cuda()
        b = [api.RayBundle(d, nx, ny, 40.0, 39.0, 1.5)]
        phi = np.zeros((N, N, N))
        full = oracle.trace_uniform(N, float(N), obs, dirs, 40.0, 39.0, 1.5, phi=phi)
        for lim in (1, 2, int(full.ncross.min()), int(np.median(full.ncross)), int(full.ncross.max())):
            if mode == "sources":
                src = [30.0, 12.2]   # a stop inside a cell is a piece of its own: up to two more
                x, y, z = (api.trace_sources(plan, t, b, obs, src, debug=g, persistent=p,
                                             max_crossings=lim)
                           for g, p in ((True, 0), (False, 0), (False, 1)))
                assert bool((x.count <= lim).all())
            else:
                x, y, z = (api.trace(plan, t, b, obs, debug=g, persistent=p, max_crossings=lim,
                                     **HOW[mode])
                           for g, p in ((True, 0), (False, 0), (False, 1)))
                assert np.array_equal(x.count.cpu().numpy(), np.minimum(full.ncross, lim)), lim
                cut = x.status.cpu().numpy() != 0
                assert np.array_equal(cut, full.ncross > lim), lim
            _same(x, y, (view, lim))
            _same(x, z, (view, lim))


def test_open_kappa_against_the_oracle(api, oracle):
    import torch

    from paper_1601_02012_amd import inputs as I
    rng = np.random.default_rng(5)
    phi = rng.standard_normal((N, N, N))
    t = api.TidalTensor(api.Grid(torch.as_tensor(phi).cuda(), float(N), boundary="open"),
                        "fp64").build()
    plan = api.Plan()
    f = np.radians(30.0)
    for obs in OBSERVERS:
        for view in VIEWS:
            dirs = I.fov_directions(view, f, f, 19, 11)
            b = [api.RayBundle(torch.as_tensor(dirs).cuda(), 19, 11, 12.0, 11.0, 0.0)]
            ref = oracle.trace_uniform(N, float(N), obs, dirs, 12.0, 11.0, 0.0, phi=phi,
                                       open_boundary=True)
            got = api.trace(plan, t, b, obs, persistent=0)
            assert np.array_equal(got.status.cpu().numpy(), ref.status)
            k = got.kappa.cpu().numpy()
            scale = max(np.abs(ref.kappa).max(), 1e-30)
            assert np.abs(k - ref.kappa).max() <= 1e-11 * scale, (obs, view)
