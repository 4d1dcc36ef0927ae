"""The uniform march's paths round alike (GPU).

A launch with debug outputs marches one cell of any kind at a time; one without
them runs along the tile's main axis and crosses single faces between the runs
(FP32: records shared within quads of lanes).  Both have to give every ray the
same bits: maps along and against every axis and off the axes, ragged tiles,
dense tiles whose quads share their cells and sparse ones whose lanes do not,
rays around a periodic grid several times, windows ending inside cells.
"""
import numpy as np
import pytest

from paper_1601_02012_amd import inputs as I

pytestmark = pytest.mark.gpu

VIEWS = [(0, 0, 1), (0, 0, -1), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0),
         (0.6, -0.48, 0.64), (-1, 1, 1)]
# rays along x and y, field of view in degrees: dense, ragged, sparse, one ray
MAPS = [(16, 8, 0.3), (9, 7, 2.0), (17, 19, 40.0), (1, 1, 0.0)]
OBS = (0.3, 1.7, -2.1)


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


def _grid(api, n, box, dtype, field="phi", seed=3):
    import torch
    rng = np.random.default_rng(seed)
    v = I.poisson_phi(I.gaussian_field(n, box, rng), box) if field == "phi" else \
        rng.standard_normal((n, n, n))
    return api.Grid(torch.as_tensor(v).to(dtype).cuda(), box, field=field)


def _tensor(api, mode, n, box, prec):
    import torch
    dt = torch.float32 if prec == "fp32" else torch.float64
    phi = _grid(api, n, box, dt)
    if mode == "method_a":
        d = _grid(api, n, box, dt, "delta", 4)
        return api.TidalTensor(d, prec).build_method_a(d, phi, 1e-5)
    if mode == "scalar":
        t = api.TidalTensor(api.Grid(phi.values, box, field="phi_dot"), prec)
        return t.build_isw(phi, _grid(api, n, box, dt, seed=5), 0.7)
    t = api.TidalTensor(phi, prec)
    return t.build_centres() if mode == "ngp" else t.build()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mode", ["kappa", "gamma2", "method_a", "scalar", "ngp", "sources"])
@pytest.mark.parametrize("nx,ny,fov", MAPS)
def test_runs_round_like_single_cells(api, mode, prec, nx, ny, fov):
    import torch
    n, box = 12, 24.0
    t = _tensor(api, mode, n, box, prec)
    plan = api.Plan()
    f = np.radians(fov)
    how = {"gamma2": dict(quantity="gamma2"), "scalar": dict(quantity="scalar"),
           "ngp": dict(integral="ngp")}.get(mode, {})
    for view in VIEWS:
        d = torch.as_tensor(I.fov_directions(view, f, f, nx, ny)).cuda()
        b = [api.RayBundle(d, nx, ny, 90.0, 83.0, 1.37)]
        if mode == "sources":
            src = [90.0, 71.3, 40.0, 5.5]
            x, y = (api.trace_sources(plan, t, b, OBS, src, debug=g, persistent=0)
                    for g in (True, False))
            assert torch.equal(x.pieces, y.pieces) and torch.equal(x.moments, y.moments), view
            assert torch.equal(x.status, y.status)
            continue
        x, y, z = (api.trace(plan, t, b, OBS, debug=g, persistent=p, **how)
                   for g, p in ((True, 0), (False, 0), (False, 1)))
        assert bool((x.count > 0).all()) and bool((x.kappa != 0).all())
        for w in (y, z):
            assert torch.equal(x.kappa, w.kappa), view
            assert torch.equal(x.status, w.status)
            if prec == "fp32":
                assert torch.equal(x.kappa_comp, w.kappa_comp), view
