"""Lanes of a wavefront that wait for the slowest one (octree march, GPU).

A ray's result does not depend on the rays that share its wavefront: a map
whose window spans many times the lead after which lanes wait (32 base cells),
through a tree that is refined in one part only, equals its rays traced one to
a bundle (a lane alone never waits) bit for bit, also where a limit on the
crossings ends some of them early.  Lanes wait only in launches of more than
two tiles per compute unit: the map is traced alone and as the first of enough
copies of it.  The reference is the march itself, so no tolerance is needed."""
import math

import numpy as np
import pytest

from paper_1601_02012_amd import inputs as I

pytestmark = pytest.mark.gpu

NX, NY, BOX = 11, 9, 24.0


@pytest.fixture(scope="module")
def setup():
    import torch
    from paper_1601_02012_amd import api as A
    rng = np.random.default_rng(5)
    t = I.random_octree(12, 3, 0.3, rng, region=(1.0, 7.0))
    phi = 1e-4 * rng.standard_normal(t.n_cells) * 0.5 ** (2 * t.cell_level)
    fov = math.radians(6.0)
    d = A.fov_directions((0.2, -0.1, 1.0), fov, fov * NY / NX, NX, NY)
    return A, t, phi, torch.as_tensor(d, device="cuda")


def _bundles(setup, chi, how):
    import torch
    A, _, _, d = setup
    if how == "map":
        return [A.RayBundle(d, NX, NY, chi, chi, 0.0)]
    if how == "copies":      # of 2 x 2 tiles each
        cus = torch.cuda.get_device_properties(0).multi_processor_count
        return [A.RayBundle(d, NX, NY, chi, chi, 0.0, ray_offset=i * NX * NY)
                for i in range(cus // 2 + 1)]
    flat = d.reshape(-1, 3)
    return [A.RayBundle(flat[i:i + 1].contiguous(), 1, 1, chi, chi, 0.0, ray_offset=i)
            for i in range(NX * NY)]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("cells", [31.0, 700.0])       # below the lead, and many times it
@pytest.mark.parametrize("mode", ["trilinear", "ngp", "limit", "sources"])
def test_waiting_changes_no_ray(setup, prec, persistent, cells, mode):
    import torch
    A, t, phi, _ = setup
    dt = torch.float32 if prec == "fp32" else torch.float64
    g = A.Grid(torch.as_tensor(phi, device="cuda").to(dt), BOX, n_base=t.n,
               child_oct=torch.as_tensor(t.child_oct, device="cuda"), max_level=t.max_level)
    tt = A.TidalTensor(g, prec)
    tt.build_centres() if mode == "ngp" else tt.build()
    chi = cells * BOX / t.n
    plan = A.Plan()
    out, limit = [], 0
    if mode == "limit":
        n = A.trace(plan, tt, _bundles(setup, chi, "map"), (3.1, 5.7, 0.9), debug=True).count
        limit = int(n.median())
    for how in ("rays", "map", "copies"):
        b = _bundles(setup, chi, how)
        obs = (3.1, 5.7, 0.9)
        if mode == "sources":
            o = A.trace_sources(plan, tt, b, obs, [chi, 0.63 * chi, 0.2 * chi],
                                persistent=persistent)
            out.append((o.moments, o.pieces, o.status))
        else:
            o = A.trace(plan, tt, b, obs, persistent=persistent,
                        integral="ngp" if mode == "ngp" else "trilinear",
                        max_crossings=limit)
            out.append((o.kappa, o.kappa_comp, o.status) if prec == "fp32"
                       else (o.kappa, o.status))
    for y in out[1:]:
        for a, b in zip(out[0], y):
            b = b.reshape(-1, a.numel())
            assert all(torch.equal(a.reshape(-1), c) for c in b)
    if mode == "limit":
        assert 0 < int((out[0][-1] != 0).sum()) < NX * NY
