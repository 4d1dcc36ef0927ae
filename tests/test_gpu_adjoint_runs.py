"""The adjoint's runs along the tile's main axis (GPU) against the oracle.

Maps along and against every axis and off the axes; tiles whose rays share
their cells (runs, retired four layers at a time: windows of 1 to 9 layers and
grids of 4 and 5 cells, where a batch wraps around the box), tiles that start
across a plane (lanes a crossing apart), ragged tiles and rays without weight.
Tolerance: the adjoint tests' 1e-4 of the largest gradient.
"""
import numpy as np
import pytest

from paper_1601_02012_amd import inputs as I
from tests._cases import gpu_bundle, gpu_grid

pytestmark = pytest.mark.gpu

VIEWS = [(0, 0, 1), (0, 0, -1), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0.6, -0.48, 0.64)]


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


@pytest.mark.parametrize("n,nx,ny,fov,hi,lo,obs", [
    (4, 8, 8, 0.02, 30.3, 0.2, (0.4, 0.6, 0.3)),
    (5, 8, 8, 0.02, 9.2, 4.4, (0.4, 0.6, 0.3)),
    (12, 17, 9, 0.05, 30.0, 0.0, (0.0, 0.0, 0.0)),
    (12, 16, 16, 0.4, 25.0, 1.5, (6.02, 6.01, 5.97)),
])
@pytest.mark.parametrize("view", VIEWS)
def test_adjoint_runs_match_oracle(api, oracle, view, n, nx, ny, fov, hi, lo, obs):
    import torch
    rng = np.random.default_rng(n * nx)
    phi = rng.standard_normal((n, n, n)).astype(np.float32)
    dirs = I.fov_directions(view, fov, fov, nx, ny)
    w = rng.standard_normal(nx * ny).astype(np.float32)
    w[::7] = 0.0
    g = gpu_grid(api, phi, float(n))
    t = api.TidalTensor(g, "fp32").build()
    b = gpu_bundle(api, dirs, nx, ny, 31.0, hi, lo)
    got = api.trace_adjoint(api.Plan(), t, g, [b], obs, torch.as_tensor(w).cuda()).cpu().numpy()
    ref = oracle.trace_adjoint_uniform(n, float(n), obs, dirs, 31.0, hi, lo, w.astype(np.float64))
    scale = np.abs(ref).max()
    assert scale > 0
    np.testing.assert_allclose(got, ref, rtol=0, atol=1e-4 * scale)
