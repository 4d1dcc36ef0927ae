"""Vertex tensors and boxes whose rows are stored through LDS (GPU).

Each shape of launch_vt beyond the small columns, with remainders on every axis:
64 x 8 x 8 into the cache and past it and 64 x 16 x 16 (FP32 with per-lane stores),
on whole grids; on boxes above 1/8 of the grid with even, odd and
wrapping origins, whose rows then start off the lines or wrap (per-lane stores),
and slabs of whole rows.  The vertices outside a box stay as they were.
Reference and tolerance: those of the ragged grids (FP64 torch; 1e-12 of the
largest component in FP64, 3e-6 in FP32).
"""
import numpy as np
import pytest

from tests.test_gpu_edges import _check, _field, _vertices

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    from paper_1601_02012_amd import api as A
    return A


# 64 x 8 x 8: FP64 from 65 a side, FP32 from 145; records beyond 160 MiB: FP64 from
# 152, FP32 from 192; 64 x 16 x 16: rows on 64-byte lines (FP32 n % 8, FP64 n % 4),
# FP32 from 250, FP64 from 190
@pytest.mark.parametrize("n,prec", [(64, "fp64"), (65, "fp64"), (73, "fp64"), (144, "fp32"),
                                    (145, "fp32"), (150, "fp64"), (155, "fp64"),
                                    (188, "fp64"), (190, "fp64"), (191, "fp64"),
                                    (197, "fp32"), (237, "fp32"), (248, "fp32"),
                                    (252, "fp64"), (264, "fp32"), (257, "fp32"),
                                    (335, "fp64"), (340, "fp64"), (408, "fp32"),
                                    (410, "fp32")])
def test_whole_grids(api, n, prec):
    p = _field(n, prec)
    t = api.TidalTensor(api.Grid(p, 1.0), prec)
    _check(t.build().to_torch().view(n, n, n, 6), _vertices(p.double()), prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,lo,size", [
    (120, (2, 0, 7), (100, 75, 91)), (120, (47, -5, 118), (95, 88, 77)),   # into the cache
    (173, (101, 3, -9), (153, 150, 141)),
    (230, (6, 3, 0), (201, 190, 180)), (230, (-7, 100, 200), (210, 165, 171)),  # past it
    (230, (173, 0, 5), (229, 230, 97)),
    (360, (0, 11, -3), (360, 350, 98))])                                   # slab of whole rows
def test_large_boxes(api, n, lo, size, prec):
    import torch
    assert 8 * np.prod(size) > n ** 3
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
