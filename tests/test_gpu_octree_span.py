"""Windows on both sides of the lengths from which lanes wait (octree march, GPU).

Lanes wait for the slowest of their wavefront from 500 base cells of chi in one
pass (many-source walks in persistent launches and the nearest-grid-point
integral: 1000).  Enough copies of a map to let them wait give the bits of its
rays traced one to a bundle, where no lane waits, just below and above each
length, and in as many passes as bring a pass below it.  The reference is the
march itself, so no tolerance is needed."""
import pytest

from tests.test_gpu_octree_wait import BOX, _bundles, setup  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("persistent", [0, 1])
@pytest.mark.parametrize("mode,cells", [("kappa", 498.0), ("kappa", 502.0), ("sources", 502.0),
                                        ("sources", 1002.0), ("ngp", 998.0), ("ngp", 1002.0)])
def test_spans(setup, prec, persistent, mode, cells):  # noqa: F811
    import torch
    A, t, phi, _ = setup
    dt = torch.float32 if prec == "fp32" else torch.float64
    g = A.Grid(torch.as_tensor(phi, device="cuda").to(dt), BOX, n_base=t.n,
               child_oct=torch.as_tensor(t.child_oct, device="cuda"), max_level=t.max_level)
    tt = A.TidalTensor(g, prec)
    tt.build_centres() if mode == "ngp" else tt.build()
    chi, obs, plan = cells * BOX / t.n, (3.1, 5.7, 0.9), A.Plan()

    def trace(b, persistent):
        if mode == "sources":
            o = A.trace_sources(plan, tt, b, obs, [chi, 0.63 * chi, 0.2 * chi],
                                persistent=persistent)
            return [o.moments, o.pieces, o.status]
        o = A.trace(plan, tt, b, obs, persistent=persistent,
                    integral="ngp" if mode == "ngp" else "trilinear")
        return [x for x in (o.kappa, o.kappa_comp, o.status) if x is not None]

    ref = trace(_bundles(setup, chi, "rays"), 0)
    copies = _bundles(setup, chi, "copies")
    outs = [trace(copies, persistent)]
    for passes in (2, 3):
        plan.set_shape(copies, persistent=persistent, passes=passes)
        outs.append(trace(copies, -1))
    for y in outs:
        for a, b in zip(ref, y):
            for c in b.reshape(-1, a.numel()):
                assert torch.equal(a.reshape(-1), c)
