"""The collocation product at the sizes where its launches change: fewer elements than one chunk, a
few chunks, several points per lane; one, three and eight densities (the result's lanes)."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


def geometry(kind):
    if kind == "tiny":
        return W.icosphere(0), W.cylinder_mantle(3.0, -2.0, 2.0, 6, 1)[:3]
    if kind == "ico":
        return W.icosphere(2), np.zeros((0, 9))
    return W.cylinder(1.0, -5.0, 5.0, 40, 30, 1200)


@pytest.mark.parametrize("kind", ["tiny", "ico", "cylinder"])
@pytest.mark.parametrize("n_rhs", [1, 3, 8])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-6)])
def test_product(kind, n_rhs, precision, tol):
    import torch

    tri, rect = geometry(kind)
    ne = len(tri) + len(rect)
    rng = np.random.default_rng(ne + n_rhs)
    sigma = rng.standard_normal((n_rhs, ne))
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri, rect)
    s = torch.tensor(sigma, device="cuda:0")
    out = ctx.collocation(s, precision)
    again = ctx.collocation(s, precision)  # reuses the near stage
    torch.cuda.synchronize()
    assert torch.equal(out, again)
    got = out.cpu().numpy()
    ctx.close()
    rows = rng.choice(ne, min(ne, 60), replace=False)
    cen = np.concatenate([W._tri_parts(tri)[0], W._rect_parts(rect)[0]])[rows]
    for r in (0, n_rhs - 1):
        ref = oracle.evaluate(tri, rect, sigma[r], cen, oracle.params(33, 7), with_abs=True)
        assert np.max(np.abs(got[r, rows] - ref["phi"]) / ref["abs_phi"]) <= tol


@pytest.mark.parametrize("shape, restart", [((9, 7, 27), 200), ((8, 16, 64), 5), ((24, 20, 240), 13), ((50, 60, 1000), 200)])
def test_solver_projections(shape, restart):
    """Elements below, at and above a workgroup of the projection, one and several partial sums of
    the dot products, short and long bases: the residual that the solver reports is the product's."""
    import torch

    half = 2.0 * np.pi * shape[1] / shape[0]  # rectangles twice as high as wide
    tri, rect = W.cylinder(1.0, -half, half, *shape)
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri, rect)
    b = torch.full((len(tri) + len(rect),), 3.0, dtype=torch.float64, device="cuda:0")
    sigma, info = ctx.solve(b, tol=1e-10, max_iter=600, restart=restart)
    again, _ = ctx.solve(b, tol=1e-10, max_iter=600, restart=restart)
    r = (b - ctx.collocation(sigma[None])[0]).norm() / b.norm()
    ctx.close()
    assert info["converged"] == 1
    # both residuals are formed from the same densities; the sums round at 1e-15
    assert abs(float(r) - info["rel_residual"]) <= 1e-13 and float(r) <= 1.001e-10
    assert torch.equal(again, sigma)
