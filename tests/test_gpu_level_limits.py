"""Rules by distance ratio with the near limit raised above a level's limit: pairs in between
belong to the near field whatever level their distance ratio asks for."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [40, 700, 3000])
def test_near_limit_above_a_level(n):
    import torch

    rng = np.random.default_rng(n)
    tri = W.icosphere(2)
    rect = W.cylinder_mantle(0.5, -0.5, 0.5, 20, 5)
    sigma = rng.standard_normal(len(tri) + len(rect))
    pts = W.shell_points(n, 1.05, 5.0, rng)
    ctx = bemc.Context(0)
    ctx.set_dr_rules(True, (20.0, 12.0, 8.0), (20.0, 12.0, 8.0))
    ctx.set_rules(33, 7, 25.0, 24)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    phi, E, _ = ctx.eval(torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0"))
    st = ctx.stats()
    phi, E = phi.cpu().numpy(), E.cpu().numpy().T
    ctx.close()
    # beyond the near limit every pair takes the coarsest level, within it none does
    cen = np.concatenate([W._tri_parts(tri)[0], W._rect_parts(rect)[0]])
    L = np.concatenate([W._tri_parts(tri)[2], W._rect_parts(rect)[2]])
    near = int(np.sum(np.linalg.norm(pts[:, None] - cen[None], axis=2) < 25.0 * L[None]))
    assert st["near_pairs"] == near
    assert st["node_interactions"] == 7 * (n * len(cen) - near)
    # 7 points at a distance ratio of 25 leave a relative error of about (0.3 / 25)^6 = 3e-12 per element
    ref = oracle.evaluate(tri, rect, sigma, pts, oracle.params(33, 7, near_dr=25.0), with_abs=True)
    assert np.max(np.abs(phi - ref["phi"]) / ref["abs_phi"]) <= 3e-11
    assert np.max(np.sum(np.abs(E - ref["E"]), axis=1) / ref["abs_E"]) <= 3e-10
