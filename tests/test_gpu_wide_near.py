"""Near limits on both sides of the one beyond which only pairs within L / 16 are walked by a whole
wavefront (lists longer than those that are walked so throughout): counts and parity, field and gradient."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("near_dr", [4.9, 5.0, 5.1, 7.0])
def test_wide_near_limits(near_dr):
    import torch

    tri, rect = W.cylinder(1.0, -5.0, 5.0, 40, 30, 1200)
    rng = np.random.default_rng(12)
    sigma = rng.standard_normal(len(tri) + len(rect))
    pts, _ = W.near_points(tri, rect, 260, rng)
    ctx = bemc.Context(0)
    ctx.set_rules(12, 5, near_dr)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    p = torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0")
    phi, E, _ = ctx.eval(p)
    st = ctx.stats()
    G, _ = ctx.eval_gradient(p)
    stg = ctx.stats()
    ctx.close()
    prm = oracle.params(12, 5, near_dr=near_dr)
    ref = oracle.evaluate(tri, rect, sigma, pts, prm, with_abs=True)
    gref = oracle.gradient(tri, rect, sigma, pts[:60], prm)
    assert st["near_pairs"] == stg["near_pairs"] == ref["stats"]["near_pairs"] > 40_000
    # (the walk's distance tests are the oracle's but for the rounding of the nodes' positions)
    assert abs(st["leaves"] - ref["stats"]["leaves"]) <= 1e-3 * ref["stats"]["leaves"] and st["leaves"] == stg["leaves"]
    assert np.max(np.abs(phi.cpu().numpy() - ref["phi"]) / ref["abs_phi"]) <= 1e-12
    assert np.max(np.sum(np.abs(E.cpu().numpy().T - ref["E"]), axis=1) / ref["abs_E"]) <= 1e-12
    assert np.max(np.abs(G.cpu().numpy().T[:60] - gref["G"]).max(axis=1) / gref["abs_T"]) <= 1e-12
