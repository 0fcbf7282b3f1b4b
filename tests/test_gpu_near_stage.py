"""The near-pair list and the walks at the sizes where their paths change: lists on both sides of
the length up to which every pair is walked by a wavefront, long chunks of elements with
points that jump across the geometry, and walks below the 24th level."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12  # FP64 parity, normalised by the sums of absolute contributions


def run(ctx, pts, E=True):
    import torch

    p = torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0")
    phi, F, _ = ctx.eval(p)
    st = ctx.stats()
    return phi.cpu().numpy(), F.cpu().numpy().T, st


def check(phi, F, ref):
    assert np.max(np.abs(phi - ref["phi"]) / ref["abs_phi"]) <= TOL
    assert np.max(np.sum(np.abs(F - ref["E"]), axis=1) / ref["abs_E"]) <= TOL


@pytest.mark.parametrize("n", [1, 3, 60, 250, 500, 640, 800])
def test_list_lengths(n):
    """A few to about 50,000 pairs: below and above the short-list length, leaf counts exact."""
    w = W.cylinder_workload(40, 30, 1200, n_points=10, near_frac=0.0, seed=3)
    rng = np.random.default_rng(n)
    pts, _ = W.near_points(w.tri, w.rect, n, rng)
    ctx = bemc.Context(0)
    ctx.upload_geometry(w.tri, w.rect)
    ctx.upload_densities(w.sigma)
    phi, F, st = run(ctx, pts)
    again = run(ctx, pts)
    ctx.close()
    ref = oracle.evaluate(w.tri, w.rect, w.sigma[0], pts, oracle.params(33, 7), with_abs=True)
    assert (st["near_pairs"], st["leaves"]) == (ref["stats"]["near_pairs"], ref["stats"]["leaves"])
    check(phi, F, ref)
    assert np.array_equal(again[0], phi) and np.array_equal(again[1], F)


def test_long_chunks_and_scattered_points():
    """200,000 points x 18,000 elements: chunks long enough for the points' own boxes, many runs of
    which cross steps of the Morton curve.  The pair count equals a plain count."""
    import torch

    tri, rect = W.cylinder(1.0, -5.0, 5.0, 100, 60, 6000)
    rng = np.random.default_rng(8)
    n = 200_000
    near, _ = W.near_points(tri, rect, n // 4, rng)
    pts = np.concatenate([near, rng.uniform([-1.2, -1.2, -6.0], [1.2, 1.2, 6.0], (n - len(near), 3))])
    sigma = rng.standard_normal((1, len(tri) + len(rect)))
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    phi, F, st = run(ctx, pts)
    ctx.close()
    cen = np.concatenate([W._tri_parts(tri)[0], W._rect_parts(rect)[0]])
    L = np.concatenate([W._tri_parts(tri)[2], W._rect_parts(rect)[2]])
    P, C = torch.tensor(pts, device="cuda:0"), torch.tensor(cen, device="cuda:0")
    t2 = torch.tensor((3.0 * L) ** 2, device="cuda:0")
    count = sum(int((((P[i:i + 4000, None, :] - C[None]) ** 2).sum(-1) < t2).sum()) for i in range(0, n, 4000))
    assert st["near_pairs"] == count
    some = rng.choice(n, 100, replace=False)
    check(phi[some], F[some], oracle.evaluate(tri, rect, sigma[0], pts[some], oracle.params(33, 7), with_abs=True))


def test_deeper_than_24_levels():
    """max_depth 30 and points 2e-9 L above an element: nodes below the 24th level."""
    tri = np.array([[0.0, 0.0, 0.0, 1.0, 0.1, 0.0, 0.3, 0.9, 0.0]])
    rect = np.array([[2.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 0.8, 0.0]])
    pts = np.array([[0.41, 0.33, 2e-9], [2.37, 0.29, 2e-9], [0.5, 0.5, 1.0]])
    sigma = np.array([[1.0, -0.7]])
    ctx = bemc.Context(0)
    ctx.set_rules(33, 7, 3.0, 30)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    phi, F, st = run(ctx, pts)
    ctx.close()
    ref = oracle.evaluate(tri, rect, sigma[0], pts, oracle.params(33, 7, max_depth=30), with_abs=True)
    assert st["max_depth"] > 24 and st["max_depth"] == ref["stats"]["max_depth"]
    assert st["leaves"] == ref["stats"]["leaves"]
    # the potential's terms grow like 1/h only: no cancellation
    assert np.max(np.abs(phi - ref["phi"]) / ref["abs_phi"]) <= TOL
