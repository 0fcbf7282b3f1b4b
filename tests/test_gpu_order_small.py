"""The one-workgroup order of a short list (at most 256 points) against the general one (257): the
same summation order, hence the same bits, on both sides of the segment length at which the ranks
change from comparisons to bits (128 pairs a point, 181 with two ranges of 131,072 elements), and no
step in time at 256 points when a point has thousands of near pairs."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


def strips(m):
    """m strips of length 2 around a cylinder of radius 1: each is near to every point beside it."""
    a = 2.0 * np.pi / m * np.arange(m)
    w, z = 2.0 * np.pi / m, np.zeros(m)
    return np.stack([np.cos(a), np.sin(a), z - 1.0, -np.sin(a) * w, np.cos(a) * w, z, z, z, z + 2.0], 1)


def points(n, rng):
    """Points in the cylinder's middle, away from its axis and from the strips by a tenth."""
    r, a = rng.uniform(0.1, 0.9, n), rng.uniform(0.0, 2.0 * np.pi, n)
    return np.stack([r * np.cos(a), r * np.sin(a), rng.uniform(-0.9, 0.9, n)], 1)


def evaluate(ctx, pts):
    import torch

    phi, E, _ = ctx.eval(torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0"))
    return phi, E, ctx.stats()


@pytest.mark.parametrize("m", [1, 127, 129, 180, 182, 1000])
@pytest.mark.parametrize("filler", [0, 163_840])
def test_same_sums(m, filler):
    import torch

    rng = np.random.default_rng(m)
    rect = strips(m)
    # elements in both ranges: thin triangles in front, uncharged far ones between them and the strips
    lead = np.concatenate([rect[:, 0:3], rect[:, 0:3] + rect[:, 3:6], rect[:, 0:3] + rect[:, 6:9]], 1)[: m // 2 if filler else 0]
    far = np.concatenate([W.icosphere(6) * 0.01 + np.tile([50.0 + k, 0.0, 0.0], 3) for k in (0, 1)])[:filler]
    tri = np.concatenate([lead, far])
    sigma = np.concatenate([rng.standard_normal(len(lead)), np.zeros(len(far)), rng.standard_normal(m)])
    pts = points(257, rng)
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    phi, E, st = evaluate(ctx, pts[:256])
    phi2, E2, st2 = evaluate(ctx, pts)
    ctx.close()
    k = len(lead) + m
    assert st["near_pairs"] == 256 * k and st2["near_pairs"] == 257 * k
    assert torch.equal(phi, phi2[:256]) and torch.equal(E, E2[:, :256])
    ref = oracle.evaluate(lead, rect, np.concatenate([sigma[: len(lead)], sigma[len(tri):]]), pts[:40],
                          oracle.params(33, 7), with_abs=True)
    assert np.max(np.abs(phi.cpu().numpy()[:40] - ref["phi"]) / ref["abs_phi"]) <= 1e-12


def test_long_segments_take_no_longer():
    """2,000 pairs a point: the one workgroup against the whole chip, within a factor of three (by
    comparisons alone it took nine times as long)."""
    rng = np.random.default_rng(2)
    rect = strips(2000)
    ctx = bemc.Context(0)
    ctx.upload_geometry(None, rect)
    ctx.upload_densities(rng.standard_normal(2000))
    pts = points(257, rng)
    small = min(evaluate(ctx, pts[:256])[2]["near_ms"] for _ in range(4))
    general = min(evaluate(ctx, pts)[2]["near_ms"] for _ in range(4))
    ctx.close()
    assert small <= 3.0 * general, (small, general)
