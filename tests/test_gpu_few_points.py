"""Evaluations of few points (an element per lane, one launch for the near pairs' order) on both
sides of the sizes where the launches change: 1, 2 | 3 points (points per lane), 32 | 33 (lanes to
a result), 128 | 129 (element per lane), 256 | 257 (order in one workgroup), 2,048 | 2,049 (points
per lane); elements fewer than one workgroup's lanes, one more than them, one kind alone."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6}  # normalised by the sums of absolute contributions


def soup(n_tri, n_rect, seed):
    rng = np.random.default_rng(seed)
    c = rng.uniform(-1.0, 1.0, (n_tri, 1, 3))
    tri = (c + rng.normal(size=(n_tri, 3, 3)) * 0.1).reshape(n_tri, 9)
    u = rng.normal(size=(n_rect, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    v = np.cross(u, rng.normal(size=(n_rect, 3)))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    s = 10.0 ** rng.uniform(-1.5, -0.7, (n_rect, 2))
    rect = np.concatenate([rng.uniform(-1.0, 1.0, (n_rect, 3)), u * s[:, :1], v * s[:, 1:]], axis=1)
    return tri, rect, rng


def points(tri, rect, n, rng):
    near, _ = W.near_points(tri, rect, max(1, n // 3), rng)
    return np.concatenate([near, rng.uniform(-4.0, 4.0, (n, 3))])[:n]


@pytest.mark.parametrize("n", [1, 2, 3, 5, 32, 33, 128, 129, 256, 257, 2048, 2049])
@pytest.mark.parametrize("dr", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_field(n, dr, precision):
    import torch

    tri, rect, rng = soup(300, 213, 100 + n)
    pts = points(tri, rect, n, rng)
    sigma = rng.standard_normal(len(tri) + len(rect))
    ctx = bemc.Context(0)
    ctx.set_dr_rules(dr)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    p = torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0")
    phi, E, _ = ctx.eval(p, precision)
    st = ctx.stats()
    only, none, _ = ctx.eval(p, precision, with_E=False)
    kept = torch.empty(n, dtype=torch.float64, device="cuda:0")
    F = torch.empty((3, n), dtype=torch.float64, device="cuda:0")
    ctx.eval_noalloc(p, kept, F, precision)
    again, _, _ = ctx.eval(p, precision)
    torch.cuda.synchronize()
    ctx.close()
    ref = oracle.evaluate(tri, rect, sigma, pts, oracle.params(33, 7, dr_rules=dr), with_abs=True)
    for k in ("near_pairs", "leaves"):
        assert st[k] == ref["stats"][k]
    for a, b in ((phi, E), (only, None), (kept, F)):
        assert np.max(np.abs(a.cpu().numpy() - ref["phi"]) / ref["abs_phi"]) <= TOL[precision]
        if b is not None:
            assert np.max(np.sum(np.abs(b.cpu().numpy().T - ref["E"]), axis=1) / ref["abs_E"]) <= TOL[precision]
    assert none is None and torch.equal(again, phi)


@pytest.mark.parametrize("n", [1, 4, 128, 129])
@pytest.mark.parametrize("dr", [False, True])
def test_gradient(n, dr):
    import torch

    tri, rect, rng = soup(300, 213, 200 + n)
    pts = points(tri, rect, n, rng)
    sigma = rng.standard_normal(len(tri) + len(rect))
    ctx = bemc.Context(0)
    ctx.set_dr_rules(dr)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    G, _ = ctx.eval_gradient(torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0"))
    got = G.cpu().numpy().T
    ctx.close()
    ref = oracle.gradient(tri, rect, sigma, pts, oracle.params(33, 7, dr_rules=dr))
    # normalised by the terms' Frobenius norms; six components of at most the norm each
    assert np.max(np.max(np.abs(got - ref["G"]), axis=1) / ref["abs_T"]) <= 1e-12


@pytest.mark.parametrize("n_tri,n_rect", [(1, 0), (0, 1), (256, 0), (257, 0), (0, 300), (255, 2)])
def test_element_counts(n_tri, n_rect):
    import torch

    tri, rect, rng = soup(n_tri, n_rect, 7)
    pts = points(tri, rect, 9, rng)
    sigma = rng.standard_normal(n_tri + n_rect)
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri if n_tri else None, rect if n_rect else None)
    ctx.upload_densities(sigma)
    phi, E, _ = ctx.eval(torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0"))
    phi, E = phi.cpu().numpy(), E.cpu().numpy().T
    ctx.close()
    ref = oracle.evaluate(tri, rect, sigma, pts, oracle.params(33, 7), with_abs=True)
    assert np.max(np.abs(phi - ref["phi"]) / ref["abs_phi"]) <= 1e-12
    assert np.max(np.sum(np.abs(E - ref["E"]), axis=1) / ref["abs_E"]) <= 1e-12


@pytest.mark.parametrize("grow", [False, True])
def test_short_list_capacity(grow):
    """More near pairs than the list holds: reported with a fixed list, grown otherwise."""
    import torch

    tri, rect, rng = soup(300, 213, 11)
    pts = points(tri, rect, 60, rng)
    sigma = rng.standard_normal(513)
    ctx = bemc.Context(0)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    ctx.set_near_capacity(16, grow=grow)
    phi, E, _ = ctx.eval(torch.tensor(np.ascontiguousarray(pts.T), device="cuda:0"))
    if not grow:
        with pytest.raises(bemc.BemcError) as err:
            ctx.stats()
        assert err.value.code == bemc.E_LIMIT
        ctx.close()
        return
    st = ctx.stats()
    phi = phi.cpu().numpy()
    ctx.close()
    ref = oracle.evaluate(tri, rect, sigma, pts, oracle.params(33, 7), with_abs=True)
    assert st["near_pairs"] == ref["stats"]["near_pairs"] > 16
    assert np.max(np.abs(phi - ref["phi"]) / ref["abs_phi"]) <= 1e-12

