"""The subdivision visit limit (2^22 nodes per pair) holds whichever way a pair is walked, also
when a wavefront hands the subtrees of a wide level to single lanes: a near limit in the thousands
asks for tens of millions of nodes and is refused, one just below the visit limit is evaluated."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc

pytestmark = pytest.mark.gpu

TRI = np.array([[0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.5, 0.75 ** 0.5, 0.0]])
RECT = np.array([[0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0, 0.0]])
LIMIT = 1 << 22


def nodes(kind, near_dr, depth=24):
    """Nodes below the root that a point at half the side above the centroid visits, level by level."""
    tri = kind == "tri"
    p = np.array([0.5, 0.75 ** 0.5 / 3.0, 0.5]) if tri else np.array([0.5, 0.5, 0.5])
    tiles = (TRI[0].reshape(1, 3, 3) if tri else np.array([[[0.0, 0, 0], [1.0, 0, 0], [0, 1.0, 0], [1.0, 1.0, 0]]]))
    total = 0
    for level in range(1, depth + 1):
        if tri:
            a, b, c = tiles[:, 0], tiles[:, 1], tiles[:, 2]
            ab, bc, ca = (a + b) / 2, (b + c) / 2, (c + a) / 2
            tiles = np.concatenate([np.stack(t, 1) for t in ((a, ab, ca), (ab, b, bc), (ca, bc, c), (bc, ca, ab))])
        else:
            half = tiles / 2 + tiles[:, :1] / 2
            d = half[:, 1:] - half[:, :1]
            tiles = np.concatenate([half, half + d[:, :1], half + d[:, 1:2], half + d[:, 2:3]])
        total += len(tiles)
        if total > 2 * LIMIT:
            return total
        near = np.linalg.norm(tiles.mean(1) - p, axis=1) < near_dr * 0.5 ** level
        tiles = tiles[near]
        if len(tiles) == 0:
            return total
    return total


@pytest.mark.parametrize("kind", ["tri", "rect"])
@pytest.mark.parametrize("near_dr", [500.0, 2000.0])
def test_limit(kind, near_dr):
    import torch

    tri, rect = (TRI, None) if kind == "tri" else (None, RECT)
    p = np.array([[0.5, 0.75 ** 0.5 / 3.0, 0.5]]) if kind == "tri" else np.array([[0.5, 0.5, 0.5]])
    over = near_dr > 1000.0
    visits = nodes(kind, near_dr)
    assert visits > 2 * LIMIT if over else LIMIT // 8 < visits < LIMIT
    ctx = bemc.Context(0)
    ctx.set_rules(4, 2, near_dr)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(np.ones(1))
    phi, E, _ = ctx.eval(torch.tensor(p.T.copy(), device="cuda:0"))
    if over:
        with pytest.raises(bemc.BemcError) as err:
            ctx.stats()
        ctx.close()
        assert err.value.code == bemc.E_LIMIT and "visit limit" in str(err.value)
        return
    st = ctx.stats()
    phi, E = phi.cpu().numpy(), E.cpu().numpy().T
    ctx.close()
    ref = oracle.evaluate(TRI if tri is not None else np.zeros((0, 9)), RECT if rect is not None else np.zeros((0, 9)),
                          np.ones(1), p, oracle.params(4, 2, near_dr=near_dr), with_abs=True)
    assert abs(st["leaves"] - ref["stats"]["leaves"]) <= 1e-3 * ref["stats"]["leaves"]
    assert abs(phi[0] - ref["phi"][0]) <= 1e-12 * ref["abs_phi"][0]
    assert np.abs(E[0] - ref["E"][0]).sum() <= 1e-12 * ref["abs_E"][0]
