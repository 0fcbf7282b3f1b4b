"""The allocation-free evaluation's potential is the same bit for bit with and without the field, on
both sides of the sizes at which the final sums change kernels (65,536 results: 16,384 points with the
four rows that are summed in either case, 65,536 points with one row)."""
import numpy as np
import pytest

from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cyl():
    return W.cylinder_workload(40, 30, 1200, n_points=65_536, near_frac=0.1, seed=5)


@pytest.mark.parametrize("n", [100, 4097, 16_383, 16_384, 16_385, 20_000, 65_535, 65_536])
@pytest.mark.parametrize("dr", [False, True])
def test_potential_with_and_without_field(cyl, n, dr):
    import torch

    ctx = bemc.Context(0)
    ctx.set_rules(cyl.tri_rule, cyl.rect_gl_n, 2.0)  # the list holds the near pairs of 65,536 points
    ctx.set_dr_rules(dr)
    ctx.upload_geometry(cyl.tri, cyl.rect)
    ctx.upload_densities(cyl.sigma)
    pts = torch.tensor(np.ascontiguousarray(cyl.points[:n].T), dtype=torch.float64, device="cuda:0")
    alone, beside = (torch.empty(n, dtype=torch.float64, device="cuda:0") for _ in range(2))
    E = torch.empty((3, n), dtype=torch.float64, device="cuda:0")
    ctx.eval_noalloc(pts, alone)
    st = ctx.stats()
    ctx.eval_noalloc(pts, beside, E)
    ctx.stats()
    ctx.close()
    assert st["near_pairs"] > n  # several near records at many points
    assert torch.equal(alone, beside)
