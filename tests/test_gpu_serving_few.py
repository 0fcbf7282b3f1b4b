"""A served batch of at most 64 points keeps one wavefront of a far workgroup's four busy: with the
rules by distance ratio it takes clearly less time than one of 256 points (the others only help to
stage the elements; when they summed the coarsest level for no point, both took the same)."""
import numpy as np
import pytest

import oracle
from paper_1606_03743_amd import bemc, workloads as W

pytestmark = pytest.mark.gpu


def test_short_batches_do_no_work_for_missing_points():
    tri, rect = W.cylinder(1.0, -5.0, 5.0, 350, 300, 90_000)
    rng = np.random.default_rng(5)
    sigma = rng.standard_normal(len(tri) + len(rect))
    r, a, z = 0.5 * rng.random(256), 2.0 * np.pi * rng.random(256), rng.uniform(-4.0, 4.0, 256)
    pts = np.ascontiguousarray(np.stack([r * np.cos(a), r * np.sin(a), z], 1))  # no near pairs
    ctx = bemc.Context(0)
    ctx.set_dr_rules(True)
    ctx.upload_geometry(tri, rect)
    ctx.upload_densities(sigma)
    ctx.server_start(mem_budget_bytes=1 << 30, max_batch_points=1 << 12, n_streams=2, precision="fp64",
                     small_query_points=0)
    took, out = {}, {}
    for _ in range(12):
        for n in (64, 256):
            phi, E = np.empty(n), np.empty((n, 3))
            i = ctx.server_wait(ctx.server_submit(pts[:n], phi, E))
            took[n] = min(took.get(n, np.inf), i["end_s"] - i["submit_s"])
            out[n] = (phi, E)
    ctx.server_stop()
    ctx.close()
    ref = oracle.evaluate(tri, rect, sigma, pts, oracle.params(33, 7, dr_rules=True), with_abs=True)
    for n, (phi, E) in out.items():
        assert np.max(np.abs(phi - ref["phi"][:n]) / ref["abs_phi"][:n]) <= 1e-12
        assert np.max(np.sum(np.abs(E - ref["E"][:n]), axis=1) / ref["abs_E"][:n]) <= 1e-12
    # 1.63 against 2.32 ms on 1,000,000 elements: 0.70; 0.98 before
    print(f"64 points {1e3 * took[64]:.3f} ms, 256 points {1e3 * took[256]:.3f} ms")
    assert took[64] <= 0.88 * took[256], took
