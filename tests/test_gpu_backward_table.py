"""Vertex gradients of meshes whose range table is the large one (more than 2^19 vertices, many rays),
with two counters to a word: blocks whose rays all hit one triangle, in a range at either end of a
word or in the last one, and blocks whose rays hit all ranges.

The triangles share no vertex, so the three gradients of a triangle add up to the sum of lam = -dL/do
over its rays, whatever their u and v.  With u, v and 1 - u - v in [0, 1] (the points are chosen
inside), m float32 terms per vertex are within (m + 1) * 2^-24 of their magnitudes' sum, and the three
weights within 4 * 2^-24 of 1."""
import numpy as np
import pytest

from paper_2511_15028_amd import workloads as W
from test_gpu_parity import B, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TRIS, RAYS = 180_001, 1024 * 700 + 13


@pytest.mark.parametrize("which", ["all", "first", "odd", "last"])
def test_large_range_table(which):
    v, t = W.soup_scene(TRIS, seed=71, spread=0.05)
    rng = np.random.default_rng(72)
    prim = {"first": np.zeros(RAYS, np.int32), "odd": np.full(RAYS, 3 * 512 // 3, np.int32),
            "last": np.full(RAYS, TRIS - 1, np.int32), "all": rng.integers(0, TRIS, RAYS).astype(np.int32)}[which]
    w = rng.dirichlet((2.0, 2.0, 2.0), RAYS)
    p = (v[t[prim]].astype(np.float64) * w[:, :, None]).sum(1)
    d = rng.normal(size=(RAYS, 3))
    rays = np.zeros((RAYS, 8), np.float32)
    rays[:, 0:3], rays[:, 4:7], rays[:, 7] = p - d, d, np.inf
    hits = np.zeros((RAYS, 4), np.float32)
    hits[:, 0] = prim.view(np.float32)
    dv, dt = dev(v), dev(t)
    g = torch.randn(RAYS, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(73))
    gv, gr = B().trace_backward(dv, dt, dev(rays), dev(hits), g)
    # the reference is summed on the host: float64 atomics of all rays on one address do not end in time
    lam = -gr[:, 0:3].cpu().numpy().astype(np.float64)

    def per_triangle(x):
        return np.stack([np.bincount(prim, x[:, c], TRIS) for c in range(3)], 1)

    want, size = per_triangle(lam), per_triangle(np.abs(lam))
    m = np.bincount(prim, minlength=TRIS)[:, None]
    got = gv.cpu().numpy().astype(np.float64)[t].sum(1)
    assert (lam != 0).any(1).mean() > 0.99  # few of the systems are singular
    assert (np.abs(got - want) <= (3 * (m + 1) + 4) * 2.0 ** -24 * size).all()
