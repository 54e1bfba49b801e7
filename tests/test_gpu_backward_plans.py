"""Vertex gradients at the sizes where the launch plan of the backward pass changes.

Each vertex's gradient is a sum of float32 terms w * lam, one per ray corner; the terms follow from
the hits and the ray gradients, so the reference adds the same terms in float64.  m terms added in
any order in float32 differ from that by at most (m + 1) * 2^-24 times the sum of their magnitudes.
"""
import pytest

from paper_2511_15028_amd import workloads as W
from test_gpu_parity import B, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# one range and 20 ranges in slices; 2^9-vertex ranges with private accumulators and, for few rays,
# a shared one; more than 2^19 vertices with the larger range table and without
@pytest.mark.parametrize("n_tris, n_rays", [(20, 200_003), (1700, 300_000), (1700, 3000),
                                            (100_000, 250_000), (100_000, 100_001),
                                            (190_000, 750_001), (190_000, 20_000)])
def test_vertex_gradients(n_tris, n_rays):
    spread = 0.3 if n_tris < 2000 else 0.03
    v, t = (dev(x) for x in W.soup_scene(n_tris, seed=n_tris, spread=spread))
    rays = dev(W.uniform_rays(n_rays, seed=n_rays))
    h = B().build(v, t, "bvh4")
    hits = h.trace(rays)
    h.close()
    g = torch.randn(n_rays, 3, device="cuda", generator=torch.Generator("cuda").manual_seed(5))
    gv, gr = B().trace_backward(v, t, rays, hits, g)
    prim = B().prim_ids(hits).long()
    hit = prim >= 0
    assert hit.float().mean() > 0.05
    lam, uv = -gr[hit, 0:3], hits[hit, 2:4]
    w = torch.stack(((1.0 - uv[:, 0]) - uv[:, 1], uv[:, 0], uv[:, 1]), 1)
    terms = (w[:, :, None] * lam[:, None, :]).reshape(-1, 3).double()
    at = t[prim[hit]].long().reshape(-1)
    want, size, m = torch.zeros_like(gv, dtype=torch.float64), torch.zeros_like(gv, dtype=torch.float64), \
        torch.zeros(len(v), 1, dtype=torch.float64, device="cuda")
    want.index_add_(0, at, terms)
    size.index_add_(0, at, terms.abs())
    m.index_add_(0, at, torch.ones(len(at), 1, dtype=torch.float64, device="cuda"))
    assert ((gv.double() - want).abs() <= (m + 1) * 2.0 ** -24 * size).all()
