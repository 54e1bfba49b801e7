"""Rays with NaN or infinite components end and miss, through every entry point that traces rays, in
launches of few rays and of many, among ordinary rays whose hits stay the oracle's."""
import numpy as np
import pytest

from paper_2511_15028_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LAYOUTS = ["bvh4", "bvh8_q8", "bvh8_q16", "aabb2", "pbrt_q16", "sg_eq", "pbrt_soaos", "pbrt_q16_soaos",
           "sg_eq_a16", "shared_slab"]
INF, NAN = np.inf, np.nan
BAD = [((0.5, 0.5, 0.5), (NAN, NAN, NAN)), ((0.5, 0.5, 0.5), (INF, INF, INF)),
       ((0.5, 0.5, 0.5), (-INF, INF, -INF)), ((NAN, NAN, NAN), (0.0, 0.0, 1.0)),
       ((INF, INF, INF), (-1.0, -1.0, -1.0)), ((0.5, NAN, 0.5), (0.0, 1.0, 0.0)),
       ((0.5, 0.5, 0.5), (INF, 0.0, 1.0)), ((0.5, 0.5, 0.5), (0.0, 0.0, 0.0))]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def scene(orc):
    v, t = W.soup_scene(1500, seed=41, spread=0.1)
    rays = W.uniform_rays(20011, seed=42)
    at = np.arange(0, 20011, 97)
    for k, i in enumerate(at):
        rays[i, 0:3], rays[i, 4:7] = BAD[k % len(BAD)]
    prim, _ = orc.brute_closest(v, t, rays)
    assert (prim[at] == -1).all() and (prim >= 0).any()
    return dev(v), dev(t), dev(np.tile(rays, (6, 1))), np.tile(prim, 6)


@pytest.mark.parametrize("n", [1, 200, 20011, 6 * 20011])
@pytest.mark.parametrize("layout", LAYOUTS)
def test_nonfinite_rays_miss(scene, layout, n):
    from paper_2511_15028_amd import bvh
    v, t, rays, prim = scene
    h = bvh.build(v, t, layout, leaf_size=2)
    r = rays[:n]
    ids = [h.trace(r), h.trace_counts(r)[0]]
    if layout != "shared_slab":
        ids.append(h.trace_noalloc(r, torch.empty_like(r[:, :4])))
    for hits in ids:
        assert np.array_equal(bvh.prim_ids(hits).cpu().numpy(), prim[:n])
    occluded = bvh.prim_ids(h.trace(r, bvh.TRACE_ANY)).cpu().numpy() >= 0
    assert np.array_equal(occluded, prim[:n] >= 0)
    h.close()


@pytest.mark.parametrize("layout", LAYOUTS[:-1])
def test_nonfinite_rays_miss_in_a_batch(scene, layout):
    from paper_2511_15028_amd import bvh
    v, t, rays, prim = scene
    b = bvh.Batch([(v, t), (v, t)], layout=layout, stack_lds=16)
    hits = b.trace(rays, [0, 5000, 6 * 20011])
    assert np.array_equal(bvh.prim_ids(hits).cpu().numpy(), prim)
    b.close()
