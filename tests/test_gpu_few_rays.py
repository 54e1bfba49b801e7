"""Launches of few rays and the last rays of a wave, which the lanes of a wave
finish together.

The hits are compared bit for bit with the exhaustive oracle (closest hit) and
with its occlusion (any hit); closest points on a soup, where no two triangles
tie, with the counting call, which answers every query in a lane of its own.
The ray counts lie around the steps of the group size (1 to 16 rays per wave),
around one chunk of 64 and above the rays that one launch spreads thin."""
import numpy as np
import pytest

from paper_2511_15028_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COUNTS = (1, 2, 5, 63, 65, 1000, 4097, 20011)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def scene(orc):
    v, t = W.soup_scene(1500, seed=31, spread=0.1)
    rays = np.concatenate([W.uniform_rays(15000, seed=32), W.shadow_rays(5011, seed=33)])
    rays[7, 7] = np.float32("nan")   # accepts no hit
    rays[11, 4:7] = (0.0, 0.0, 1.0)  # the two-rounding slab distances
    prim, tuv = orc.brute_closest(v, t, rays)
    return dev(v), dev(t), dev(rays), prim, tuv


@pytest.mark.parametrize("stack_lds", [8, 16, 32])
@pytest.mark.parametrize("layout", ["aabb2", "bvh4", "bvh8_q8", "bvh8_q16", "pbrt_q16", "sg_eq_a16",
                                    "pbrt_q16_soaos"])
def test_few_rays_match_oracle(scene, layout, stack_lds):
    from paper_2511_15028_amd import bvh
    v, t, rays, prim, tuv = scene
    h = bvh.build(v, t, layout, leaf_size=2, stack_lds=stack_lds)
    for n in COUNTS:
        for hits in (h.trace(rays[:n]), h.trace_noalloc(rays[:n], torch.empty_like(rays[:n, :4]))):
            got = hits.cpu().numpy()
            assert np.array_equal(got[:, 0].view(np.int32), prim[:n]), (layout, n)
            assert np.array_equal(got[:, 1:].view(np.uint32), tuv[:n].view(np.uint32)), (layout, n)
        occluded = bvh.prim_ids(h.trace(rays[:n], bvh.TRACE_ANY)).cpu().numpy() >= 0
        assert np.array_equal(occluded, prim[:n] >= 0), (layout, n)
    h.close()


@pytest.mark.parametrize("leaf_mode", ["compact", "indexed"])
@pytest.mark.parametrize("layout", ["aabb2", "bvh4", "bvh8_q8", "pbrt_q16"])
def test_few_queries_match_counting_call(layout, leaf_mode):
    from paper_2511_15028_amd import bvh
    v, t = W.soup_scene(1500, seed=31, spread=0.05)
    q = W.box_points(20011, (0, 0, 0), (1, 1, 1), seed=34)
    q[::3, 3] = np.float32(0.01)     # bounded queries
    q[5, 0] = np.float32("nan")      # and dead ones
    q[6, 3] = np.float32(-1.0)
    h = bvh.build(dev(v), dev(t), layout, leaf_mode=leaf_mode)
    dq = dev(q)
    ref = h.closest_point_counts(dq)[0].cpu().numpy().view(np.uint32)
    for n in COUNTS:
        got = h.closest_point(dq[:n]).cpu().numpy().view(np.uint32)
        assert np.array_equal(got, ref[:n]), (layout, n)
    h.close()


def test_few_rays_on_a_scene_without_triangles():
    from paper_2511_15028_amd import bvh
    v, t = W.soup_scene(3, seed=1)
    for layout in ("aabb2", "bvh4"):
        h = bvh.build(dev(v), dev(t[:0]), layout)
        got = h.trace(dev(W.uniform_rays(17, seed=2))).cpu().numpy()
        assert (got[:, 0].view(np.int32) == -1).all() and np.isinf(got[:, 1]).all()
        near = h.closest_point(dev(W.box_points(17, (0, 0, 0), (1, 1, 1), seed=3)))
        assert (bvh.prim_ids(near).cpu().numpy() == -1).all()
        h.close()
