"""Builds that take the device memory of earlier handles, and the SAH build at the sizes where its
levels change shape.

Released blocks go to the next builds, whatever their thread and stream, so every build must give
the bytes that it gives in fresh memory, and what stays allocated must be bounded.  The SAH levels
work in chunks of 2,048 primitives with 64 chunks to a scan step, and nodes of 1,024 leave them: the
trees just above and below those sizes must be the oracle's.
"""
import threading

import numpy as np
import pytest

from paper_2511_15028_amd import workloads as W
from test_gpu_parity import B, check_closest, dev, gpu_trace, oracle_ref
from test_gpu_sah import check_tree

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KEPT = 512 << 20  # what the library may keep of released memory


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 2049, 2048 * 64 + 1, 2048 * 65 + 3])
def test_sah_chunk_edges(orc, n):
    v, t = W.soup_scene(n, seed=n)
    check_tree(orc, v, t, 4)


def buffers(v, t, layout):
    h = B().build(v, t, layout)
    out = h.read_buffer(0), h.read_buffer(1)
    h.close()
    return out


@pytest.mark.parametrize("layout", ["bvh4", "bvh8_q8", "aabb2"])
def test_reused_blocks_give_the_same_bytes(layout):
    meshes = [tuple(dev(x) for x in W.soup_scene(n, seed=n)) for n in (5, 900, 1000, 1100, 40_000)]
    want = [buffers(v, t, layout) for v, t in meshes]
    for k in (3, 1, 4, 0, 2, 1, 3):  # sizes that fit another's block and sizes that do not
        assert buffers(*meshes[k], layout) == want[k]


def test_threads_and_streams_share_released_blocks():
    meshes = [tuple(dev(x) for x in W.soup_scene(n, seed=n)) for n in (2000, 2100, 2200, 2300)]
    want = [buffers(v, t, "bvh4") for v, t in meshes]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for i in range(20):
                j = (k + i) % len(meshes)
                if buffers(*meshes[j], "bvh4") != want[j]:
                    bad.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not bad


def test_kept_memory_is_bounded():
    v, t = (dev(x) for x in W.soup_scene(1_000_000, seed=1))
    B().build(v, t, "bvh4").close()  # the work areas have their sizes now
    handles = [B().build(v, t, "bvh4") for _ in range(12)]
    held = sum(h.stats()["nodes_buffer_bytes"] + h.stats()["leaf_buffer_bytes"] for h in handles)
    assert held > KEPT  # or this test shows nothing
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for h in handles:
        h.close()
    # every allocation may be rounded up to 2 MiB pages
    assert torch.cuda.mem_get_info()[0] - before >= held - KEPT - (2 << 20) * 24



def morton_order(verts, tris, bits):
    """The stable order of the triangles by the Morton key of their boxes' centres, in float32."""
    f, p = np.float32, verts[tris]
    c = f(0.5) * p.min(1) + f(0.5) * p.max(1)
    lo, ext = c.min(0), c.max(0) - c.min(0)
    inv = np.where(ext > 0, f(1) / np.where(ext > 0, ext, f(1)), f(0)).astype(f)
    cells = f(2 ** bits)
    q = np.clip((c - lo) * inv * cells, f(0), cells - f(1)).astype(np.uint64)
    key = np.zeros(len(tris), np.uint64)
    for b in range(bits):
        for a in range(3):
            key |= ((q[:, a] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - a)
    return np.argsort(key, kind="stable")


@pytest.mark.parametrize("layout", ["bvh4", "bvh8_q16", "aabb2"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4095, 4096, 4097])
def test_small_hierarchy(orc, n, layout):
    """The sizes around which the order and hierarchy of a small mesh, made by one workgroup, change
    rows, and where the separate kernels take over."""
    v, t = W.soup_scene(n, seed=90 + n, spread=0.1)
    t = t.copy()
    t[n // 2:n // 2 + 40] = t[0]  # equal keys keep the order of the input
    h = B().build(dev(v), dev(t), layout, 4, "indexed")
    lg = max(1, (n - 1).bit_length())
    bits = max(4, (lg + 2) // 3 + 4)
    if (3 * bits) % 8 in (1, 2, 3):
        bits -= 1
    np.testing.assert_array_equal(np.frombuffer(h.read_buffer(1), np.int32), morton_order(v, t, bits))
    # every triangle is found: the hits are the oracle's
    rays = W.uniform_rays(2000, seed=n)
    prim, tuv = gpu_trace(h, rays)
    check_closest(orc, v, t, rays, prim, tuv, oracle_ref(orc, v, t, rays))
    h.close()
