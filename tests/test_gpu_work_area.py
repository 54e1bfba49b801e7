"""The work area of a trace is never larger for fewer rays: a call that has been made warms its
stream up for every smaller one, also under capture (where an area cannot grow)."""
import numpy as np
import pytest

from paper_2511_15028_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def test_capture_of_fewer_rays_after_a_larger_call():
    from paper_2511_15028_amd import bvh
    v, t = W.soup_scene(1500, seed=53)
    h = bvh.build(dev(v), dev(t), "bvh4")
    # counts around which the rays per wave, and with them the grid, change
    big, sizes = 5121 + 4096, (5120, 4097, 4096, 1000)
    rays = dev(W.uniform_rays(big, seed=54))
    hits = torch.empty((big, 4), device="cuda")
    counts = torch.empty((big, 2), dtype=torch.int32, device="cuda")
    s = torch.cuda.Stream()

    def call(n):
        assert bvh.lib().bvh_trace_counts(h.handle, rays.data_ptr(), n, hits.data_ptr(), 0,
                                          counts.data_ptr(), s.cuda_stream) == bvh.OK

    with torch.cuda.stream(s):
        call(big)
        s.synchronize()
        want = hits.clone()
        for n in sizes:
            g = torch.cuda.CUDAGraph()
            s.synchronize()
            with torch.cuda.graph(g, stream=s):
                call(n)
            for _ in range(3):  # replays, with work of the program's own between them
                hits.fill_(7.0)
                g.replay()
                s.synchronize()
                assert torch.equal(hits[:n].view(torch.int32), want[:n].view(torch.int32))
                assert (hits[n:] == 7.0).all()
    h.close()
