"""The pool of released device blocks: its rules on the host, over a stand-in for the runtime's
allocator (compiled here, no GPU), and that no allocation of the library passes it by."""
import glob
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2511_15028_amd", "csrc")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    from paper_2511_15028_amd._build import HIPCC
    d = tmp_path_factory.mktemp("pool")
    flags = ["-std=c++17", "-O1", "-fPIC", f"-I{os.path.join(HERE, '..', 'include')}", f"-I{CSRC}"]
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", *flags, "-c",
                    os.path.join(CSRC, "workspace.hip"), "-o", str(d / "w.o")], check=True, capture_output=True)
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", *flags, "-c",
                    os.path.join(HERE, "pool_host.cpp"), "-o", str(d / "p.o")], check=True, capture_output=True)
    subprocess.run(["g++", str(d / "p.o"), str(d / "w.o"), "-o", str(d / "pool_host"), "-lpthread"],
                   check=True, capture_output=True)
    out = subprocess.run([str(d / "pool_host")], check=True, capture_output=True, text=True).stdout
    return out.splitlines()


def test_allocations_get_the_idle_blocks(lines):
    assert lines[0] == "kept 400"  # released, and kept for the next builds
    assert lines[1] == "malloc 0 used 900"  # their memory was what was missing
    assert lines[2] == "refused 2 null 1 last 0"  # and the error does not reach the next call


def test_a_device_s_blocks_age_by_its_own_releases(lines):
    assert lines[3] == "ages 10 50"  # 200 releases on device 0 leave device 1's blocks
    assert lines[4] == "aged 10 10"  # 64 of its own do not


def test_trim_gives_one_device_s_blocks_back(lines):
    assert lines[5] == "trimmed 0 10"


@pytest.mark.gpu
def test_trim_after_the_last_handle():
    import torch
    from paper_2511_15028_amd import bvh, workloads as W
    v, t = (torch.from_numpy(x).cuda() for x in W.soup_scene(1_000_000, seed=1))
    h = bvh.build(v, t, "bvh4")  # the work areas have their sizes now
    held = h.stats()["nodes_buffer_bytes"] + h.stats()["leaf_buffer_bytes"]
    h.close()
    bvh.trim()
    before = torch.cuda.mem_get_info()[0]
    bvh.build(v, t, "bvh4").close()
    assert before - torch.cuda.mem_get_info()[0] >= held // 2  # kept for the next build
    bvh.trim()
    assert torch.cuda.mem_get_info()[0] == before


def test_every_device_allocation_is_the_pool_s():
    for path in glob.glob(os.path.join(CSRC, "*")):
        calls = re.findall(r"\bhipMalloc(?:Async)?\(", open(path).read())
        assert len(calls) == (2 if path.endswith("workspace.hip") else 0), path
