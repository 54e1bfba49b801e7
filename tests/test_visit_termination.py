"""A wide traversal ends for every ray: no visit may report an empty child slot as met (its
reference would be taken for an interior node), whatever the ray's floats are.  The layouts' visit
code runs on the host (compiled here, no GPU)."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(HERE, "..", "paper_2511_15028_amd")


@pytest.fixture(scope="module")
def visits(tmp_path_factory):
    from paper_2511_15028_amd._build import HIPCC
    exe = str(tmp_path_factory.mktemp("visit") / "visit_host")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-ffp-contract=off",
                    f"-I{os.path.join(HERE, '..', 'include')}", f"-I{os.path.join(PKG, 'csrc')}",
                    os.path.join(HERE, "visit_host.hip"), "-o", exe], check=True, capture_output=True)
    lines = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    return [line.split() for line in lines]


@pytest.mark.parametrize("layout", ["bvh4", "bvh8_q8", "bvh8_q16"])
def test_no_empty_slot_is_met(visits, layout):
    rows = [(name, int(n), int(empty)) for lay, name, _, _, _, n, _, empty in visits if lay == layout]
    assert len(rows) == 12
    for name, n, empty in rows:
        assert empty == 0, (layout, name)
        assert n <= 2, (layout, name, n)  # the tree has two nodes
    assert dict((name, n) for name, n, _ in rows)["plain"] == 2


def test_rays_that_can_hit_are_finite(visits):
    for _, name, _, finite, _, _, _, _ in visits:
        bad = name.endswith(("nan-direction", "inf-direction", "nan-origin", "inf-origin", "mixed"))
        assert finite == ("0" if bad else "1"), name
