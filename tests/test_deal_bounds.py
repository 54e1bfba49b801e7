"""Launches that no fallback pass follows finish every ray in a group of lanes: their reserve must
hold whatever the tree's stack bound lets a ray need.  The launch rule's own code runs on the host
(compiled here, no GPU) against a model of the shared stack."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(HERE, "..", "paper_2511_15028_amd")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    from paper_2511_15028_amd._build import HIPCC
    exe = str(tmp_path_factory.mktemp("deal") / "deal_host")
    subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1",
                    f"-I{os.path.join(HERE, '..', 'include')}", f"-I{os.path.join(PKG, 'csrc')}",
                    os.path.join(HERE, "deal_host.hip"), "-o", exe], check=True, capture_output=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()


def test_groups_without_a_fallback_pass_have_room(lines):
    rows = [tuple(int(x) for x in line.split()) for line in lines[:81]]
    assert any(r[3] > 8 for r in rows)
    for arity, ring, bound, launches, least in rows:
        assert launches == 0 or least >= 0, (arity, ring, bound, least)


def test_no_list_is_written_without_a_fallback_pass(lines):
    assert lines[82] == "list 1 2 5 9 0"


def test_spill_runs_cover_every_ray_and_never_shrink(lines):
    assert lines[81] == "runs 0 0 1"
