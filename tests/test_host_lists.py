"""What the list operators of the tile kernel work out without a GPU, compiled for the CPU and run under sanitizers."""
import os

from test_host_sanitizers import ROOT, _build, _run

CSRC = os.path.join(ROOT, "paper_2210_07768_amd", "csrc")


def test_a_sign_finds_its_pair_whichever_lane_a_permute_hears(tmp_path):
    exe = _build(tmp_path, "lists_driver", "g++", [os.path.join(ROOT, "tests", "sanitize", "lists_driver.cpp")], extra=["-std=c++17", "-I", CSRC])
    assert _run([exe]).strip() == "ok"
