"""The traversal's quantized node on the CPU: the source the kernels are built
from, compiled for the host, checked in extended precision (nodeq_host.cpp).
Rejecting a box that the ray enters loses its hits, so planes must lie outside
their boxes by what the walk's arithmetic rounds."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_22780_amd", "csrc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("nodeq")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text("#pragma once\n")  # the harness brings what the header takes from it
    exe = d / "nodeq_host"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", str(d), "-I", CSRC, "-o", str(exe),
                    os.path.join(HERE, "nodeq_host.cpp")], check=True)

    def run(name):
        words = subprocess.run([str(exe), name], check=True, capture_output=True, text=True).stdout.split()
        return dict(zip(words[::2], map(int, words[1::2])))

    return run


def test_planes_lie_outside_their_boxes(host):
    """Also far from the origin, where a node is a few units in the last place
    of its coordinates long; and with infinite or NaN corners."""
    r = host("planes")
    assert r["planes"] > 300_000
    assert r["inside"] == 0 and r["wide"] == 0, r


def test_slack_covers_the_roundings(host):
    """Rays that meet a box's near plane of one axis and its far plane of
    another at the same depth, with every rounding of the two against them."""
    r = host("slack")
    assert r["pairs"] > 100
    assert r["lost"] == 0 and r["kept"] == 0, r
