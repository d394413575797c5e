"""The 48-byte BVH nodes that the traversal reads (binary16 plane offsets): no
ray loses its closest hit, for scenes from 1e-3 to 1e6 across, at the origin and
far from it, rays along the axes and from far away (CPU only; every box is
rounded outwards, so none may be lost)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = [os.path.join(ROOT, "tests", "sanitize", "packed_nodes_check.cpp"),
       os.path.join(ROOT, "paper_2606_14173_amd", "csrc", "bvh_build.cpp")]


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("nodes") / "packed_nodes_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all"] + SRC + ["-o", exe])
    return exe


@pytest.mark.parametrize("size,shift", [(1.0, 0.0), (1e-3, 0.0), (1e6, 0.0), (1.0, 300.0), (0.02, 3.0), (1e-3, 1e4)])
def test_no_ray_loses_its_closest_hit(prog, size, shift):
    r = subprocess.run([prog, repr(size), repr(shift)], capture_output=True, text=True, timeout=600)
    print(r.stdout[-2000:], r.stderr[-2000:])
    assert r.returncode == 0 and "lost 0" in r.stdout
