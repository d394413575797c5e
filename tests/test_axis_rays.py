"""Rays along the axes find every triangle, up to coordinates of 1e15 (the
reciprocal of a zero direction component times a coordinate stays finite), and
small scenes as before (CPU only)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = [os.path.join(ROOT, "tests", "sanitize", "axis_rays_check.cpp"),
       os.path.join(ROOT, "paper_2606_14173_amd", "csrc", "bvh_build.cpp")]


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rays") / "axis_rays_check")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all"] + SRC + ["-o", exe])
    return exe


@pytest.mark.parametrize("size,shift", [(1e-6, 0.0), (0.05, 0.1), (1.0, 300.0), (1e6, 0.0), (4e8, 0.0), (1e12, 0.0),
                                        (1e15, 0.0), (1e5, 1e9)])
def test_every_triangle_is_found(prog, size, shift):
    r = subprocess.run([prog, repr(size), repr(shift)], capture_output=True, text=True, timeout=600)
    print(r.stdout[-2000:], r.stderr[-2000:])
    assert r.returncode == 0 and "lost 0" in r.stdout
