"""The tree as the device walks it, on the host with the device's arithmetic:
no reference may leave the scene's part of the pools, however far away a ray
starts and whatever its direction.  From about 1e37 on, a box the wrong way
round (an empty child slot's) is one distance like every other, and its slot
is entered; so it is with an infinite direction."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from neb_inputs import scenes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1909_00573_amd", "csrc")


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("walk")
    exe = str(d / "bvh_walk_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "bvh_walk_check.cpp"), os.path.join(CSRC, "neb_bvh.cpp"),
                    "-o", exe], check=True)

    def run(vertices, tris, rays, *args):
        path = str(d / "mesh.bin")
        with open(path, "wb") as f:
            np.array([len(vertices), len(tris)], dtype=np.int32).tofile(f)
            np.ascontiguousarray(vertices, dtype=np.float32).tofile(f)
            np.ascontiguousarray(tris, dtype=np.int32).tofile(f)
        out = subprocess.run([exe, path, str(rays), *map(str, args)], check=True, capture_output=True, text=True)
        return {k: int(v) for k, v in (kv.split("=") for kv in out.stdout.split())}
    return run


def test_from_inside(walk):
    sc = scenes.tiny_box()
    r = walk(sc.vertices, sc.tris, 3000, -1, 0)
    assert r["hits"] > 2500 and r["differing"] == r["outside"] == r["empty"] == 0


@pytest.mark.parametrize("infinite", [0, 1])
@pytest.mark.parametrize("far", [0, 5, 30, 36, 37, 38, 38.5])
def test_from_far_away(walk, far, infinite):
    sc = scenes.tiny_box()
    r = walk(sc.vertices, sc.tris, 300, far, infinite)
    assert r["outside"] == r["differing"] == 0
    assert r["hits"] == 0 or (far < 30 and not infinite)
    if far >= 38 or infinite:
        assert r["empty"] > 0  # the case this test is about
