"""Launch shapes of the traversal, on the host: rays are dealt out, and grids
sized for it, only where the kernel launched can deal (pools of at most 4 GB,
frames of at most 65 536 pixels); grids never leave a wave less than eight rays
of a dealt queue or less than one per lane of another."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1909_00573_amd", "csrc")
FOUR_GB = 1 << 32


@pytest.fixture(scope="module")
def shape(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("shape") / "trace_shape_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "host", "trace_shape_check.cpp"),
                    "-o", exe], check=True)

    def ask(*line):
        out = subprocess.run([exe], input=" ".join(map(str, line)), check=True, capture_output=True, text=True)
        return out.stdout.split()
    return ask


@pytest.mark.parametrize("npix,nodes,tris,deals", [
    (1, 128, 48, 1), (65536, 128, 48, 1), (65537, 128, 48, 0), (4096, FOUR_GB - 1, FOUR_GB - 1, 1),
    (4096, FOUR_GB, 48, 0), (4096, 128, FOUR_GB, 0), (1 << 20, FOUR_GB, FOUR_GB, 0)])
def test_deals_where_the_kernel_does(shape, npix, nodes, tris, deals):
    assert shape("deals", npix, nodes, tris) == [str(deals)]


@pytest.mark.parametrize("cap,bpc,deals,blocks", [
    (4096, 8, 0, 64), (4097, 8, 0, 65), (4096, 8, 1, 512), (4089, 8, 1, 512), (4088, 8, 1, 511), (1 << 20, 8, 1, 2048), (1, 8, 1, 1),
    (0, 8, 0, 1), (1 << 20, -1, 0, 256 * 16), (1 << 20, 20, 0, 256 * 16), (4096, 0, 0, 64), (4096, 0, 1, 64),
    (1 << 27, 0, 0, 1 << 20)])
def test_blocks(shape, cap, bpc, deals, blocks):
    assert shape("blocks", 256, cap, bpc, 16, deals) == [str(blocks)]


@pytest.mark.parametrize("stack,accepted", [(32, 20), (48, 13), (64, 10)])
def test_resident_blocks_fit(shape, stack, accepted):
    lds, resident, named = map(int, shape("lds", stack))
    # stacks and 20 bytes a lane for shared rays
    assert lds == stack * 256 + 1280 and lds * resident <= 160 * 1024 < lds * (resident + 1)
    assert named == accepted  # what configurations could name before rays were shared
