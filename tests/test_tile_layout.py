"""Workspace layout of the tiled recurrence (host arithmetic, no GPU): the planes each
kind of run takes lie inside the workspace its size query reports."""
import os
import subprocess

import pytest

from paper_2509_06525_amd import build, tbkpm

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def layouts(tmp_path_factory):
    if not os.path.exists(tbkpm.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("native") / "tile_layout")
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.INCLUDE, "-I", build.CSRC, "-I",
                    os.path.join(rocm, "include"), os.path.join(HERE, "native", "tile_layout.cpp"), tbkpm.LIB_PATH,
                    "-Wl,-rpath," + os.path.dirname(tbkpm.LIB_PATH), "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [tuple(int(x) for x in line.split()) for line in out.splitlines()]


def test_planes_lie_inside_the_workspace(layouts):
    """kpm_moments (two planes with one vector, six otherwise) and stacks of one structure
    and of several (five, whatever the vectors)."""
    seen = set()
    for n, d, R, f64, onsite, M, segs, sweep, off_planes, total, planes, taken, vec, whole in layouts:
        assert taken <= planes and whole
        assert sweep <= off_planes
        assert off_planes + taken * vec <= total
        seen.add((segs, R))
    assert {(1, 1), (1, 3), (0, 1), (7, 64)} <= seen
