"""Workspace layout of the tiled recurrence (host arithmetic, no GPU): the planes each
kind of run takes lie inside the workspace its size query reports."""
import os
import subprocess

import pytest

from paper_2509_06525_amd import build, tbkpm

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not os.path.exists(tbkpm.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("native") / "tile_layout")
    rocm = os.path.dirname(os.path.dirname(build.HIPCC))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.INCLUDE, "-I", build.CSRC, "-I",
                    os.path.join(rocm, "include"), os.path.join(HERE, "native", "tile_layout.cpp"), tbkpm.LIB_PATH,
                    "-Wl,-rpath," + os.path.dirname(tbkpm.LIB_PATH), "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(rocm, "lib"), "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def layouts(program):
    out = subprocess.run([program], check=True, capture_output=True, text=True).stdout
    return [tuple(int(x) for x in line.split()) for line in out.splitlines()]


def test_planes_lie_inside_the_workspace(layouts):
    """kpm_moments (a pair of planes with one vector, five planes otherwise) and stacks of one
    structure and of several (a pair beside the sweep's vectors, whatever their number)."""
    seen = set()
    for n, d, R, f64, onsite, M, segs, sweep, off_planes, total, planes, taken, vec, whole in layouts:
        assert taken <= planes and whole
        assert sweep <= off_planes
        assert off_planes + taken * vec <= total
        seen.add((segs, R))
    assert {(1, 1), (1, 3), (0, 1), (7, 64)} <= seen


def test_a_larger_number_of_moments_never_needs_less(layouts):
    """One buffer sized for the largest M serves every call of a run split over calls."""
    last = {}
    for n, d, R, f64, onsite, M, segs, sweep, off_planes, total, *_ in layouts:
        key = (n, d, R, f64, onsite, segs)
        assert last.get(key, (0, 0))[0] < M and last.get(key, (0, 0))[1] <= total
        last[key] = (M, total)


def test_planes_are_bounded_whatever_the_vectors(layouts):
    """100 M rows: the sweep's workspace, the lists and 32 GB of planes at most."""
    for n, d, R, f64, onsite, M, segs, sweep, off_planes, total, planes, taken, vec, whole in layouts:
        if n == 100000000 and segs == 0 and R > 1:
            assert total - off_planes <= (32 << 30) + 4096
            assert off_planes - sweep <= n * 160 + (64 << 20) + M * R * 64 * 1024


def test_the_static_workspace_is_what_its_runs_take(program):
    """Every run whose sweep kpm_moments_noalloc takes fits its array on tiles, too (the
    same form, so the same sums, as with a caller's workspace), with a few MiB to spare."""
    out = subprocess.run([program, "static"], check=True, capture_output=True, text=True).stdout
    runs, off, most, static = (int(x) for x in out.split())
    assert runs > 100000 and off == 0
    assert static - (8 << 20) < most <= static
