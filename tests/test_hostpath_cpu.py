"""The library's host path without a GPU: tests/hostpath.cpp stands in for the
HIP runtime, notes the launches of the real libcubestats.so and checks their
order, arguments and memory.  One scenario per test."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1111_6661_amd")


@pytest.fixture(scope="module")
def scenario(tmp_path_factory):
    lib = os.path.join(PKG, "libcubestats.so")
    if not os.path.exists(lib):
        from paper_1111_6661_amd import build
        build.build()
    exe = str(tmp_path_factory.mktemp("hostpath") / "hostpath")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unused-result", "-rdynamic",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "hostpath.cpp"), lib,
                           f"-Wl,-rpath,{PKG}", "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib",
                           "-lpthread"])

    def run(name):
        r = subprocess.run([exe, name], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
    return run


def test_calls_that_share_a_stream_keep_their_launches_together(scenario):
    """Two threads on one stream: the pass and the launch that reads its
    workspace (the rows of many bins, the range of a two-pass call) have no
    other call's launches between them."""
    scenario("shared_stream")


def test_results_in_host_memory_are_written_through(scenario):
    """Also those of a min/max call's first pass, by the second, which says that
    it is done."""
    scenario("host_results")


def test_a_stream_that_ends_without_results_is_an_error(scenario):
    scenario("lost_results")


def test_projections_that_share_a_stream_keep_their_launches_together(scenario):
    scenario("shared_projection")


def test_a_projection_without_room_for_slices_takes_one(scenario):
    scenario("projection_without_partials")


def test_partials_of_a_captured_projection_are_kept(scenario):
    scenario("captured_partials")


def test_images_of_any_size_are_projected_by_quads(scenario):
    scenario("projection_kernels")


def test_small_images_take_one_pixel_per_lane(scenario):
    scenario("projection_slices")


def test_rows_under_four_voxels_are_spread_over_the_chip(scenario):
    scenario("thin_rows")


def test_histograms_of_large_boxes_have_the_copies_that_fit(scenario):
    scenario("histogram_copies")


def test_rows_of_counts_are_allocated_where_they_are_written(scenario):
    scenario("rows_memory")
