"""Host checks of the LDS geometry of the matrix-core kernels (compiled with the host compiler, no GPU)."""
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build_and_run(name):
    src = os.path.join(ROOT, "tests", "host_checks", name + ".cpp")
    with tempfile.TemporaryDirectory() as tmp:
        exe = os.path.join(tmp, name)
        subprocess.run(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(ROOT, "paper_2409_09083_amd", "csrc"), src, "-o", exe], check=True)
        out = subprocess.run([exe], capture_output=True, text=True)
        assert out.returncode == 0, out.stdout
        assert out.stdout.startswith("ok")


def test_wgrad_chunks_fit_their_lds_limits():
    _build_and_run("chunk_check")


def test_conv_tiles_fit_their_lds_limits_and_cover_every_pixel_once():
    _build_and_run("conv_tile_check")


def test_first_layer_tiles_fit_their_lds_limits():
    _build_and_run("stem_tile_check")


def test_orders_of_workgroups_name_each_once_and_load_the_xcds_evenly():
    _build_and_run("order_check")


def test_quotients_by_reciprocals_are_exact():
    _build_and_run("quot_check")


def test_large_launches_are_told_from_small_ones_before_they_are_cut():
    _build_and_run("small_launch_check")


def test_direct_16_bit_gradients_multiply_every_pixel_once():
    _build_and_run("wgrad16_walk_check")


def test_rows_of_narrow_maps_of_any_height_are_exact():
    _build_and_run("quot_rows_check")
