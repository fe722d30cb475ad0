"""Host checks of the fp32 kernels on the bfloat matrix cores (no GPU)."""
from tests.test_chunks_host import _build_and_run


def test_split_patches_fit_their_lds_area():
    _build_and_run("split_tile_check")


def test_split_filter_gradient_chunks_fit_and_cover():
    _build_and_run("wsplit_check")
