"""Forms that a rule on sizes chooses, at both sides of it, against the oracle (integers exactly, see test_gpu_parity)."""
import pytest

from paper_2102_04782_amd import workloads as wl
from test_gpu_kernel_edges import on_random_codes

pytestmark = pytest.mark.gpu
by_name = dict(ids=lambda l: l.name)


@pytest.mark.parametrize("layer", [
    wl.Layer("c19", 1, 1100, 66, 66, 1030, 1, 1, 1, 0),      # 19 chunks of a workgroup: addresses made by scalar instructions
    wl.Layer("c20", 1, 1100, 69, 69, 1030, 1, 1, 1, 0),      # 20: by vector instructions
    wl.Layer("c23_s2", 100, 1040, 15, 13, 1050, 1, 1, 2, 0),
], **by_name)
def test_requests_of_the_1x1_filter_gradient(layer):
    on_random_codes(layer, 91)


@pytest.mark.parametrize("layer", [
    wl.Layer("p8", 3, 500, 7, 7, 20, 1, 1, 1, 0),            # eight pairs of row blocks, no whole lines
    wl.Layer("p16", 2, 1000, 5, 9, 33, 1, 1, 1, 0),
    wl.Layer("p27", 2, 1700, 9, 7, 20, 1, 1, 1, 0),
    wl.Layer("p17", 1, 1050, 8, 8, 130, 1, 1, 1, 0),         # whole lines, more than sixteen pairs
    wl.Layer("many", 21, 300, 45, 47, 150, 1, 1, 1, 0),      # more than 128 channels and 48 MiB: two quads
    wl.Layer("many4", 40, 250, 37, 39, 130, 1, 1, 1, 0),     # four pairs: eight quads
], **by_name)
def test_blocks_of_the_streaming_form(layer):
    on_random_codes(layer, 92)


@pytest.mark.parametrize("layer", [
    wl.Layer("whole", 16, 130, 7, 7, 300, 1, 1, 1, 0),       # eight tiles of two images, one after the other in a row tile
    wl.Layer("whole_odd", 9, 200, 9, 9, 290, 1, 1, 1, 0),
    wl.Layer("whole_s2", 7, 150, 13, 15, 100, 1, 1, 2, 0),
    wl.Layer("rows", 2, 70, 16, 16, 300, 1, 1, 1, 0),        # tiles of eight whole rows, on lines
    wl.Layer("rows_s2", 3, 70, 32, 32, 100, 1, 1, 2, 0),
    wl.Layer("shared", 3, 70, 13, 13, 300, 1, 1, 1, 0),      # lines shared: tile after tile
    wl.Layer("ragged", 66, 260, 7, 7, 300, 1, 1, 1, 0),      # 33 tiles, five row tiles: tile after tile
], **by_name)
def test_order_of_128_pixel_tiles(layer):
    on_random_codes(layer, 93)
