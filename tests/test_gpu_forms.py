"""Forms that a rule on sizes chooses, at both sides of it, against the oracle (integers exactly, see test_gpu_parity)."""
import numpy as np
import pytest
import torch

from paper_2102_04782_amd import binding as daq
from paper_2102_04782_amd import workloads as wl
from test_gpu_kernel_edges import on_random_codes
from test_gpu_parity import close, descs, dev, ref, t

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


@pytest.mark.parametrize("layer", [
    wl.Layer("eights", 16, 1600, 16, 16, 260, 1, 1, 1, 0),   # sixteen tiles of an image
    wl.Layer("left_over", 44, 1500, 14, 14, 260, 1, 1, 1, 0),   # 44 tiles, 1056 workgroups: five eights and four
    wl.Layer("rows", 5, 1500, 48, 32, 260, 1, 1, 1, 0),      # tiles of eight whole rows
    wl.Layer("pieces", 2, 1500, 48, 48, 260, 1, 1, 1, 0),    # nine tiles of 16 x 16 an image
    wl.Layer("few", 18, 1500, 14, 14, 260, 1, 1, 1, 0),      # 18 tiles, 432 workgroups: an eighth to each XCD
], **by_name)
def test_order_of_256_pixel_tiles(layer):
    on_random_codes(layer, 97)


def codes_of(layer, seed):
    rng = np.random.default_rng(seed)
    q = [rng.integers(-127, 128, shape).astype(np.int8) for shape in (layer.x_shape, layer.w_shape, layer.y_shape)]
    return (*q, (10.0 ** rng.uniform(-4, -1, layer.Cout)).astype(np.float32))


@pytest.mark.parametrize("layer", [
    wl.Layer("w1", 33, 4065, 9, 15, 272, 1, 1, 1, 0),        # 2112 workgroups of a 1 x 1 filter: waves of 32 rows x 128 pixels
    wl.Layer("wt", 33, 1009, 9, 15, 20, 1, 3, 1, 0),         # run-time tap list, one chunk
    wl.Layer("wt_chunks", 33, 1009, 9, 15, 80, 1, 3, 1, 0),
    wl.Layer("t9_256", 16, 1009, 9, 15, 80, 3, 3, 1, 1),
], **by_name)
def test_bf16_results_of_the_wide_waves(layer):
    d, rd = descs(layer)
    _, qW, qG, _ = codes_of(layer, 94)
    s_g, s_w = (torch.tensor([v], dtype=torch.float32, device=dev()) for v in (0.03, 0.11))
    got = torch.full(d.x_shape, float("nan"), dtype=torch.bfloat16, device=dev())
    daq.conv_bwd_data_int8_bf16(d, t(daq.layout_qg(d).pack(qG)), s_g, t(daq.layout_qw(d).pack(d, qW)), s_w, dX=got)
    torch.cuda.synchronize()
    want = ref.conv_bwd_data_int8_bf16(rd, qG, 0.03, qW, 0.11)
    assert np.array_equal(got.view(torch.int16).cpu().numpy().view(np.uint16), want)


@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("stride", [1, 2])
def test_filter_gradient_results_at_any_element(shift, stride):
    """3 x 3, complete tiles of a channel count that allows four results at a time: only where the result begins on 16 bytes."""
    layer = wl.Layer("dW", 1, 64, 7 * stride, 7 * stride, 40, 3, 3, stride, 1)
    d, rd = descs(layer)
    qX, _, qG, s_c = codes_of(layer, 95)
    buf = torch.full((shift + int(np.prod(layer.w_shape)) + 4,), 7.0, device=dev())
    dW = buf[shift:shift + int(np.prod(layer.w_shape))].view(layer.w_shape)
    daq.conv_bwd_filter_int8(d, t(daq.layout_qx_cnhw(d).pack(qX)), torch.tensor([2.5], device=dev()), t(daq.layout_vq(d).pack(qG)), t(s_c), dW=dW)
    torch.cuda.synchronize()
    close(dW.cpu().numpy(), ref.conv_bwd_filter_int8(rd, qX, 2.5, qG, s_c)[0], "dW")
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + dW.numel():] == 7).all())


@pytest.mark.parametrize("layer", [
    wl.Layer("odd", 33, 700, 17, 19, 70, 1, 1, 2, 0),
    wl.Layer("odd_columns", 12, 1000, 34, 37, 65, 1, 1, 2, 0),
    wl.Layer("odd_lines", 12, 1000, 37, 34, 65, 1, 1, 2, 0),
], **by_name)
def test_strided_1x1_products_on_odd_rows(layer):
    on_random_codes(layer, 96)
