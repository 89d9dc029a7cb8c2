"""Sizes at which a kernel's loop or a dispatch rule turns over, against the oracle (integers exactly, see test_gpu_parity)."""
import numpy as np
import pytest
import torch

from paper_2102_04782_amd import binding as daq
from paper_2102_04782_amd import workloads as wl
from test_gpu_parity import check_forward, check_quantize_grad, check_quantize_grad_bf16, run_convs_on_codes

pytestmark = pytest.mark.gpu


def on_random_codes(layer, seed):
    rng = np.random.default_rng(seed)
    qX = rng.integers(-127, 128, layer.x_shape).astype(np.int8)
    qW = rng.integers(-127, 128, layer.w_shape).astype(np.int8)
    qG = rng.integers(-127, 128, layer.y_shape).astype(np.int8)
    s_c = (10.0 ** rng.uniform(-4, -1, layer.Cout)).astype(np.float32)
    run_convs_on_codes(layer, qX, qW, qG, 2.5, 0.11, 0.03, s_c)


@pytest.mark.parametrize("batch", [1, 4, 8, 12, 16, 20, 24])
@pytest.mark.parametrize("stride", [1, 2])
def test_filter_gradient_ring_remainders(batch, stride):
    """3 x 3: one to seven 256-byte chunks of the flat axis, all in one workgroup: whole rounds of the load ring and every
    remainder."""
    on_random_codes(wl.Layer("ring", batch, 20, 7 * stride, 7 * stride, 24, 3, 3, stride, 1), 40 + batch)


@pytest.mark.parametrize("stride,width", [(1, w) for w in (*range(14, 30), 1, 2, 3, 121, 122, 123)] + [(2, w) for w in (*range(28, 60, 2), 1, 3, 105, 106, 107)])
def test_filter_gradient_row_pitches(stride, width):
    """3 x 3: rows of every length modulo 16 (a loop of its own each), the shortest, and the longest that the staged rows hold and one more."""
    on_random_codes(wl.Layer("pitch", 2, 35, 6 * stride, width, 33, 3, 3, stride, 1), 300 + width)


@pytest.mark.parametrize("layer", [
    wl.Layer("t3x5", 6, 160, 20, 20, 96, 3, 3, 1, 1),        # 15 tiles: 17 splits fill the chip, 18 would need a second round
    wl.Layer("t1x1_odd", 5, 200, 17, 17, 344, 1, 1, 1, 0),   # 24 tiles of 64 x 64
    wl.Layer("t130", 2, 416, 10, 10, 320, 3, 3, 1, 1),       # 130 tiles: two rounds cannot pay, one split
], ids=lambda l: l.name)
def test_filter_gradient_splits(layer):
    on_random_codes(layer, 77)


@pytest.mark.parametrize("layer", [
    wl.Layer("one", 1, 1, 1, 1, 1, 1, 1, 1, 0),             # one element of everything
    wl.Layer("tile_less1", 2, 31, 9, 9, 33, 3, 3, 1, 1),    # one short of a 32-channel tile, one past it
    wl.Layer("tile_past", 2, 65, 6, 6, 32, 1, 1, 1, 0),     # a second 64-channel block of the contraction axis
    wl.Layer("two_taps", 3, 40, 7, 7, 70, 1, 2, 1, 0),
    wl.Layer("ten_taps", 2, 33, 8, 12, 34, 2, 5, 1, 2),     # three chunks of three taps and one of one
    wl.Layer("stem", 2, 3, 15, 15, 33, 7, 7, 2, 3),         # 49 taps: sixteen chunks of three, one of one
    wl.Layer("grouped", 2, 36, 6, 8, 54, 3, 3, 1, 1, groups=2),
    wl.Layer("depthwise", 2, 33, 5, 6, 33, 3, 3, 2, 1, groups=33),
], ids=lambda l: l.name)
@pytest.mark.parametrize("schedule", [None, daq.SCHEDULE_EARLY_COPY])
def test_forward_quantization_tiles(layer, schedule):
    """q(W) in all arrangements and both copies of q(X), byte for byte."""
    check_forward(layer, 91, schedule)


@pytest.mark.parametrize("layer", [
    wl.Layer("both_narrow", 2, 16, 9, 10, 20, 3, 3, 1, 1),       # one contraction chunk, at most 32 result channels
    wl.Layer("both_chunk", 3, 48, 11, 12, 40, 3, 3, 1, 1),       # one chunk, 64-row tiles
    wl.Layer("both_taps9", 4, 70, 9, 15, 130, 3, 3, 1, 1),       # several chunks
    wl.Layer("both_split", 24, 33, 14, 13, 65, 3, 3, 1, 1),      # the filter gradient split, its reduction a launch of its own
    wl.Layer("both_1x1", 3, 100, 9, 9, 150, 1, 1, 1, 0),
    wl.Layer("both_1x1_chunk", 4, 40, 10, 11, 50, 1, 1, 1, 0),
    wl.Layer("both_1x1_s2", 3, 40, 13, 12, 90, 1, 1, 2, 0),
    wl.Layer("both_248", 31, 60, 32, 16, 24, 3, 3, 1, 1),        # 62 tiles of the data gradient
    wl.Layer("both_past", 62, 60, 32, 32, 24, 3, 3, 1, 1),       # 248: the last one to have room beside it
], ids=lambda l: l.name)
def test_both_gradients_of_a_small_layer(layer):
    on_random_codes(layer, 55)


@pytest.mark.parametrize("kH,kW,pad,stride", [(1, 2, 0, 1), (2, 2, 1, 1), (5, 1, 0, 1), (2, 3, 1, 2), (7, 1, 2, 1), (2, 4, 1, 1), (2, 5, 0, 1), (4, 7, 2, 1),
                                              (5, 6, 2, 1), (7, 7, 3, 2)])
@pytest.mark.parametrize("batch", [1, 5, 13])
def test_filter_gradient_of_any_extent(kH, kW, pad, stride, batch):
    """Tap counts at both sides of the kernel's forms; K steps from fewer than the load ring holds to several rounds of it."""
    on_random_codes(wl.Layer("taps", batch, 3 if kH == 7 and kW == 7 else 20, 12, 11, 70, kH, kW, stride, pad), 60 + batch)


# (images, rows, columns) by the load units - four elements, the last of a plane fewer - that the resident quantizer gives a
# thread: planes of 1, 2 and 3 mod 4 elements, and of fewer than four
RESIDENT_PLANES = {
    2: [(5, 13, 13), (7, 10, 13), (6, 7, 13), (9, 1, 2), (11, 1, 3), (3, 1, 5)],
    4: [(50, 13, 13), (70, 10, 13), (95, 7, 13)],
    8: [(100, 13, 13), (130, 10, 13), (190, 7, 13)],
    16: [(200, 13, 13), (260, 10, 13), (370, 7, 13)],
}


@pytest.mark.parametrize("per_thread,n,h,w", [(u, *p) for u, planes in RESIDENT_PLANES.items() for p in planes])
@pytest.mark.parametrize("k", [1, 3])
def test_resident_quantizer_on_planes_of_any_size(per_thread, n, h, w, k):
    """Codes straight from registers (1 x 1: no padding in the plane) and through the image in LDS (3 x 3)."""
    units = n * -(-h * w // 4)
    assert units <= per_thread * 1024 and (per_thread == 2 or units > per_thread * 512)
    layer = wl.Layer("resident", n, 1, h, w, 128, k, k, 1, k // 2)   # (so many that the largest are not left to the sweeps)
    dY = wl.make_dY(layer, wl.seed_for(21, n))
    st = wl.make_state(dY, wl.seed_for(21, n))
    for mode, seed in ((daq.ROUND_NEAREST, 0), (daq.ROUND_STOCHASTIC, 31 + n)):
        check_quantize_grad(layer, dY, st, mode=mode, seed=seed)
        check_quantize_grad_bf16(layer, dY, st, mode=mode, seed=seed)


# Channel counts by the groups of 16 that the counting pass gives a workgroup's waves, in blocks of up to four: one to three groups
# (several tiles at a time), whole blocks, last blocks of one and of two groups
@pytest.mark.parametrize("channels", [9, 24, 48, 90, 144, 190, 208, 330])
@pytest.mark.parametrize("n,h,w", [(5, 8, 8), (3, 7, 7), (4, 6, 9), (9, 1, 3), (3, 7, 6), (5, 4, 10), (4, 6, 2)], ids=lambda v: str(v))
@pytest.mark.parametrize("schedule", [daq.SCHEDULE_THREE_SWEEPS, daq.SCHEDULE_EARLY_COPY])
def test_counting_pass_units_and_blocks(channels, n, h, w, schedule):
    """Planes of whole units of four, with a shorter last unit, and of less than one; rows of whole units, even and odd ones; both copies byte for byte, with guessed classes
    that hold and (lambda 0 and 1) that do not."""
    for k in (1, 3):
        layer = wl.Layer("units", n, 1, h, w, channels, k, k, 1, k // 2)
        dY = wl.make_dY(layer, wl.seed_for(22, channels))
        st = wl.make_state(dY, wl.seed_for(22, channels))
        for mode, seed, lam in ((daq.ROUND_NEAREST, 0, 0.3), (daq.ROUND_STOCHASTIC, 7 + n, 0.0), (daq.ROUND_STOCHASTIC, 8 + n, 1.0)):
            check_quantize_grad(layer, dY, st, lam=lam, mode=mode, seed=seed, schedule=schedule)


@pytest.mark.parametrize("n,h,w", [(3, 7, 6), (5, 4, 10), (4, 6, 2), (2, 9, 14), (3, 5, 7), (3, 6, 3)], ids=lambda v: str(v))
@pytest.mark.parametrize("channels", [3, 40, 90])
def test_forward_early_copy_of_rows_off_the_units(channels, n, h, w):
    """Units that run on into the next row: after two pixels, after any number, over several rows."""
    for k in (1, 3):
        check_forward(wl.Layer("rows", n, channels, h, w, 20, k, k, 1, k // 2), 26, schedule=daq.SCHEDULE_EARLY_COPY)


# Forward tensors that take blocks of eight groups: five and seven of them, 8 + 1, 8 + 5, 8 + 8 + 8 + 1; rows of whole units, odd and even ones
@pytest.mark.parametrize("channels,n,h,w,k", [(80, 101, 56, 56, 1), (100, 79, 57, 57, 3), (129, 59, 58, 58, 3), (208, 25, 71, 70, 1), (400, 77, 27, 31, 3),
                                              (72, 23400, 3, 5, 3)])
def test_forward_wide_blocks(channels, n, h, w, k):
    check_forward(wl.Layer("wide", n, channels, h, w, 4, k, k, 1, k // 2), wl.seed_for(27, channels))


# Blocks of more than four groups, which tensors of that size take (widths and last blocks: counting_pass() of tests/host/dispatch.hip): a
# whole record, 8 + 7, 8 + 5 and 8 + 8 + 1 groups, and of the large ones 7 + 6, 9 + 8, 9 + 9 + 7 and a whole record of twelve
@pytest.mark.parametrize("channels,n,h,w,k", [
    (112, 4, 140, 139, 3), (240, 3, 112, 112, 1), (200, 20, 45, 49, 1), (272, 11, 55, 57, 3),
    (208, 20, 101, 103, 1), (270, 16, 99, 101, 3), (400, 35, 56, 56, 3), (186, 73, 56, 56, 1),
])
def test_counting_pass_wide_blocks(channels, n, h, w, k):
    """Every workgroup walks several tiles, so both LDS tiles take their turns; both copies byte for byte, codes of both roundings, with
    guessed classes that hold and that do not, and one population for the whole layer."""
    layer = wl.Layer("wide", n, 1, h, w, channels, k, k, 1, k // 2)
    dY = wl.make_dY(layer, wl.seed_for(25, channels))
    st = wl.make_state(dY, wl.seed_for(25, channels))
    check_quantize_grad(layer, dY, st, mode=daq.ROUND_STOCHASTIC, seed=9 + n, schedule=daq.SCHEDULE_EARLY_COPY)
    check_quantize_grad(layer, dY, st, lam=0.0, schedule=daq.SCHEDULE_EARLY_COPY, check_padding=False)
    check_quantize_grad(layer, dY, st, lam=1.0, mode=daq.ROUND_STOCHASTIC, seed=n, schedule=daq.SCHEDULE_THREE_SWEEPS, check_padding=False)
    if n * h * w * channels < 2 ** 24:
        check_quantize_grad(layer, dY, st, scheme=daq.SCHEME_MCS, mode=daq.ROUND_STOCHASTIC, seed=n, check_padding=False)
        check_quantize_grad_bf16(layer, dY, st, mode=daq.ROUND_STOCHASTIC, seed=5)


FEW_TILES = [
    wl.Layer("d_one", 1, 1, 1, 1, 1, 3, 3, 1, 1),                # one pixel, one record unit a tap, five steps
    wl.Layer("d_units1", 2, 16, 9, 11, 33, 5, 5, 1, 2),          # one 16-byte unit a record: a step spans two taps
    wl.Layer("d_units3", 3, 40, 7, 9, 65, 3, 3, 1, 1),           # three: a step may, or may not
    wl.Layer("d_units5", 2, 70, 13, 5, 31, 1, 7, 1, 3),
    wl.Layer("d_stem", 3, 3, 17, 15, 40, 7, 7, 2, 3),            # 49 taps: the forward's eighth wave has the odd step
    wl.Layer("d_s2", 4, 50, 14, 13, 60, 3, 3, 2, 1),             # four parity classes of 1, 2, 2 and 4 taps
    wl.Layer("d_s2_1x1", 3, 130, 9, 8, 20, 1, 1, 2, 0),          # three of them without a tap: zeros
    wl.Layer("d_s2_dil", 2, 33, 15, 14, 40, 3, 3, 2, 2, dil=2),  # even dilation: all taps in one class
    wl.Layer("d_s3", 2, 20, 14, 16, 40, 3, 3, 3, 1),             # forward only
    wl.Layer("d_ks1", 41, 20, 64, 65, 40, 5, 5, 2, 2),           # forward, tiles enough for a wave each: 25 steps, ragged last workgroup
    wl.Layer("d_ks1_x", 19, 80, 35, 41, 5, 5, 5, 1, 2),          # data gradient, a wave each: 13 steps
    wl.Layer("d_ks8", 12, 96, 32, 33, 64, 3, 3, 2, 1),           # forward only
]


@pytest.mark.parametrize("layer", FEW_TILES, ids=lambda l: l.name)
def test_products_of_few_tiles(layer):
    """Both products without staging, 1 to 8 waves to a tile, records of 1 to 17 units, every class of taps (which of the two takes the
    kernel, and the waves: products() of tests/host/dispatch.hip)."""
    on_random_codes(layer, 71)
    check_forward(layer, 72)


@pytest.mark.parametrize("layer", [
    wl.Layer("t_narrow", 40, 70, 21, 23, 40, 3, 3, 1, 1),
    wl.Layer("t_taps9", 16, 140, 21, 23, 100, 3, 3, 1, 1),
    wl.Layer("t_ring", 30, 300, 25, 27, 300, 1, 1, 1, 0),
    wl.Layer("t_ring_s2", 40, 90, 31, 33, 330, 1, 1, 2, 0),
    wl.Layer("t_r128_s2", 40, 70, 41, 43, 70, 3, 3, 2, 1),
    wl.Layer("t_s2", 60, 30, 41, 43, 40, 3, 3, 2, 1),
    wl.Layer("t_s3", 8, 20, 9, 9, 20, 3, 3, 3, 1),
], ids=lambda l: l.name)
def test_products_of_many_ragged_tiles(layer):
    """Tiles enough for the tile kernel's forms, odd images, channel counts off every block."""
    on_random_codes(layer, 73)
    check_forward(layer, 74)


@pytest.mark.parametrize("channels,n,h,w", [(80, 4, 16, 16), (81, 4, 16, 16), (16, 25, 5, 8), (7, 205, 1, 5), (33, 3, 13, 13), (79, 147, 1, 1), (1, 1, 1, 3), (40, 300, 1, 3),
                                            (300, 5, 4, 4), (400, 7, 5, 3), (1024, 16, 1, 1), (1024, 5, 2, 2), (1025, 16, 1, 1)])
@pytest.mark.parametrize("k", [1, 3])
def test_resident_quantizer_writes_both_copies(channels, n, h, w, k):
    """Small tensors, both sides of the line to a launch of its own for the global copy, in every kind of load unit."""
    layer = wl.Layer("all", n, 1, h, w, channels, k, k, 1, k // 2)
    dY = wl.make_dY(layer, wl.seed_for(23, channels))
    st = wl.make_state(dY, wl.seed_for(23, channels))
    for mode, seed in ((daq.ROUND_NEAREST, 0), (daq.ROUND_STOCHASTIC, 41 + n)):
        check_quantize_grad(layer, dY, st, mode=mode, seed=seed, degenerate=n * h * w == 1)
        check_quantize_grad(layer, dY, st, mode=mode, seed=seed, degenerate=n * h * w == 1, side=torch.cuda.Stream())
        check_quantize_grad_bf16(layer, dY, st, mode=mode, seed=seed)


@pytest.mark.parametrize("channels,n,h,w", [(20, 5, 9, 7), (65, 3, 8, 5), (70, 4, 7, 9), (33, 6, 1, 3)])
def test_depthwise_copies_from_one_sweep(channels, n, h, w):
    """Both channel-major copies of a gradient of odd rows from the counting pass, with guessed classes that hold and that do not."""
    layer = wl.Layer("dwise", n, channels, h, w, channels, 3, 3, 1, 1, groups=channels)
    dY = wl.make_dY(layer, wl.seed_for(24, channels))
    st = wl.make_state(dY, wl.seed_for(24, channels))
    for mode, seed, lam in ((daq.ROUND_NEAREST, 0, 0.3), (daq.ROUND_STOCHASTIC, 3, 0.0), (daq.ROUND_STOCHASTIC, 4, 1.0)):
        check_quantize_grad(layer, dY, st, lam=lam, mode=mode, seed=seed, schedule=daq.SCHEDULE_EARLY_COPY)
        check_quantize_grad(layer, dY, st, lam=lam, mode=mode, seed=seed, schedule=daq.SCHEDULE_EARLY_COPY, side=torch.cuda.Stream())


@pytest.mark.parametrize("batch,size,channels", [(1, 8, 3), (2, 9, 20), (3, 13, 33), (40, 30, 9), (5, 31, 64)])
def test_depthwise_filter_gradient_at_stride_2(batch, size, channels):
    """Row pitches of every residue, one slab and several."""
    for w in range(size, size + 4):
        on_random_codes(wl.Layer("dws2", batch, channels, size, 2 * w, channels, 3, 3, 2, 1, groups=channels), 80 + w)


@pytest.mark.parametrize("batch,stride", [(1, 1), (3, 1), (5, 1), (7, 1), (1, 2), (3, 2)])
def test_tiles_dealt_to_the_xcds_with_remainders(batch, stride):
    on_random_codes(wl.Layer("deal", batch, 90, 11, 13, 70, 3, 3, stride, 1), 83)


@pytest.mark.parametrize("layer", [
    wl.Layer("w1", 33, 4065, 9, 15, 272, 1, 1, 1, 0),          # 2112 workgroups of one 256-pixel tile each: waves of 32 rows x 128 pixels
    wl.Layer("w1_less", 32, 4065, 9, 15, 272, 1, 1, 1, 0),     # 2048: 64 x 64
    wl.Layer("w1_s2", 33, 4065, 17, 29, 272, 1, 1, 2, 0),
    wl.Layer("wt", 33, 1009, 9, 15, 80, 1, 3, 1, 0),           # run-time tap list, several chunks: 528
    wl.Layer("wt_less", 32, 1009, 9, 15, 80, 1, 3, 1, 0),      # 512: 64 x 64
    wl.Layer("wt_one", 33, 1009, 9, 15, 40, 3, 3, 1, 1),       # one chunk
    wl.Layer("wt_s2", 9, 1009, 17, 29, 80, 3, 3, 2, 1),        # parity classes: 576
    wl.Layer("r128", 9, 1009, 17, 29, 40, 3, 3, 2, 1),         # one chunk by parity class: 128-row tiles
    wl.Layer("t9_256", 16, 1009, 9, 15, 80, 3, 3, 1, 1),       # constant taps: 256 workgroups, 256-pixel tiles
    wl.Layer("t9_128", 15, 1009, 9, 15, 80, 3, 3, 1, 1),       # fewer: 128-pixel tiles
], ids=lambda l: l.name)
def test_forms_of_the_halo_kernel(layer):
    """Both sides of the lines between the tile kernel's forms, result channels off every block."""
    on_random_codes(layer, 83)


@pytest.mark.parametrize("layer", [
    wl.Layer("eighths", 9, 70, 13, 13, 40, 1, 1, 1, 0),     # 96 blocks (two pairs of row blocks), an eighth for each XCD
    wl.Layer("eighths_few", 1, 30, 5, 5, 20, 1, 1, 1, 0),   # fewer blocks than XCDs
    wl.Layer("turns", 12, 250, 8, 8, 130, 1, 1, 1, 0),      # planes of whole lines, four pairs: 16 blocks a turn, some left over
    wl.Layer("plain", 12, 130, 8, 8, 40, 1, 1, 1, 0),       # three pairs
    wl.Layer("large", 9, 250, 75, 75, 20, 1, 1, 1, 0),      # more than 48 MiB: eight quads a turn
], ids=lambda l: l.name)
def test_blocks_of_the_streaming_form(layer):
    """Orders in which the XCDs take the blocks, with remainders."""
    on_random_codes(layer, 85)
