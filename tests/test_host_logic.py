"""CPU-only checks of the C-ABI library: it loads, exports every declared symbol, and its host
logic (layouts, workspace sizes, argument validation) behaves.  No kernel is launched."""
import ctypes as C
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2102_04782_amd import binding as daq
from paper_2102_04782_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(ROOT, "include", "daq.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(daq_[a-z0-9_]+)\s*\(", hdr))
    assert {"daq_quantize_grad", "daq_conv_fwd_int8", "daq_conv_bwd_data_int8", "daq_conv_bwd_filter_int8"} <= declared
    L = C.CDLL(daq.LIB_PATH)
    for name in sorted(declared):
        assert hasattr(L, name), f"{name} declared in daq.h but not exported"
    assert declared == set(daq.EXPORTS)


CASES = [
    dict(N=2, Cin=3, Hin=9, Win=7, Cout=5, kH=3, kW=3, strideH=1, strideW=1, padH=1, padW=1),
    dict(N=2, Cin=4, Hin=9, Win=8, Cout=6, kH=3, kW=3, strideH=2, strideW=2, padH=1, padW=1),
    dict(N=1, Cin=3, Hin=15, Win=15, Cout=4, kH=7, kW=7, strideH=2, strideW=2, padH=3, padW=3),
    dict(N=3, Cin=8, Hin=5, Win=5, Cout=8, kH=1, kW=1),
    dict(N=2, Cin=8, Hin=6, Win=6, Cout=16, kH=1, kW=1, strideH=2, strideW=2),
    dict(N=2, Cin=6, Hin=7, Win=7, Cout=6, kH=3, kW=3, padH=1, padW=1, groups=6),
    dict(N=1, Cin=2, Hin=8, Win=8, Cout=2, kH=3, kW=3, padH=2, padW=2, dilH=2, dilW=2),
    dict(N=1, Cin=2, Hin=6, Win=5, Cout=3, kH=3, kW=3, padH=3, padW=3),
]


@pytest.mark.parametrize("kw", CASES)
def test_layouts_are_injective_in_bounds_and_tap_shifts_are_constant(kw):
    d = daq.ConvDesc.make(**kw)
    Ho, Wo = d.Ho, d.Wo
    layouts = [daq.layout_vq(d), daq.layout_qg(d), daq.layout_qx_nhwc(d), daq.layout_qx_cnhw(d)]
    for L in layouts:
        off = L.offsets().ravel()
        assert off.min() >= 0 and off.max() < L.bytes
        assert len(np.unique(off)) == off.size
        rng = np.random.default_rng(0)
        codes = rng.integers(-127, 128, (L.N, L.C, L.H, L.W)).astype(np.int8)
        assert np.array_equal(L.unpack(L.pack(codes)), codes)
    # the property the filter-gradient kernel relies on: for a fixed tap, the activation element that
    # multiplies gradient element f sits at f + const in the activation's plane, or is zero padding
    Lg, Lx = daq.layout_vq(d), daq.layout_qx_cnhw(d)
    assert (Lg.img_rows, Lg.row_pitch) == (Lx.img_rows, Lx.row_pitch)
    # zero halo: whatever a tap can reach from a real gradient element, before the first image or behind the
    # last one, is inside the plane (and zero, which the GPU tests check on real buffers)
    reach = ((d.kH - 1) * d.dilH + 1) * Lg.row_pitch + (d.kW - 1) * d.dilW
    assert Lg.lead >= reach and Lg.plane_pitch - (Lg.lead + d.N * Lg.img_rows * Lg.row_pitch) >= reach
    assert Lx.lead >= Lg.lead
    rng = np.random.default_rng(1)
    X = rng.integers(1, 128, (d.N, d.Cin, d.Hin, d.Win)).astype(np.int8)  # strictly positive: zero means padding
    buf = Lx.pack(X)
    for kh in range(d.kH):
        for kw_ in range(d.kW):
            hh, ww = kh * d.dilH, kw_ * d.dilW
            if d.strideH == 1 and d.strideW == 1:
                plane, delta = 0, hh * Lx.row_pitch + ww  # the activation's lead already holds the padding shift
                base = 0
            else:
                plane = (hh % d.strideH) * d.strideW + (ww % d.strideW)
                delta = (hh // d.strideH) * Lx.row_pitch + ww // d.strideW
                base = 0
            for n in range(d.N):
                for ho in range(Ho):
                    for wo in range(Wo):
                        f = Lg.lead + (n * Lg.img_rows + ho) * Lg.row_pitch + wo
                        h = ho * d.strideH + hh - d.padH
                        w = wo * d.strideW + ww - d.padW
                        inside = 0 <= h < d.Hin and 0 <= w < d.Win
                        got = buf[0 * Lx.chan_pitch + plane * Lx.plane_pitch + base + f + delta]
                        assert got == (X[n, 0, h, w] if inside else 0)
    # reading 16 bytes past any gradient position plus the largest tap shift stays inside the plane
    max_delta = ((d.kH - 1) * d.dilH // d.strideH) * Lx.row_pitch + (d.kW - 1) * d.dilW // d.strideW
    assert Lg.plane_pitch % 256 == 0 and Lg.plane_pitch + max_delta + 16 <= Lx.plane_pitch


@pytest.mark.parametrize("kw", [
    dict(N=2, Cin=3, Hin=9, Win=7, Cout=3, kH=3, kW=3, padH=1, padW=1, groups=3),
    dict(N=2, Cin=2, Hin=12, Win=11, Cout=2, kH=3, kW=3, strideH=2, strideW=2, padH=1, padW=1, groups=2),
    dict(N=2, Cin=2, Hin=11, Win=12, Cout=2, kH=3, kW=3, strideH=2, strideW=2, padH=0, padW=0, groups=2),
    dict(N=3, Cin=2, Hin=13, Win=13, Cout=2, kH=5, kW=5, strideH=2, strideW=2, padH=2, padW=2, groups=2),
    dict(N=2, Cin=2, Hin=10, Win=10, Cout=2, kH=3, kW=3, padH=2, padW=2, dilH=2, dilW=2, groups=2),
    dict(N=2, Cin=2, Hin=9, Win=9, Cout=2, kH=3, kW=3, padH=0, padW=0, groups=2),
    dict(N=2, Cin=2, Hin=16, Win=16, Cout=2, kH=7, kW=7, strideH=4, strideW=4, padH=3, padW=3, groups=2),
])
def test_planar_gradient_neighbours_are_the_element_or_zero(kw):
    """The depthwise data-gradient kernels read G'[c] at lead + (n*img_rows + ho)*row_pitch + wo for every
    (ho, wo) a tap asks for, in range or not, without a bounds test."""
    d = daq.ConvDesc.make(**kw)
    L = daq.layout_qg(d)
    assert L.kind == daq.LAYOUT_CNHW
    rng = np.random.default_rng(5)
    G = rng.integers(1, 128, (d.N, d.Cout, d.Ho, d.Wo)).astype(np.int8)   # strictly positive: zero means padding
    buf = L.pack(G)
    for c in range(d.Cout):
        for n in range(d.N):
            for h in range(d.Hin):
                for w in range(d.Win):
                    for kh in range(d.kH):
                        th = h + d.padH - kh * d.dilH
                        if th % d.strideH:
                            continue
                        for kw_ in range(d.kW):
                            tw = w + d.padW - kw_ * d.dilW
                            if tw % d.strideW:
                                continue
                            ho, wo = th // d.strideH, tw // d.strideW
                            pos = c * L.chan_pitch + L.lead + (n * L.img_rows + ho) * L.row_pitch + wo
                            assert 0 <= pos < L.bytes
                            inside = 0 <= ho < d.Ho and 0 <= wo < d.Wo
                            assert buf[pos] == (G[n, c, ho, wo] if inside else 0), (n, h, w, kh, kw_)


def test_weight_packing_roundtrip():
    for kw in CASES:
        d = daq.ConvDesc.make(**kw)
        L = daq.layout_qw(d)
        rng = np.random.default_rng(2)
        qW = rng.integers(-127, 128, d.w_shape).astype(np.int8)
        buf = L.pack(d, qW)
        cig, cog, taps = d.Cin // d.groups, d.Cout // d.groups, d.kH * d.kW
        fwd = buf[L.off_fwd:L.off_fwd + taps * d.Cout * L.cig_pitch].reshape(taps, d.Cout, L.cig_pitch)
        bwd = buf[L.off_bwd:L.off_bwd + taps * d.Cin * L.cog_pitch].reshape(taps, d.Cin, L.cog_pitch)
        for co in range(d.Cout):
            g = co // cog
            for cl in range(cig):
                for t in range(taps):
                    v = qW[co, cl, t // d.kW, t % d.kW]
                    assert fwd[t, co, cl] == v and bwd[t, g * cig + cl, co % cog] == v


def test_workspace_and_validation_without_a_gpu():
    d = daq.ConvDesc.make(N=2, Cin=4, Hin=8, Win=8, Cout=4, kH=3, kW=3, padH=1, padW=1)
    for op in range(4):
        assert daq.workspace_bytes(op, d) >= 256
    assert daq.workspace_bytes(7, d) == 0
    bad = daq.ConvDesc.make(N=0, Cin=4, Hin=8, Win=8, Cout=4, kH=3, kW=3)
    assert daq.workspace_bytes(0, bad) == 0
    L = daq.Layout()
    assert daq.lib().daq_layout_vq(C.byref(bad), C.byref(L)) == daq.ERR_INVALID_ARG
    for kw in (dict(Cin=5, groups=2), dict(kH=9), dict(strideH=0), dict(padH=-1), dict(dilW=0)):
        base = dict(N=1, Cin=4, Hin=8, Win=8, Cout=4, kH=3, kW=3)
        base.update(kw)
        assert daq.workspace_bytes(0, daq.ConvDesc.make(**base)) == 0
    # null pointers / bad enums / short workspace are rejected on the host, before any launch
    lib = daq.lib()
    one = C.c_void_p(256)  # never dereferenced: validation fails first
    assert lib.daq_quantize_grad(C.byref(d), None, one, 1.0, 0.8, 0.3, 0, 0, one, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_quantize_grad(C.byref(d), one, one, 1.0, 0.8, 0.3, 5, 0, one, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_quantize_grad(C.byref(d), one, one, 1.0, 0.8, 0.3, 0, 0, one, one, one, one, one, None, one, 8, None) == daq.ERR_WORKSPACE
    assert lib.daq_quantize_grad(C.byref(d), one, one, 1.0, 0.8, 0.3, 0, 0, one, one, one, one, one, None, C.c_void_p(257), 1 << 20, None) == daq.ERR_WORKSPACE
    assert lib.daq_quantize_grad(C.byref(bad), one, one, 1.0, 0.8, 0.3, 0, 0, one, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_conv_bwd_data_int8(C.byref(d), None, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_conv_bwd_filter_int8(C.byref(d), one, one, one, one, None, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_conv_bwd_filter_int8(C.byref(d), one, one, one, one, one, None, None, 0, None) == daq.ERR_WORKSPACE
    assert lib.daq_conv_fwd_int8(C.byref(d), one, None, one, one, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    both = lambda **kw: lib.daq_conv_bwd_int8(C.byref(kw.get("desc", d)), kw.get("qx", one), one, kw.get("vq", one), one, kw.get("dW", one),
                                              None, one, one, one, one, kw.get("dX", one), None, kw.get("ws", one), kw.get("wsb", 1 << 24), None)
    assert both(dW=None) == daq.ERR_INVALID_ARG and both(dX=None) == daq.ERR_INVALID_ARG and both(desc=bad) == daq.ERR_INVALID_ARG
    assert both(ws=None) == daq.ERR_WORKSPACE and both(wsb=256) == daq.ERR_WORKSPACE
    assert both(vq=C.c_void_p(257)) == daq.ERR_INVALID_ARG
    assert daq.workspace_bytes(daq.OP_CONV_BWD, d) == daq.workspace_bytes(daq.OP_CONV_BWD_FILTER, d) + daq.workspace_bytes(daq.OP_CONV_BWD_DATA, d)
    # misaligned int8 buffers
    odd = C.c_void_p(257)
    assert lib.daq_conv_bwd_data_int8(C.byref(d), odd, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_conv_bwd_filter_int8(C.byref(d), one, one, odd, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    assert lib.daq_quantize_grad(C.byref(d), one, one, 1.0, 0.8, 0.3, 0, 0, odd, one, one, one, one, None, one, 1 << 20, None) == daq.ERR_INVALID_ARG
    sch = lambda scheme, ws=one, wsb=1 << 20: lib.daq_quantize_grad_scheme(C.byref(d), one, one, 1.0, 0.8, 0.3, 0, 0, scheme, one, one,
                                                                            one, one, one, None, ws, wsb, None)
    assert sch(4) == daq.ERR_INVALID_ARG and sch(-1) == daq.ERR_INVALID_ARG
    assert all(sch(s, wsb=8) == daq.ERR_WORKSPACE for s in range(4))           # a known scheme gets as far as the workspace check
    chan = lambda desc=d, vq=one: lib.daq_conv_bwd_data_int8_chan(C.byref(desc), vq, one, one, one, one, None, one, 1 << 20, None)
    assert chan() == daq.ERR_UNSUPPORTED                                       # a dense layer
    assert chan(vq=None) == daq.ERR_INVALID_ARG and chan(vq=odd) == daq.ERR_INVALID_ARG and chan(desc=bad) == daq.ERR_INVALID_ARG
    b16 = lambda dY=one, scheme=0, wsb=1 << 20: lib.daq_quantize_grad_bf16(C.byref(d), dY, one, 1.0, 0.8, 0.3, 0, 0, scheme, one, one,
                                                                        one, one, one, None, one, wsb, None)
    assert b16(dY=None) == daq.ERR_INVALID_ARG and b16(dY=odd) == daq.ERR_INVALID_ARG and b16(scheme=9) == daq.ERR_INVALID_ARG
    assert b16(wsb=8) == daq.ERR_WORKSPACE
    assert daq.status_string(daq.ERR_WORKSPACE).startswith("workspace")


def _run_host_program(name, tmp_path, *extra):
    """Compiles tests/host/<name> against the library's sources and runs it (no GPU call)."""
    exe, pkg = str(tmp_path / "prog"), os.path.join(ROOT, "paper_2102_04782_amd")
    res = subprocess.run(["hipcc", "-O1", "-std=c++17", *extra, "-Wno-unused-function", "-Wno-pass-failed", "-I", os.path.join(ROOT, "include"), "-I",
                          os.path.join(pkg, "csrc"), os.path.join(ROOT, "tests", "host", name), "-o", exe, "-L" + pkg, "-ldaq", "-Wl,-rpath," + pkg],
                         capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert run.returncode == 0, run.stdout + run.stderr


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_frame_copies_of_3d_layers_stay_inside_the_workspace(tmp_path):
    _run_host_program("frame_copies.hip", tmp_path, "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_split_search_finds_the_cheapest_count_among_few(tmp_path):
    _run_host_program("split_search.hip", tmp_path, "--offload-arch=gfx950")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_dispatch_rules(tmp_path):
    _run_host_program("dispatch.hip", tmp_path, "--offload-arch=gfx950")


def test_workload_tables():
    r50 = wl.config4()
    assert len(r50) == 53 and len({(l.Cin, l.Hin, l.Cout, l.kH, l.stride) for l in r50}) == 23
    total = sum(l.macs for l in r50)
    assert abs(total - 261.6e9) / 261.6e9 < 0.01          # 2 x 261.6 GMAC x 2 convs = 1046 GOP backward
    assert sum(int(np.prod(l.y_shape)) for l in r50) == 711_294_976           # gradient elements the quantizer sweeps
    mb = wl.config5()
    assert len(mb) == 50 and sum(1 for l in mb if l.groups > 1) == 17
    assert abs(sum(int(np.prod(l.y_shape)) for l in mb) - 795.4e6) < 1e6
    l2 = wl.config2()[0]
    assert l2.y_shape == (32, 64, 56, 56) and 2 * l2.macs == 7_398_752_256     # 7.40 GOP per GEMM
    # generators are seeded and follow the recipe: even channels bell-shaped, odd channels long-tailed
    layer, X, W, dY, st = wl.make_inputs(1)
    _, _, _, dY2, _ = wl.make_inputs(1)
    assert np.array_equal(dY, dY2) and dY.dtype == np.float32
    kurt = lambda v: np.mean((v - v.mean()) ** 4) / np.var(v) ** 2
    assert all(kurt(dY[:, c].ravel()) < 4 for c in range(0, 16, 2))
    assert all(kurt(dY[:, c].ravel()) > 20 for c in range(1, 16, 2))
    assert np.all(st > 0)


def test_bench_prices_every_layer_by_the_early_copy_it_takes():
    import argparse
    import bench

    Mi = 2 ** 20
    for net in (wl.config4(), wl.config5()):
        for layer in net:
            d = daq.ConvDesc.make(*layer.desc_fields())
            qg_nhwc = daq.layout_qg(d).kind == daq.LAYOUT_NHWC
            for rounding, bf16 in (("stochastic", False), ("nearest", False), ("nearest", True)):
                at = bench.early_copy_from(argparse.Namespace(rounding=rounding, dy_bf16=bf16), d, qg_nhwc)
                assert at == 4 * Mi if rounding == "stochastic" else at in (4 * Mi, 6 * Mi, 8 * Mi, float("inf"))
