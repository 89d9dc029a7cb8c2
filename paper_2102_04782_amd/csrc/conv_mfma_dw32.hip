// Filter gradient  q(G_W) = q(X') (x) vq(G')  for 3 x 3 (k_dw32) and 1 x 1 (k_dw11) filters at unit stride and
// dilation, on the full-rate v_mfma_i32_32x32x32_i8 with both operands staged through LDS.
//
// Same shifted-correlation form as conv_mfma_dw.hip:
//     acc[co][ci][kh][kw] = sum_f  G[co][f] * X[ci][f + kh*row_pitch + kw]
// A workgroup stages, per 256-byte chunk of the flat axis, gradient rows and activation rows (the latter as
// much longer as the last tap's window reaches), multiplies with four waves, each a 32 (co) x 32 (ci) x 9 (tap) accumulator tile (144
// registers), and derives the windows of neighbouring columns with v_alignbyte_b32.  k_dw32_ring: the four waves share one tile and take two
// of the eight K steps of every chunk each, combined through LDS at the end, four more waves ask for the operands (dw32_role.h); K
// can also be split across workgroups: partial tiles are written with coalesced stores and summed
// by k_dw_reduce.  k_dw32, for layers with 256 and more tiles of 64 x 64: a tile for each wave, coalesced loads, double buffered in LDS behind
// registers that keep the next chunk in flight.
#include <algorithm>

#include "daq_internal.h"
#include "dw32_role.h"
#include "dw_tail.h"

namespace daq {

namespace {

constexpr int kDwReducePerWave = 16;   // up to this many K splits a wave of the reduction sums a group of results alone

// Sum of the K-split partial tiles, then dW = acc * ((s_x/127) * (s_chan[co]/127)), for both kernels of this file
// (the same code serves as a role inside the data-gradient kernel, see dw_tail.h).  With many splits a workgroup
// takes one group of 64 results and its four waves share the splits; with few, every wave takes a group of its own
// and keeps all of its loads in flight - no LDS, no barrier.
__global__ __launch_bounds__(256) void k_dw_reduce(DwTail t) {
    __shared__ int32_t l_sum[4 * kWave];
    if (blockIdx.y > 0) {   // depth tap of a 3-D layer
        const int entries = t.blocks;
        t.part += (int64_t)blockIdx.y * entries * t.splits * kWave;
        t.dW += blockIdx.y * t.taps;
        if (t.acc_out) t.acc_out += blockIdx.y * t.taps;
    }
    if (t.splits > kDwReducePerWave) {
        dw_reduce_role(t, (int)blockIdx.x, l_sum);
        return;
    }
    const int lane = threadIdx.x % kWave;
    const int e = (int)blockIdx.x * 4 + (int)(threadIdx.x / kWave);
    if (e >= t.blocks) return;
    int64_t stride;
    const int32_t* src = dw_tail_source(t, e, lane, stride);
    int32_t v[kDwReducePerWave];
#pragma unroll
    for (int s = 0; s < kDwReducePerWave; ++s) v[s] = src[(int64_t)min(s, t.splits - 1) * stride];
    int32_t a = 0;
#pragma unroll
    for (int s = 0; s < kDwReducePerWave; ++s) a += s < t.splits ? v[s] : 0;
    int co;
    const int64_t off = dw_tail_element(t, e, lane, co);
    if (off < 0) return;
    store_result(t.dW, off, (float)a * ((*t.s_x / 127.0f) * (t.s_chan[co] / 127.0f)), t.bf16);
    if (t.acc_out) t.acc_out[off] = a;
}

template <int WQ4>
__global__ __launch_bounds__(256) void k_dw32(Dw32Args p) {
    dw32_role<WQ4>(p, (int)blockIdx.x);
}

template <bool S2>
__global__ __launch_bounds__(512) void k_dw32_ring(Dw32Args p) {
    dw32_ring_role<S2>(p, (int)blockIdx.x);
}

template <int WM, int WN, int WK, int PF, int CH, bool DMA = false, bool LONG = false>
__global__ __launch_bounds__(64 * WM * WN * WK) void k_dw11(Dw32Args p) {
    dw11_role<WM, WN, WK, PF, CH, DMA, LONG>(p, (int)blockIdx.x);
}

// K splits across workgroups.  A workgroup fills a CU (its stage buffers are 100 to 150 KB of LDS), so a launch of more than 256 runs in
// rounds, and 264 take as long as 512; a split launch is followed by
// the reduction, which costs a launch and the partial tiles' way to memory and back.  The split that minimises
//     rounds * (chunks of a workgroup * t_chunk + t_fixed) + (reduction, if any)
// with 4 us of prologue, combine and stores and
//     nine taps               0.65 us a chunk, 2.5 for a reduction and its launch, partial tiles at 0.83 TB/s there and back
//     nine taps at stride 2   1.0, 4.5, 0.83
//     one tap                 0.5, 3.3, 1
// is 1.7 (2.9 with 1.1 us, 3.3 and 1 TB/s, as the kernel took before), 1.5 (4.5 with 2.0) and 2 % from the fastest of up to 20 counts on average, over 152, 65 and
// 230 layers.  (64 -> 64, 3 x 3 x 3 on 8 x 56 x 56: 22 splits are 264 workgroups and take 1.7 times as long as 21, which are 252.)
SplitModel split_model(const Plan32& pl, int depth) {
    const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n * depth;
    const double t_chunk = pl.k11 ? 0.5 : pl.s2 ? 1.0 : 0.65, t_reduce = pl.k11 ? 3.3 : pl.s2 ? 4.5 : 2.5;
    const double part_us = pl.k11 ? 64 * 64 * 4 / 1e6 : 1.2 * 32 * 32 * kT * 4 / 1e6;   // of a partial tile
    return SplitModel{pl.nchunks, tiles, 4 * 256 / tiles, t_chunk, 4.0, 0.0, t_reduce, (double)tiles * part_us};
}

// 1 x 1 filters hardly reuse an operand inside a workgroup, and with 3, 5, 6 or 7 splits every XCD reads nearly all of both (dw_block_map):
// a chunk takes half as long again (434 -> 689 at 8 x 46, batch 43: 26.9 us with three splits, 20.2 with two).  And a split has to save
// what the reduction's launch takes the host, 2.5 us: networks of such small layers are enqueued more slowly than they run (384 -> 64 at
// 14 x 14, batch 16: 10.1 us in one part, 8.8 in two launches, 5.7 and 7.4 on the host; 24 of 157 layers, 0.3 us each on the GPU).
int choose_splits(const Plan32& pl, int depth) {
    const SplitModel m = split_model(pl, depth);
    int s = cheapest_split(m);
    if (pl.k11 && m.cost(1) < m.cost(s) + 2.5) return 1;
    if (!pl.k11 || s < 3 || s == 4 || s > 7) return s;
    SplitModel scattered = m;
    scattered.t_step *= 1.5;
    double best = scattered.cost(s);
    for (int64_t near : {1, 2, 4, 8})
        if (near <= std::min(m.limit, m.n) && m.cost(near) < best) { best = m.cost(near); s = (int)near; }
    return s;
}

// The split where a later kernel takes the reduction along, from 33 splits on (dw_tail_worthwhile): 2.8 us for its launch are
// saved.  (Whatever the model charges for launch and reduction together: 150 layers, both gradients, with 2.2 and 1.5 up to 0.87 of the speed at
// stride 2, 3.5 and 5 within 0.1 %.  7 -> 106, 3 x 3 on 99 x 12, batch 30, both gradients: 23 us with 25 splits and a reduction, 21 with 64.)
int choose_splits_tail(const Plan32& pl) {
    const SplitModel m = split_model(pl, 1);
    const int64_t top = std::min(m.limit, m.n);
    if (pl.wk == 1 || pl.splits > 32 || top <= 32 || !dw_tail_worthwhile((int)(pl.part_slots / kWave), 33)) return pl.splits;
    int best_s = pl.splits;
    double best = m.cost(pl.splits) + 2.8;
    int64_t s = 33;
    for (int i = 0; i < 3 && s <= top; ++i) {   // the next lengths of the longest part: from there on partial tiles cost more than they save
        const int64_t longest = ceil_div(m.n, s);
        if (m.cost(s) < best) { best = m.cost(s); best_s = (int)s; }
        if (longest <= 1) break;
        s = ceil_div(m.n, longest - 1);
    }
    return best_s;
}

// Rectangles per split for 1, 2 or 4 splits (8, 4 or 2 XCDs share a split): the cut of the tile grid that makes an
// XCD touch the fewest operand rows, rows of the two operands weighted by their tile heights - unless its largest rectangle takes
// a round over the XCD's 32 CUs more than the tiles dealt out evenly (513 -> 193, 3 x 3 on 77 x 6, batch 90: 238 workgroups in
// rectangles of up to 35, 113 us; dealt out 66).
void choose_bands(Plan32& pl, int bm, int bn, int depth = 1) {
    pl.bands_m = pl.bands_n = pl.band_m = pl.band_n = 0;
    pl.blocks = (int64_t)pl.tiles_m * pl.tiles_n * pl.splits;
    if (pl.splits != 1 && pl.splits != 2 && pl.splits != 4) return;
    const int rects = kXcd / pl.splits;
    int64_t best = -1;
    for (int rm = 1; rm <= rects; rm *= 2) {
        const int rn = rects / rm;
        if (rm > pl.tiles_m || rn > pl.tiles_n) continue;
        const int64_t hm = ceil_div(pl.tiles_m, rm), hn = ceil_div(pl.tiles_n, rn);
        const int64_t rows = hm * bm + hn * bn;
        if (ceil_div(hm * hn * depth, 32) > ceil_div(pl.blocks * depth, 256)) continue;
        if (best < 0 || rows < best) { best = rows; pl.bands_m = rm; pl.bands_n = rn; pl.band_m = (int)hm; pl.band_n = (int)hn; }
    }
    if (best < 0) { pl.bands_m = pl.bands_n = 0; return; }
    pl.blocks = (int64_t)kXcd * pl.band_m * pl.band_n;
}

}  // namespace

// 1 x 1: from how many chunks of a workgroup on its requests are addressed by vector instructions.  Operands from memory, scalar and vector
// addresses: 512 -> 2048 at 7 x 7, batch 128, 25 chunks, 19.8 and 19.4 us; 512 -> 1024 at stride 2, 28 x 28, batch 128, 50 chunks, 37.8 and 36.4;
// 32 -> 1312 at stride 2, 70 x 70, batch 3, 15 chunks, 9.7 and 10.3; 64 -> 384 at 14 x 14, batch 64, 9.1 and 9.3.  By chunks, over 182 layers: below 9
// 0.987 of the time with scalar addresses, 9 to 19 0.994, 20 to 33 1.008, from 34 on 1.013.
bool dw11_long(int64_t chunks) { return chunks >= 20; }

Plan32 make_plan32(const daq_conv_desc& d, int depth) {
    Plan32 pl{};
    if (d.groups != 1) return pl;
    const bool unit = d.strideH == 1 && d.strideW == 1 && d.dilH == 1 && d.dilW == 1;
    // a 1 x 1 filter pairs gradient position f with byte f of the activation's first stride-phase plane whatever the
    // stride (and dilation means nothing), so the plain GEMM serves strided shortcuts too
    const bool k33 = unit && d.kH == 3 && d.kW == 3, k11 = d.kH == 1 && d.kW == 1;
    const bool k33s2 = d.kH == 3 && d.kW == 3 && d.strideH == 2 && d.strideW == 2 && d.dilH == 1 && d.dilW == 1;
    if (!k33 && !k11 && !k33s2) return pl;
    daq_layout Lg, Lx;
    if (daq_layout_vq(&d, &Lg) != DAQ_OK || daq_layout_qx_cnhw(&d, &Lx) != DAQ_OK) return pl;
    if (Lg.bytes >= ((int64_t)1 << 32) || Lx.bytes >= ((int64_t)1 << 32)) return pl;   // 32-bit per-lane offsets
    pl.nchunks = (int)(Lg.plane_pitch / kKC);
    if (k11) {
        // plain GEMM: 64 x 64 per wave; 128 x 128 per workgroup when that alone fills the chip, else eight waves on one
        // 64 x 64 tile with K split among them and across workgroups
        pl.k11 = true;
        const int64_t t128 = ceil_div(d.Cout, 128) * ceil_div(d.Cin, 128);
        if (t128 >= 256) { pl.wm = 2; pl.wn = 2; pl.wk = 1; }
        else { pl.wm = 1; pl.wn = 1; pl.wk = 8; }
        pl.tiles_m = (int)ceil_div(d.Cout, 64 * pl.wm);
        pl.tiles_n = (int)ceil_div(d.Cin, 64 * pl.wn);
        const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n;
        pl.splits = pl.wk == 1 ? 1 : choose_splits(pl, depth);
        // One chunk per LDS stage.  (Two chunks per barrier were measured on the late ResNet-50 layers: the K loop of a
        // workgroup - 13 chunks of 32 KiB in 7 us on every CU at once, bound by the staging through registers and LDS and
        // its two waits per chunk - gets a quarter shorter per byte, and the first stage arrives that much later.)
        pl.ch = 1;
        const size_t stage = (size_t)64 * (pl.wm + pl.wn) * (pl.ch * kKC + 16);
        pl.lds_bytes = std::max<size_t>(pl.wk > 1 ? (size_t)4 * 128 * kKC : 2 * stage, pl.wk > 1 ? (size_t)(pl.wk - 1) * 64 * kWave * 4 : 0);   // staging (four unpadded stages in the direct-to-LDS form); one-round combine
        pl.part_slots = tiles * pl.wm * pl.wn * 64 * kWave;
        pl.splits_tail = choose_splits_tail(pl);
        choose_bands(pl, 64 * pl.wm, 64 * pl.wn, depth);
        pl.ok = true;
        return pl;
    }
    if (k33s2) {
        // the strided form relies on the slot geometry the two operands share and on the four phase planes of a channel
        if (Lx.phases_h != 2 || Lx.phases_w != 2 || Lx.row_pitch != Lg.row_pitch || Lx.img_rows != Lg.img_rows ||
            Lx.lead != Lg.lead || Lx.chan_pitch != 4 * Lx.plane_pitch)
            return pl;
        pl.s2 = true;
    }
    if (Lx.row_pitch > (pl.s2 ? ring32_max_pitch<true>() : ring32_max_pitch<false>())) return pl;
    const int64_t t64 = ceil_div(d.Cout, 64) * ceil_div(d.Cin, 64);
    if (t64 >= 256 && !pl.s2) { pl.wm = 2; pl.wn = 2; pl.wk = 1; }
    else { pl.wm = 1; pl.wn = 1; pl.wk = 8; }   // the ring: one tile of 32 x 32 to a workgroup, eight waves (dw32_ring_role)
    const int bm = 32 * pl.wm, bn = 32 * pl.wn;
    pl.tiles_m = (int)ceil_div(d.Cout, bm);
    pl.tiles_n = (int)ceil_div(d.Cin, bn);
    const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n;
    if (pl.wk == 1) {
        // bytes of an activation row a chunk needs: its own 256 plus the largest tap offset, plus the bytes the
        // six-dword reads of the last K step touch beyond that
        pl.b_units = (int)ceil_div(kKC + 2 * Lx.row_pitch + 2 + 8, 16);
        pl.pb = 16 * pl.b_units + 4;          // pitch/4 odd: the 32 rows of a fragment read fall into 32 different banks
        pl.splits = 1;
        pl.lds_bytes = 2 * ((size_t)bm * kPA + (size_t)bn * pl.pb);
    } else {
        pl.b_units = ring32_units(pl.s2, Lx.row_pitch);
        pl.splits = choose_splits(pl, depth);
        pl.lds_bytes = pl.s2 ? Ring32<true>::LDS : Ring32<false>::LDS;
    }
    pl.part_slots = tiles * pl.wm * pl.wn * kT * 16 * kWave;
    pl.splits_tail = choose_splits_tail(pl);
    choose_bands(pl, bm, bn, depth);
    pl.ok = true;
    return pl;
}

namespace {

Dw32Args fill_args(const Plan32& pl, const daq_conv_desc& d, const daq_layout& Lx, const daq_layout& Lg, const int8_t* qx, const float* s_x,
                   const int8_t* vq, const float* s_chan, float* dW, int32_t* acc, void* ws, bool bf16, const DwDepth* dp) {
    const int depth = dp ? dp->kD : 1;
    Dw32Args a{};
    a.g = vq;
    a.x = qx;
    a.klen = Lg.plane_pitch;
    a.x_chan_pitch = Lx.chan_pitch;
    a.x_plane_pitch = Lx.plane_pitch;
    a.Cout = d.Cout;
    a.Cin = d.Cin;
    a.row_pitch = Lx.row_pitch;
    a.pb = pl.pb;
    a.b_units = pl.b_units;
    a.nchunks = pl.nchunks;
    a.splits = pl.splits;
    a.tiles_n = pl.tiles_n;
    a.tiles_m = pl.tiles_m;
    a.bands_m = pl.bands_m; a.bands_n = pl.bands_n; a.band_m = pl.band_m; a.band_n = pl.band_n;
    a.part = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(ws) + 256);
    a.s_x = s_x;
    a.s_chan = s_chan;
    a.dW = dW;
    a.acc_out = acc;
    a.bf16 = bf16 ? 1 : 0;
    const int taps = pl.k11 ? 1 : kT;
    a.taps_all = taps * depth;
    a.sD = 1;
    if (dp) {
        // the activation's buffer holds more frames than the gradient's and as many copies as the depth stride
        a.dD = dp->dD;
        a.sD = dp->sD;
        a.x_chan_pitch = dp->x_chan_pitch;
        a.x_plane_pitch = dp->x_plane_pitch;
        a.x_frame = (int64_t)Lx.img_rows * Lx.row_pitch;
        a.x_depth_phase = dp->x_depth_phase;
        a.part_kd = pl.part_slots * pl.splits;
    }
    return a;
}

DwTail tail_of(const Plan32& pl, const Dw32Args& a, const daq_conv_desc& d, int depth) {
    const int taps = pl.k11 ? 1 : kT;
    return DwTail{a.part, (int)(pl.part_slots / kWave), pl.splits, pl.tiles_n, pl.wm, pl.wn, d.Cout, d.Cin, taps, a.s_x, a.s_chan, a.dW, a.acc_out,
                  a.bf16, taps * depth};
}

// The last stage of a K-split launch: left to the caller's next kernel where that pays, a launch of its own otherwise.
daq_status finish(const Plan32& pl, const DwTail& t, DwTail* defer, int depth, hipStream_t st) {
    if (pl.splits == 1) return DAQ_OK;
    if (defer && dw_tail_worthwhile(t.blocks, pl.splits)) {
        *defer = t;
        return DAQ_OK;
    }
    return launch_dw_reduce(t, depth, st);
}

daq_status launch32(const Plan32& pl, const Dw32Args& a, hipStream_t st, int depth) {
    const dim3 grid((unsigned)pl.blocks, (unsigned)depth);
    if (pl.wk == 1) {
        const int wq4 = a.row_pitch & 3;
        auto kern = wq4 == 0 ? k_dw32<0> : wq4 == 1 ? k_dw32<1> : wq4 == 2 ? k_dw32<2> : k_dw32<3>;
        if (!allow_lds((const void*)kern, pl.lds_bytes)) return DAQ_ERR_HIP;
        DAQ_LAUNCH("conv_bwd_filter_dw32", st, hipLaunchKernelGGL(kern, grid, dim3(256), pl.lds_bytes, st, a));
    } else {
        auto kern = pl.s2 ? k_dw32_ring<true> : k_dw32_ring<false>;
        if (!allow_lds((const void*)kern, pl.lds_bytes)) return DAQ_ERR_HIP;
        DAQ_LAUNCH("conv_bwd_filter_dw32", st, hipLaunchKernelGGL(kern, grid, dim3(512), pl.lds_bytes, st, a));
    }
    return DAQ_OK;
}

}  // namespace

size_t bwd_filter_lds_ws_bytes(const Plan32& pl, int depth) {
    const int splits = depth == 1 ? std::max(pl.splits, pl.splits_tail) : pl.splits;
    if (!pl.ok || splits == 1) return 0;
    return (size_t)round_up(pl.part_slots * splits * depth * 4, 256);
}

int64_t bwd_filter_lds_row_bytes(const Plan32& pl) { return (int64_t)(pl.nchunks - 1) * kKC + (pl.k11 ? kKC : 16 * pl.b_units); }

daq_status conv_bwd_filter_lds(const daq_conv_desc& d, const Plan32& plan, const int8_t* qx, const float* s_x, const int8_t* vq,
                               const float* s_chan, float* dW, int32_t* acc, void* ws, hipStream_t st, DwTail* defer, bool bf16, const DwDepth* dp) {
    if (defer) defer->blocks = 0;
    const int depth = dp ? dp->kD : 1;
    Plan32 pl = plan;
    if (defer && pl.splits_tail != pl.splits) {
        pl.splits = pl.splits_tail;
        choose_bands(pl, pl.k11 ? 64 : 32, pl.k11 ? 64 : 32);
    }
    if (!pl.ok) return DAQ_ERR_UNSUPPORTED;
    daq_layout Lx, Lg;
    if (daq_layout_qx_cnhw(&d, &Lx) != DAQ_OK || daq_layout_vq(&d, &Lg) != DAQ_OK) return DAQ_ERR_INVALID_ARG;
    const Dw32Args a = fill_args(pl, d, Lx, Lg, qx, s_x, vq, s_chan, dW, acc, ws, bf16, dp);
    if (pl.k11) {
        const dim3 grid((unsigned)pl.blocks, (unsigned)depth);
        if (pl.wk == 1) {
            auto kern = k_dw11<2, 2, 1, 1, 1>;
            if (!allow_lds((const void*)kern, pl.lds_bytes))
                return DAQ_ERR_HIP;
            DAQ_LAUNCH("conv_bwd_filter_dw11", st, hipLaunchKernelGGL(kern, grid, dim3(256), pl.lds_bytes, st, a));
        } else {
            auto kern = dw11_long(ceil_div(pl.nchunks, pl.splits)) ? k_dw11<1, 1, 8, 3, 1, true, true> : k_dw11<1, 1, 8, 3, 1, true>;
            if (!allow_lds((const void*)kern, pl.lds_bytes))
                return DAQ_ERR_HIP;
            DAQ_LAUNCH("conv_bwd_filter_dw11", st, hipLaunchKernelGGL(kern, grid, dim3(512), pl.lds_bytes, st, a));
        }
        return finish(pl, tail_of(pl, a, d, depth), defer, depth, st);
    }
    const daq_status rc = launch32(pl, a, st, depth);
    if (rc != DAQ_OK) return rc;
    return finish(pl, tail_of(pl, a, d, depth), defer, depth, st);
}

bool bwd_filter_beside(const daq_conv_desc& d, Plan32 pl, const int8_t* qx, const float* s_x, const int8_t* vq, const float* s_chan, float* dW,
                       int32_t* acc, void* ws, int max_blocks, double other_us, bool other_streams, DwBeside& out) {
    daq_layout Lx, Lg;
    if (!pl.ok || pl.wk != 8 || pl.s2 || daq_layout_qx_cnhw(&d, &Lx) != DAQ_OK || daq_layout_vq(&d, &Lg) != DAQ_OK) return false;
    const int64_t tiles = (int64_t)pl.tiles_m * pl.tiles_n;
    if (tiles > max_blocks) return false;
    // With the streaming data gradient behind it, which is as short as a launch and takes the reduction along, the product is faster by
    // itself (62 -> 10 at 59 x 59, batch 6: 10.8 us, 12.4 in one launch and a reduction).
    if (other_streams && dw_tail_worthwhile((int)(pl.part_slots / kWave), pl.splits)) return false;
    const bool rides = dw_tail_worthwhile((int)(pl.part_slots / kWave), pl.splits_tail);
    // Otherwise: one after the other, the product has the whole chip; beside the other work what CUs are left, but one launch less (4 ->
    // 395 on 33 x 33, 3 x 3, batch 26, 22 workgroups left: 65 us against 38).  Half the CUs and more are idle in such a launch, a chunk takes
    // 0.4 us (one tap 0.3), and beginning and end are the longer ones of the two parts, 4 us.  Over 630 small layers 0.6 % from the
    // fastest split (with 0.6 and 6.5: 2.1 %, one tap 0.9); together 0.70 of the time apart.
    SplitModel m = split_model(pl, 1);
    const double apart = m.cost(pl.splits_tail) - (rides ? 2.8 : 0.0) + 1.5 + other_us;
    m.t_step = pl.k11 ? 0.3 : 0.4;
    m.t_fixed = 4.0;
    m.limit = std::min<int64_t>(pl.splits, max_blocks / tiles);   // (the workspace holds pl.splits partial tiles)
    m.t_floor = other_us;
    pl.splits = cheapest_split(m);
    if (m.cost(pl.splits) >= apart) return false;
    choose_bands(pl, pl.k11 ? 64 : 32, pl.k11 ? 64 : 32);
    if (pl.blocks > max_blocks) {   // rectangles of unequal size pad the grid
        pl.bands_m = pl.bands_n = 0;
        pl.blocks = tiles * pl.splits;
    }
    out.a = fill_args(pl, d, Lx, Lg, qx, s_x, vq, s_chan, dW, acc, ws, false, nullptr);
    out.k11 = pl.k11;
    out.blocks = (int)pl.blocks;
    out.lds_bytes = pl.lds_bytes;
    out.tail = tail_of(pl, out.a, d, 1);
    if (pl.splits == 1) out.tail.blocks = 0;
    return true;
}

daq_status launch_dw_reduce(const DwTail& t, int depth, hipStream_t st) {
    const unsigned blocks = t.splits > kDwReducePerWave ? (unsigned)t.blocks : (unsigned)ceil_div(t.blocks, 4);
    DAQ_LAUNCH("dw_reduce", st, hipLaunchKernelGGL(k_dw_reduce, dim3(blocks, (unsigned)depth), dim3(256), 0, st, t));
    return DAQ_OK;
}

}  // namespace daq
