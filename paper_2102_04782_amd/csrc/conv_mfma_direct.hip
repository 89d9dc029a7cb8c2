// Channel-contracting int8 implicit GEMM without staging: the data gradient q(G_X) = q(G) (.) q(W) (Eq. "gx", strides 1 and 2) and
// the forward convolution (any stride) of layers whose tiles are too few to fill the chip.
//
//     C[row channel][pixel] = sum over (tap, k)  Wp[tap][row][k] * P[src_pixel(pixel, tap)][k]
//
// The tile kernel (conv_mfma_halo.hip) gives a workgroup 64 rows x 128 or 256 pixels and the whole contraction axis, a step of one
// tap and 64 channels about 0.35 us: 768 -> 52, 5 x 5, 6 images of 5 x 5 is one workgroup and 300 steps.  Here a tile is 32 rows x
// 32 pixels, and the waves of a workgroup share its contraction axis: each walks its part of it in units of 16 contraction bytes
// of one tap, two to an MFMA step (one a half wave), both operands straight from global memory into the registers the MFMA reads,
// and the partial tiles meet in LDS.  What bounds it is those loads, 2 KiB a step and wave through a CU's 64 B/clk, so it does not
// pay where the tile kernel, which reads its pixels from LDS for all taps, has enough workgroups.  A unit belongs to a tap, not a step, so thin
// records (16 channel bytes: a network's first layer) waste none of a step on padding.
#include <algorithm>

#include "daq_internal.h"
#include "dw_tail.h"

namespace daq {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
constexpr int kWaves = 8;                 // of a workgroup
constexpr int kRing = 8;                  // steps requested ahead
constexpr uint32_t kOob = 0x80000000u;    // a buffer offset past every extent: such a load returns zeros
constexpr int kTapRoom = 128;             // taps of a filter, with room for the two entries behind the last one

struct DirectArgs {
    const int8_t* src;    // pixel operand, NHWC [N][Hs][Ws][cp]
    const int8_t* wfrag;  // filter operand in fragment order
    uint32_t src_bytes, wfrag_bytes;
    int N, Hs, Ws, cp, Hd, Wd;
    int Crow, RB, T, kW;
    int fwd, s_log2;      // backward: the stride is 1 << s_log2, and destination pixels are split by parity class
    int sH, sW, pH, pW, dH, dW;
    int PH, PW;           // a class's image
    uint32_t px;          // its pixels, over all images
    int upt;              // 16-byte units of a record
    // live taps of a class, per axis: first, step, number
    int kh0[4], kw0[4], nkh[4], nkw[4], khs, kws;
    int tiles;            // 32 x 32 tiles of a class
    int per_xcd;          // workgroups of a class on an XCD
    FastDiv div_pw, div_php, div_rb, div_upt, div_blocks;
    const float* s_a;
    const float* s_b;
    float* out;
    int32_t* acc_out;
    DwTail tail;
    int main_blocks, bf16;
};

// KS: waves that share a tile
template <int KS>
__global__ __launch_bounds__(kWaves* kWave, 4) void k_conv_direct(DirectArgs p) {
    constexpr int kTiles = kWaves / KS;   // of a workgroup
    __shared__ int4 l_tap[kTapRoom];      // row, column and byte offset of the source, byte offset of the filter
    __shared__ int32_t l_acc[KS > 1 ? kWaves * 16 * kWave : kWaves * kWave];
    if (p.tail.blocks > 0 && (int)blockIdx.x >= p.main_blocks) {   // uniform
        dw_reduce_role(p.tail, (int)blockIdx.x - p.main_blocks, l_acc);
        return;
    }
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = tid % kWave;
    const int l32 = lane & 31, lh = lane >> 5;
    // An XCD takes an eighth of the tiles, neighbours: round-robin, each L2 fetched every pixel (24 x 864 x 31 x 35 -> 17, 5 x 5, 119 -> 92 us;
    // 10 x 32 x 103 x 103 <- 224, 3 x 3, 47 -> 41; 130 products 3 % faster).  Shares by rows instead of pixels gain no more.
    const int cls = (int)fdiv(blockIdx.x, p.div_blocks);
    const int in_cls = (int)blockIdx.x - cls * kXcd * p.per_xcd;
    const int blk = in_cls % kXcd * p.per_xcd + in_cls / kXcd;
    if (blk * kTiles >= p.tiles) return;   // uniform
    const int s = 1 << p.s_log2, pa = cls >> p.s_log2, pb = cls & (s - 1);
    const int taps = p.nkh[cls] * p.nkw[cls];
    for (int t = tid; t < taps + 2; t += kWaves * kWave) {
        const int i = t / max(p.nkw[cls], 1), kh = p.kh0[cls] + i * p.khs, kw = p.kw0[cls] + (t - i * p.nkw[cls]) * p.kws;
        const int oh = p.fwd ? kh * p.dH - p.pH : (pa + p.pH - kh * p.dH) >> p.s_log2;   // exact: the tap is live
        const int ow = p.fwd ? kw * p.dW - p.pW : (pb + p.pW - kw * p.dW) >> p.s_log2;
        l_tap[t] = t < taps ? make_int4(oh, ow, (oh * p.Ws + ow) * p.cp, (kh * p.kW + kw) * p.RB * 2048) : make_int4(1 << 24, 1 << 24, 0, (int)kOob);
    }
    const __amdgpu_buffer_rsrc_t rs_src = __builtin_amdgcn_make_buffer_rsrc((void*)p.src, 0, (int)p.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.wfrag, 0, (int)p.wfrag_bytes, 0x00020000);
    const float scale = (*p.s_a / 127.0f) * (*p.s_b / 127.0f);

    // tile -> (32 pixels, 32 rows): row blocks of the same pixels are neighbours
    const int tile = blk * kTiles + wave / KS, part = wave % KS;
    const bool live_tile = tile < p.tiles;   // uniform per wave
    const int tp = (int)fdiv((uint32_t)(live_tile ? tile : 0), p.div_rb), rb = (live_tile ? tile : 0) - tp * p.RB;
    const uint32_t P = (uint32_t)tp * 32u + (uint32_t)l32;
    const bool ok = live_tile && P < p.px;
    const uint32_t Pc = P < p.px ? P : 0u;
    const int n = (int)fdiv(Pc, p.div_php);
    const int rem = (int)(Pc - (uint32_t)n * (uint32_t)(p.PH * p.PW));
    const int th = (int)fdiv((uint32_t)rem, p.div_pw), tw = rem - th * p.PW;
    const int hb = ok ? (p.fwd ? th * p.sH : th) : -(1 << 23), wb = p.fwd ? tw * p.sW : tw;
    const int base = ((n * p.Hs + (p.fwd ? th * p.sH : th)) * p.Ws + wb) * p.cp;
    const uint32_t a_lane = (uint32_t)(rb * 2048 + l32 * 16), chunk = (uint32_t)(p.T * p.RB) * 2048u;

    const int steps = (taps * p.upt + 1) / 2;
    const int first = steps * part / KS, end = steps * (part + 1) / KS;
    int tap = (int)fdiv((uint32_t)(2 * first + lh), p.div_upt), q = 2 * first + lh - tap * p.upt;
    v4i A[kRing], B[kRing];
    int next = first;
    auto fetch = [&](int slot) {
        const bool live = next < end;   // uniform
        const int4 e = l_tap[live ? tap : taps];
        const bool in = (unsigned)(hb + e.x) < (unsigned)p.Hs && (unsigned)(wb + e.y) < (unsigned)p.Ws;
        const uint32_t boff = in ? (uint32_t)(base + e.z + 16 * q) : kOob;
        const uint32_t aoff = (uint32_t)e.w + ((uint32_t)q >> 2) * chunk + ((uint32_t)q & 3u) * 512u + a_lane;
        A[slot] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, (int)aoff, 0, 0);
        B[slot] = __builtin_amdgcn_raw_buffer_load_b128(rs_src, (int)boff, 0, 0);
        ++next;
        q += 2;
#pragma unroll
        for (int k = 0; k < 2; ++k) {   // a record of one unit: two taps on
            const bool over = q >= p.upt;
            tap += over ? 1 : 0;
            q -= over ? p.upt : 0;
        }
    };
    v16i acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0;
    __syncthreads();
#pragma unroll
    for (int d = 0; d < kRing - 1; ++d) fetch(d);
    for (int s0 = first; s0 < end; s0 += kRing) {
#pragma unroll
        for (int u = 0; u < kRing; ++u) {   // (steps past the end multiply zeros)
            fetch((u + kRing - 1) % kRing);
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[u], B[u], acc, 0, 0, 0);
        }
    }

    // register r: row 8*(r/4) + 4*lh + r%4 of the row block, the lane's pixel
    const int h = (th << (p.fwd ? 0 : p.s_log2)) + (p.fwd ? 0 : pa), w = (tw << (p.fwd ? 0 : p.s_log2)) + (p.fwd ? 0 : pb);
    const bool inside = ok && h < p.Hd && w < p.Wd;
    const int HWd = p.Hd * p.Wd, row0 = 32 * rb + 4 * lh;
    const int64_t at = ((int64_t)n * p.Crow + row0) * HWd + h * p.Wd + w;
    float* const out = p.out;
    int32_t* const acc_out = p.acc_out;
    const int bf16 = p.bf16, Crow = p.Crow;
    auto store = [&](int r, int32_t v) {
        const int dr = 8 * (r >> 2) + (r & 3);
        if (!inside || row0 + dr >= Crow) return;
        store_result(out, at + (int64_t)dr * HWd, (float)v * scale, bf16);
        if (acc_out) acc_out[at + (int64_t)dr * HWd] = v;
    };
    if constexpr (KS == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) store(r, acc[r]);
    } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) l_acc[(wave * 16 + r) * kWave + lane] = acc[r];
        __syncthreads();
        constexpr int kEach = 16 / KS;   // registers of the tile a wave sums up and stores
        const int w0 = wave - part;
#pragma unroll
        for (int i = 0; i < kEach; ++i) {
            const int r = part * kEach + i;
            int32_t v = 0;
#pragma unroll
            for (int k = 0; k < KS; ++k) v += l_acc[((w0 + k) * 16 + r) * kWave + lane];
            store(r, v);
        }
    }
}

struct DirectPlan {
    bool ok;
    DirectArgs a;
    int ks;
    int64_t blocks;
};

DirectPlan plan_direct(bool backward, const daq_conv_desc& d) {
    DirectPlan g{};
    daq_layout Ls;
    daq_wpack_layout Lw;
    if (d.groups != 1 || d.kH * d.kW > kTapRoom - 2 || daq_layout_qw(&d, &Lw) != DAQ_OK) return g;
    if ((backward ? daq_layout_qg(&d, &Ls) : daq_layout_qx_nhwc(&d, &Ls)) != DAQ_OK || Ls.kind != DAQ_LAYOUT_NHWC) return g;
    if (backward && (d.strideH != d.strideW || d.strideH > 2)) return g;
    const int64_t wbytes = backward ? Lw.bytes - Lw.off_bwd_frag : Lw.off_bwd_frag - Lw.off_fwd_frag, lim = (int64_t)1 << 31;
    if (Ls.bytes >= lim || wbytes >= lim) return g;
    DirectArgs& a = g.a;
    a.src_bytes = (uint32_t)Ls.bytes;
    a.wfrag_bytes = (uint32_t)wbytes;
    a.N = d.N; a.Hs = Ls.H; a.Ws = Ls.W; a.cp = Ls.c_pitch;
    a.Hd = backward ? d.Hin : daq_out_h(&d);
    a.Wd = backward ? d.Win : daq_out_w(&d);
    a.Crow = backward ? d.Cin : d.Cout;
    a.RB = (int)ceil_div(a.Crow, 32);
    a.T = d.kH * d.kW; a.kW = d.kW;
    a.fwd = backward ? 0 : 1;
    a.s_log2 = backward && d.strideH == 2 ? 1 : 0;
    a.sH = d.strideH; a.sW = d.strideW; a.pH = d.padH; a.pW = d.padW; a.dH = d.dilH; a.dW = d.dilW;
    if (std::max((int64_t)d.kH * d.dilH, (int64_t)d.kW * d.dilW) + std::max(d.padH, d.padW) >= (1 << 20)) return g;
    if ((int64_t)std::max(a.Hd, a.Hs) + std::max(a.Wd, a.Ws) >= (1 << 20)) return g;
    const int s = 1 << a.s_log2, classes = s * s;
    a.khs = a.s_log2 && (d.dilH & 1) ? 2 : 1;
    a.kws = a.s_log2 && (d.dilW & 1) ? 2 : 1;
    // taps of one axis that reach parity p: those with p + pad - k * dil even - all or none where the dilation is even
    auto axis = [&](int p, int pad, int dil, int k, int& k0, int& num) {
        k0 = 0;
        num = k;
        if (!a.s_log2) return;
        if (dil & 1) {
            k0 = (p + pad) & 1;
            num = k > k0 ? (k - k0 + 1) / 2 : 0;
        } else if ((p + pad) & 1) {
            num = 0;
        }
    };
    for (int c = 0; c < classes; ++c) {
        axis(c >> a.s_log2, d.padH, d.dilH, d.kH, a.kh0[c], a.nkh[c]);
        axis(c & (s - 1), d.padW, d.dilW, d.kW, a.kw0[c], a.nkw[c]);
    }
    a.PH = (int)ceil_div(a.Hd, s);
    a.PW = (int)ceil_div(a.Wd, s);
    const int64_t px = (int64_t)d.N * a.PH * a.PW, tiles = ceil_div(px, 32) * a.RB;
    if (px >= lim - 64 || tiles >= lim / 8) return g;
    a.px = (uint32_t)px;
    a.tiles = (int)tiles;
    a.upt = a.cp / 16;
    a.div_pw = make_fastdiv((uint32_t)a.PW);
    a.div_php = make_fastdiv((uint32_t)(a.PH * a.PW));
    a.div_rb = make_fastdiv((uint32_t)a.RB);
    a.div_upt = make_fastdiv((uint32_t)a.upt);
    const int64_t steps = ceil_div((int64_t)a.T * a.upt, 2 * classes);
    // as many waves to a tile as there are tiles too few, a wave at least four steps
    g.ks = 1;
    const int64_t waves = steps < 40 ? 2048 : 4096;
    while (g.ks < kWaves && tiles * classes * g.ks < waves && steps >= 4 * g.ks) g.ks *= 2;
    a.per_xcd = (int)ceil_div(ceil_div(tiles, kWaves / g.ks), kXcd);
    a.div_blocks = make_fastdiv((uint32_t)(kXcd * a.per_xcd));
    g.blocks = (int64_t)kXcd * a.per_xcd * classes;
    g.ok = g.blocks < lim - 4096;
    return g;
}

// Both sides' costs in us, one launch between events, fitted to products of random layers (here and the last two columns there to 992, the others to 680 as
// the forms are now); MB of result included:
//     here   7.6 + 0.13 * steps of a wave + 27 * thousands of steps a CU + 0.27 * MB (by parity class, every other pixel of a line: 0.55)
//            + 0.09 * (tiles a CU beyond 40) + 0.28 * (MB of source beyond 16, which the L2s no longer hold)
//     there  fixed + (step + turn * max(1, workgroups / 256)) * steps of a workgroup + mb * MB
// These kernels are taken where they are 3 % faster by that, 20 % from 60 us on, where few were fitted (1280 <- 824, 5 x 5, 17 of 7 x 7, 102 us there and 134
// here): of 1080 products 80 then go to the form that is more than 2 % slower (114 with the prices of the
// forms before: 208 <- 637, 3 x 3, 2 of 27 x 27, went here, 18.6 us, 13.8 there).  E.g. 768 -> 52, 5 x 5, 6 images of 5 x 5, 97 us there and 14 here; 3 -> 96, 7 x 7
// stride 2, 23 of 16 x 16, 46 and 7; 256 -> 304, 5 x 5, 3 of 15 x 15, 37 and 20.
//   The model holds less well for the 1 x 1 ring form, several workgroups of which share a CU, and the re-staging form (13 to 20 % off: 512 <- 2048 at 7 x 7, batch 128,
// 23.4 us there, 47 here): against those these have to be 7 % faster, 20 % from 30 us on, and not for 1 x 1 layers of many workgroups; and forward
// + 2 * MB of filter, which the launch before has just written, count here (against the other forms that sent 400 <- 224, 5 x 5, 16 of 12 x 12, there, with
// the quantizers 61 us, 49.5 here; of 120 forward products 12 to the slower form, 3 without it).
// The line about large tensors came from products of 5 to 130 MB of source: 1219 -> 16 1 x 1, 16 of 63 x 50, 27 there and 35
// here, 1093 -> 16, 64 of 31 x 17, 17 and 23; 7 -> 4 3 x 3, 71 of 135 x 135, 36 and 49; 5 <- 10 5 x 5 stride 2, 101 of 123 x 123, 45 and 57.  It does
// not count against the re-staging form, whose own cost such products are further above its fit (3 -> 96 3 x 3 stride 2, 39 of 133 x 133, 56 there and 32 here).
bool faster(const DirectPlan& g, const OtherKernel& o, int classes, bool bf16) {
    struct Cost { double fixed, step, turn, mb; };
    //                             3 x 3                       32 rows at most            any taps                    1 x 1, ring                  re-staging
    static const Cost kUnit[] = {{6.74, -0.089, 0.195, 0.303}, {7.04, 0.061, 0.187, 0.17}, {7.95, 0.1, 0.205, 0.242}, {5.6, -0.35, 0.69, 0.32}, {11.6, -1.53, 2.13, 0.4}};
    static const Cost kClasses[] = {{0, 0, 0, 0}, {7.21, 0.275, 0.007, 0.328}, {8.0, 0.095, 0.26, 0.285}, {8.0, 0.1, 0.1, 0.2}, {0, 0, 0, 0}};
    const DirectArgs& a = g.a;
    const double mb = (double)a.N * a.Crow * a.Hd * a.Wd * (bf16 ? 2 : 4) * 1e-6;
    const double steps = (double)ceil_div((int64_t)a.T * a.upt, 2 * classes), tiles = (double)a.tiles * classes;
    const bool rough = o.form == TileForm::kRing1 || o.form == TileForm::kNhwc;
    const double here = 7.6 + 0.13 * steps / g.ks + 27.0 * tiles * steps / 256e3 + (classes > 1 ? 0.55 : 0.27) * mb +
                        (a.fwd && rough ? 2e-6 * a.wfrag_bytes : 0.0);
    const double read = 1e-6 * a.src_bytes / (a.fwd && a.T == 1 ? a.sH * a.sW : 1);
    const double large = o.form == TileForm::kNhwc ? 0.0 : 0.09 * std::max(0.0, tiles / 256.0 - 40.0) + 0.28 * std::max(0.0, read - 16.0);
    const Cost& c = (o.classes ? kClasses : kUnit)[(int)o.form];
    const double held = o.form == TileForm::kNhwc ? 512.0 : 256.0;
    const double there = c.fixed + (c.step + c.turn * std::max(1.0, (double)o.blocks / held)) * o.steps + c.mb * mb;
    const double margin = there > (rough ? 30.0 : 60.0) ? 0.8 : rough ? 0.93 : 0.97;
    return (o.form != TileForm::kRing1 || o.blocks <= 512) && here + large < margin * there;
}

daq_status launch_direct(DirectPlan& g, const char* name, const DwTail* tail, hipStream_t st) {
    DirectArgs& a = g.a;
    if (tail) a.tail = *tail;
    a.main_blocks = (int)g.blocks;
    const dim3 grid((unsigned)(g.blocks + a.tail.blocks));
    auto kern = g.ks == 1 ? k_conv_direct<1> : g.ks == 2 ? k_conv_direct<2> : g.ks == 4 ? k_conv_direct<4> : k_conv_direct<8>;
    DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, grid, dim3(kWaves * kWave), 0, st, a));
    return DAQ_OK;
}

}  // namespace

static DirectPlan direct_if_faster(bool backward, const daq_conv_desc& d, const OtherKernel& other, bool bf16) {
    DirectPlan g = plan_direct(backward, d);
    g.ok = g.ok && faster(g, other, backward ? 1 << 2 * g.a.s_log2 : 1, bf16);
    return g;
}

int direct_waves(bool backward, const daq_conv_desc& d, const OtherKernel& other, bool bf16) {
    const DirectPlan g = direct_if_faster(backward, d, other, bf16);
    return g.ok ? g.ks : 0;
}

bool conv_direct(bool backward, const daq_conv_desc& d, const OtherKernel& other, const int8_t* src, const int8_t* qw, const float* s_a,
                 const float* s_b, float* out, int32_t* acc, hipStream_t st, const DwTail* tail, bool bf16, daq_status& rc) {
    DirectPlan g = direct_if_faster(backward, d, other, bf16);
    daq_wpack_layout Lw;
    if (!g.ok || daq_layout_qw(&d, &Lw) != DAQ_OK) return false;
    g.a.src = src;
    g.a.wfrag = qw + (backward ? Lw.off_bwd_frag : Lw.off_fwd_frag);
    g.a.s_a = s_a; g.a.s_b = s_b;
    g.a.out = out; g.a.acc_out = acc;
    g.a.bf16 = bf16 ? 1 : 0;
    rc = launch_direct(g, backward ? "conv_bwd_data_direct" : "conv_fwd_direct", tail, st);
    return true;
}

}  // namespace daq
