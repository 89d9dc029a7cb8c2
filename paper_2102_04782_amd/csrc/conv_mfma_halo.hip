// Channel-contracting int8 implicit GEMM, halo-tile form: the data gradient q(G_X) = q(G) (.) q(W)
// (Eq. "gx") for strides 1 and 2, and the unit-stride forward convolution.
//
//     C[row channel][pixel] = sum over (tap, k)  Wp[tap][row][k] * P[src_pixel(pixel, tap)][k]
//
// A workgroup owns NI images x (TH x TW) destination pixels (<= 256) and 64 row channels (128 in one form).
// Per 64-byte chunk of the contraction axis it stages the SOURCE WINDOW of its tile in LDS once -
// (TH + reach) x (TW + reach) pixel slots of 64 channel bytes - and every filter tap reads that
// window at a shifted slot, so no pixel is staged more than once and the loop over the taps has no
// LDS writes and no barrier.  The filter operand never goes through LDS: it is stored in fragment
// order (see daq_wpack_layout), so a wave fetches each 32-row x 32-byte tile as one contiguous KiB
// straight into the registers the MFMA reads, one step ahead.  The window of the next chunk is
// fetched while the taps of the current one run and is written to the other LDS buffer at the
// chunk's last tap: one barrier per chunk.
//
// Stride 2 (data gradient only): destination pixels are split by parity (h % 2, w % 2).  Pixels of
// one parity class see the same subset of taps, each at a unit-stride position of the source, so a
// workgroup handles one class and issues only the taps that are live for it - no multiplies by
// stride-skipped zeros.
#include <algorithm>
#include <cstddef>

#include "daq_internal.h"
#include "dw32_role.h"
#include "dw_tail.h"

namespace daq {

// Blocks of the streaming form that an XCD takes in a row (0: block by block).  A pair of row blocks of four pixel groups is a block, 512 bytes of each of
// its planes.  Where planes are no multiple of 64 bytes neighbouring blocks share lines, which then meet in one L2: an eighth of
// the blocks each (384 <- 64 at 14 x 14, batch 128, operands from memory, 16.9 us dealt out one by one, 13.0; 48 <- 16 at 45 x 45, batch 86, 14.4 and
// 11.9) or, of large results, which lose the order of their pages that way, eight quads (320 <- 16 at 61 x 61, batch 34, 57.4, 52.5 by
// eighths, 49.8; 244 <- 32 at 79 x 75, batch 27, 56, 53 and 48), or two where a wave of many channels leaves few blocks to deal (1368 <- 192 at 75 x 75,
// batch 12, 168 and 161; four pairs and fewer are enough for eight: 240 <- 256 at 45 x 44, batch 84, 62.9 and 61.1).  On other planes only the source is shared, among the pairs of row blocks: four quads from
// four pairs and 128 bytes a pixel on (512 <- 256 at 28 x 28, batch 64, 35.1 and 26.1; 144 <- 24 at 56 x 56, batch 128, three pairs, 44.8 and 45.4, 336 <- 32 at
// 52 x 52, batch 50, 39.6 and 42.6: not there) up to sixteen pairs (1776 <- 128 at 24 x 26, batch 18, 28 pairs, 21.5 and 23.9).
//   Lines shared and a multiple of eight pairs: one by one, an XCD has the same row blocks of every quad, neighbours meet anyway, and the pages keep their order
// (1499 <- 59 at 43 x 43, batch 50, 180 us and 208 dealt; 512 <- 16 at 22 x 22, batch 44, 12.3 and 14.1), but for eight pairs of many
// channels, whose source counts too (480 <- 256 at 50 x 51, batch 65, 143 us and 132).  So it nearly is with 27 pairs and more, and what
// is won is less than the order of large results (1936 <- 48 at 20 x 18, batch 53, 31 pairs, 45.4 and 50.6; 26 pairs: 1616 <- 56 at 67 x 67, batch 4,
// 35.4 and 32.9; 1664 <- 24 at 72 x 73, batch 11, 129.5 and 131.8).
int64_t stream_deal(int64_t out_bytes, int64_t plane_bytes, int cp, int pairs, int64_t blocks) {
    if (plane_bytes % 64 == 0) return pairs >= 4 && pairs <= 16 && cp >= 128 ? 4 * pairs : 0;
    const bool large = out_bytes > (48 << 20), many = cp > 128;
    if (pairs % kXcd == 0 && !(large && many && pairs == kXcd)) return 0;
    if (!large) return blocks / kXcd;
    if (many) return (pairs >= 5 ? 2 : 8) * pairs;
    return pairs >= 27 ? 0 : 8 * pairs;
}

// Whether two tiles of a 1 x 1 product share a 64-byte line of the result: not where they are whole images, or whole rows or pieces of rows that begin and
// end with a line.
static bool tiles_share_lines(int TH, int TW, int tiles_h, int tiles_w, int stride, int Hd, int Wd, int bytes) {
    if (tiles_h * tiles_w == 1) return false;
    if (tiles_w > 1) return (int64_t)stride * TW * bytes % 64 != 0 || (int64_t)Wd * bytes % 64 != 0;
    return (int64_t)stride * TH * Wd * bytes % 64 != 0 || (int64_t)Hd * Wd * bytes % 64 != 0;
}

// 1 x 1 products on 128-pixel tiles, whose workgroups all run at once: where no two tiles share a line of the result
// only the filter is left to share, and the blocks go out one by one, row tile after row tile, all tiles of one filter tile together.  (Operands from memory, tile after tile and so: 512 <- 2048 at 7 x 7, batch 128, 24.0 us and 23.4; 256 <- 768 at 48 x 48,
// batch 4, 1.12 times the speed; 105 layers at stride 2 1.018, 12 at unit stride with cut images 1.03.)  Not with many tiles that are no multiple of eight:
// the row tiles of one then lie on several XCDs, each of which fetches its window (512 <- 80 at stride 2, 24 x 24, batch 33, 66 tiles, 13.8 and 15.3;
// 928 <- 1104 at 7 x 7, batch 82, 41 tiles, 22.3 and 24.2).
bool tiles_by_rows(int TH, int TW, int tiles_h, int tiles_w, int stride, int Hd, int Wd, int bytes, int64_t tiles, int row_tiles) {
    if (tiles % kXcd != 0 && tiles >= 32 && row_tiles > 3) return false;
    return !tiles_share_lines(TH, TW, tiles_h, tiles_w, stride, Hd, Wd, bytes);
}

// 1 x 1 products at unit stride on 256-pixel tiles that share no line: an eighth of the result to each XCD has them write eight places at once whose
// distance may be one of the memory channels' (48 x 48: 512 <- 320, batch 58, 148 us; 256 <- 320, batch 62, 82).  An XCD has
// every eighth tile instead, still with all its row tiles, and the chip writes one place (118 and 71; 1.05 times the speed over 25 layers of more
// than 1000 workgroups, worst 0.98).  Of fewer workgroups only where that leaves no tile over (1024 <- 384 at 20 x 20, batch 19, 38 tiles, 0.89 times the speed).
bool tiles_spread(int TH, int TW, int tiles_h, int tiles_w, int Hd, int Wd, int bytes, int64_t tiles, int row_tiles) {
    if (tiles % kXcd != 0 && tiles * row_tiles <= 1000) return false;
    return !tiles_share_lines(TH, TW, tiles_h, tiles_w, 1, Hd, Wd, bytes);
}

// A run-time tap list: whether the waves take 32 rows x 128 pixels instead of 64 x 64 (see halo_role), from 512 workgroups on.  Not with several
// chunks of many taps, 28 steps (tap x chunk) and more: beginning and end, which a second workgroup on the CU hides, are little of those, and a step
// of 64 x 64 reads LDS half as often (848 <- 144 forward, 5 x 5 at 24 x 24, batch 34, with the quantizers 149 us wide, 140; 723 <- 376, 5 x 5, 18 x 18, batch 37, 0.945 of the time; 45 layers
// 0.97, of fewer steps 1.01, of one chunk 1.06).
bool wide_waves(int64_t blocks, int chunks, int taps) { return blocks > 512 && !(chunks > 1 && chunks * taps >= 28); }

// The same of 1 x 1 filters, 256-pixel tiles: from 2048 workgroups on, and at stride 2 on rows of odd length, whose results leave element by
// element: two workgroups to a CU then hide that (64 x 64 and wide: 1128 <- 64 at 17 x 17, batch 25, 25.7 us and 21.3; 1146 <- 192 at 41 x 41, batch 13, 60.2 and 52.7; 80 <- 192
// at 49 x 49, batch 72, 1.13 times the speed; 24 layers 1.08, none slower.  On rows of even length 0.90 to 1.10, 29 layers 1.00).
bool wide_waves1(int64_t blocks, int stride, int Wd) { return blocks > 2048 || (stride == 2 && (Wd & 1)); }

namespace {

constexpr int kPxWg = 256;         // destination pixels per workgroup (128 in the small-tile form of 1 x 1 filters)
constexpr int kKc = 64;            // contraction bytes per step (two MFMA K-steps of 32)
constexpr int kPitch = kKc + 16;   // LDS pitch of a window slot: eight consecutive slots cover all banks
constexpr int kMaxTaps = 49;
constexpr int kMaxUnits = 8;       // 16-byte units of the window a thread stages: up to 512 slots
constexpr int kMaxPhases = 4;
constexpr int kRingA = 4;          // filter tiles are requested kRingA - 1 steps ahead of their use
constexpr uint32_t kOob = 0x80000000u;  // a buffer offset past every extent: such a load returns zeros

struct alignas(64) HaloArgs {
    // What a workgroup finds its tile by, in one line of 64 bytes: arguments arrive in such lines, a quarter of a microsecond each when one is asked for
    // behind another.  Then what it needs up to its first loads.
    int main_blocks;      // the product's workgroups; those behind them finish a deferred filter gradient (tail)
    int by_rows;          // tiles_by_rows
    int row_tiles;        // (by_rows: the tiles of a row tile)
    int tiles_h, tiles_w;
    int zfill;            // stride 2, only parity class (0, 0) has taps: its workgroups also write the zeros of the other three
    FastDiv div_row_tiles, div_tiles_hw, div_tiles_w;
    int spread;           // tiles_spread: the workgroups of whole eights of tiles
    int NI, TH, TW;       // destination tile, NI images, in pixels of one parity class
    int SH, SW;           // source window per image (the largest over the classes)
    int N, Hs, Ws, cp;
    int units;            // 16-byte window units per thread
    FastDiv div_si, div_sw;
    const int8_t* src;    // pixel operand, NHWC [N][Hs][Ws][cp]
    const int8_t* wfrag;  // filter operand in fragment order
    uint32_t src_bytes, wfrag_bytes;
    const float* s_a;
    const float* s_b;
    int RB, T;            // 32-row blocks of the filter copy, kH*kW
    // per parity class: live taps, window origin relative to the tile's first pixel
    int ph_taps[kMaxPhases], ph_org_h[kMaxPhases], ph_org_w[kMaxPhases];
    FastDiv div_tw, div_thw;
    int double_buffer;    // more than one contraction chunk: two window buffers
    int Hd, Wd;
    int Crow;             // result channels
    int stride;           // 1, or 2 (parity classes)
    int groups;
    int bf16;             // the result is stored as bfloat16 (round to nearest even) instead of fp32
    int nt;               // the result is large: streaming stores, so that it does not push the next kernels' operands out of the caches
    float* out;           // fp32 [N][Crow][Hd][Wd]
    int32_t* acc_out;
    // 3-D layers: an "image" is one frame of a sample, N counts frames, and the contraction runs over kD depth taps of nkc_frame
    // chunks each (see D3 below)
    int Dd, Ds, kD, sD_log2, pD, dD, fwd, nkc_frame;
    FastDiv div_dd, div_nkc;
    DwTail tail;          // tail.blocks > 0: that many workgroups behind the first main_blocks finish a deferred filter
                          // gradient instead (they are dispatched last and fill the slots this kernel's own tiles leave)
    // 32-bit entries: a uniform index then costs a scalar load, not a vector-memory round trip
    int tap_slot[kMaxPhases][kMaxTaps];  // slot offset a tap adds inside the window
    int tap_id[kMaxPhases][kMaxTaps];    // kh*kW + kw of the tap
};
static_assert(offsetof(HaloArgs, NI) == 64 && offsetof(HaloArgs, src) == 128 && offsetof(HaloArgs, ph_org_h) <= 192, "lines of arguments");

__device__ __forceinline__ v4i buffer_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voffset, uint32_t soffset) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voffset, (int)soffset, 0);
}

// WR = waves along the row (output channel) axis, WAVES = waves per workgroup; a wave owns 32 * NX rows (64 with WR = 1) and an equal share of
// the PX pixels.  On four waves: (WR 1, NX 2) 64 rows x 64 pixels each, (WR 2, NX 1) 32 x 128 (PX = 256) or 32 x 64 (PX = 128).  On eight:
// (WR 2, NX 2) 64 x 64, a workgroup of 128 rows.
//   Filter tiles come through the vector memory pipe, 64 bytes a clock for the whole CU, pixels from LDS, 128 bytes a clock.  With waves of 64 x 64 each of the
// four asks for the same 4 KiB of filter a step, 256 clocks for 256 of multiplies, and registers allow one workgroup to a CU, so that its prologue, its
// barriers and its stores show.  With 32 x 128 a wave asks for 2 KiB, LDS delivers twice as much, and two workgroups fit (3 x 3: 245 registers for 310, 250 in 3-D).
// Data gradient, operands from memory: 312 <- 80, 3 x 3 at 41 x 41, batch 40, 63.6 us and 41.7; 400 <- 16 at 49 x 49, batch 53, 62 and 49; 451 <- 368 at 15 x 15,
// batch 66, 47 and 38; 1.13 times the speed over 24 drawn 3 x 3 layers.  128-pixel tiles of 3 x 3 filters: 512 <- 512 at 7 x 7, batch 64, 16.6 us with 64 x 32,
// 13.8 with 32 x 64.  What is left is where a step with fewer reads of LDS is the shorter one, hardly a workgroup to a CU or hardly any arithmetic:
// 64 x 64 up to 512 workgroups with a run-time tap list or with many steps (wide_waves; 80 <- 992, 5 x 5 at 34 x 34, batch 37, 141 us and 154), up to 2048 of 1 x 1 filters (wide_waves1; 512 <-
// 1024 at 14 x 14, batch 64, 22.5 and 23.5; beyond, 912 <- 560 at stride 2, 81 x 81, batch 75, 650 and 601), 64 x 32 for 128-pixel tiles of 1 x 1 filters (2048 <- 512 at
// 7 x 7, batch 64, 18.2 and 21.5).
// DB = the contraction axis has more than one 64-byte chunk (two window buffers, restaged per chunk).
// ST = stride (1 or 2): with one parity class its tables are indexed with constants.
// TAPS > 0 (unit stride; TAPS = 1 also stride 2 with a single live parity class): the number of filter taps is this constant.  The loop over the taps of a chunk is
// then unrolled, the ring of filter tiles has one slot per tap (slot = tap, so each tile is requested TAPS - 1
// steps before its use), the tap tables are read once, and the pixel fragments of the next tap are read from LDS
// before the multiplies of the current one: with one or two waves per SIMD little else hides those latencies.
// NX = 32-row blocks of a wave that can hold result rows; WR = 1, NX = 1 is for results of at most 32 channels (the data gradient of a
// network's first layer), whose second block would only multiply zeros - dynamic-tap form only.
// PX = destination pixels per workgroup: 128 for layers with so few pixels that 256-pixel tiles would leave CUs without a workgroup.
// D3: a 3-D layer.  Its frames are the images of the tile; a depth tap kd of the filter reads the same window of another
// frame of the sample (zeros where there is none), so the depth taps are further chunks of the contraction axis - chunk
// kd * nkc_frame + kc - and nothing else in the loop changes; the filter copy is in the same order (k_frag3 writes it).
// (3 x 3 x 3, 64 -> 64, 8 x 56 x 56, batch 8, data gradient: 365 us with dot products, 36 us here.)
template <int WR, bool DB, int ST, int WAVES, int TAPS, int NX, int PX, bool D3>
__device__ __forceinline__ void halo_role(const HaloArgs& p, const uint32_t bid) {
    constexpr int RW = WR == 1 ? 64 : 32 * NX, ROWS = RW * WR;   // result rows of a wave, of the workgroup
    constexpr int WPX = WAVES / WR;
    constexpr int SPT = 16 * WAVES;   // window slots one pass of the workgroup stages (four lanes per slot)
    constexpr int PXW = PX / WPX;
    constexpr int BF = PXW / 32;
    extern __shared__ __align__(16) int8_t lds[];   // one or two window buffers of S slots

    // (kept whole by the empty statement: the compiler would ask piece by piece, with a wait for each)
    uint32_t main_blocks = (uint32_t)p.main_blocks, row_tiles = (uint32_t)p.row_tiles, rows_first = (uint32_t)p.by_rows, spread = (uint32_t)p.spread;
    int tiles_h = p.tiles_h, tiles_w = p.tiles_w, zfill = p.zfill;
    FastDiv div_row_tiles = p.div_row_tiles, div_tiles_hw = p.div_tiles_hw, div_tiles_w = p.div_tiles_w;
    asm volatile("" : "+s"(main_blocks), "+s"(row_tiles), "+s"(rows_first), "+s"(spread), "+s"(tiles_h), "+s"(tiles_w), "+s"(zfill), "+s"(div_row_tiles.mul),
                      "+s"(div_row_tiles.shift), "+s"(div_row_tiles.one), "+s"(div_tiles_hw.mul), "+s"(div_tiles_hw.shift), "+s"(div_tiles_hw.one),
                      "+s"(div_tiles_w.mul), "+s"(div_tiles_w.shift), "+s"(div_tiles_w.one) : "s"(p.TH), "s"(p.src));   // (and the next two lines are on their way)
    const int NI = p.NI;
    if (bid >= main_blocks) {   // uniform
        dw_reduce_role(p.tail, (int)(bid - main_blocks), reinterpret_cast<int32_t*>(lds));
        return;
    }
    const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
    const int l32 = lane & 31, lh = lane >> 5;
    const int wr = wave % WR, wp = wave / WR;
    // block -> (image group, tile row, tile column, row tile, parity class)
    // Blocks i, i + 8, i + 16, ... run on one XCD: it takes an eighth of that list, in its order.  Neighbouring tiles share lines of the
    // result (a row of a tile seldom ends with a line), and the four parity classes of a tile interleave in memory pixel by pixel: their
    // pieces meet in one L2 instead of going to memory one by one, and a window is fetched into one L2 for all row tiles.  (Dealt out tile by
    // tile, row tile after row tile: data gradient of 384 <- 129, 1 x 1 at stride 2, 86 x 86, batch 94, 210 us and 154 here; of 128 <- 128, 3 x 3 at
    // stride 2, 56 x 56, batch 64, 60.8 and 51; 1.10 times the speed over 50 drawn layers, of which every twelfth is slower, by up to 6 %: 256 <-
    // 512, 1 x 1 at stride 2, 56 x 56, batch 64, 59.8 and 63.  An XCD's tiles 4 or 16 at a time, or its row tiles one after the other, were slower.)
    const uint32_t xcd = bid % kXcd, each = main_blocks / kXcd, more = main_blocks % kXcd;
    const bool by_rows = TAPS == 1 && PX == 128 && rows_first != 0;   // tiles_by_rows: the blocks' own order, row tile after row tile
    constexpr bool kSpread = TAPS == 1 && PX == kPxWg && ST == 1;
    const bool dealt = kSpread && bid < spread;   // tiles_spread: of every eight tiles an XCD has one, with all its row tiles; what is left over, block by block
    uint32_t at = by_rows || (kSpread && spread > 0 && !dealt) ? bid : bid / kXcd + (dealt ? 0u : xcd * each + min(xcd, more));
    int phase = 0;
    if (ST > 1 && !zfill) {
        phase = (int)(at % (ST * ST));
        at /= ST * ST;
    }
    const int quot = (int)fdiv(at, div_row_tiles), left = (int)(at - (uint32_t)quot * row_tiles);   // (by rows: of the tiles of a row tile)
    const int tp = by_rows ? left : dealt ? quot * kXcd + (int)xcd : quot, tr = by_rows ? quot : left;
    const int pa = phase / ST, pb = phase % ST;
    const int grp = (int)fdiv((uint32_t)tp, div_tiles_hw);
    const int trem = tp - grp * tiles_h * tiles_w;
    const int tih = (int)fdiv((uint32_t)trem, div_tiles_w);
    const int tiw = trem - tih * tiles_w;
    const int row0 = tr * ROWS;
    const int n0 = grp * NI, h0 = tih * p.TH, w0 = tiw * p.TW;
    const int SI = p.SH * p.SW, S = NI * SI;
    const int halo_bytes = S * kPitch;
    const int nkc = D3 ? p.kD * p.nkc_frame : (p.cp + kKc - 1) / kKc;
    const int taps = p.ph_taps[phase];
    const int NS = nkc * taps;
    const int org_h = p.ph_org_h[phase], org_w = p.ph_org_w[phase];

    const __amdgpu_buffer_rsrc_t rs_src = __builtin_amdgcn_make_buffer_rsrc((void*)p.src, 0, (int)p.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.wfrag, 0, (int)p.wfrag_bytes, 0x00020000);
    // the de-quantization factor is requested here, not in the epilogue, where its latency would show
    const float scale = (*p.s_a / 127.0f) * (*p.s_b / 127.0f);

    // ---- window staging: unit i of a thread is chunk (tid & 3) of slot (tid >> 2) + SPT*i ----
    const int sc = tid & 3;
    uint32_t hoff[kMaxUnits];
    // D3: the destination frame's depth (below 65536, plan3), two in a register where those are scarce; hoff is then the offset in frame 0 of the sample
    constexpr bool kPacked = D3 && TAPS == 9 && PX == kPxWg;
    uint32_t hz[D3 ? kPacked ? kMaxUnits / 2 : kMaxUnits : 1] = {};
#pragma unroll
    for (int i = 0; i < kMaxUnits; ++i) {
        hoff[i] = kOob;
        if (i < p.units) {   // uniform
            const int slot = (tid >> 2) + SPT * i;
            const int img = (int)fdiv((uint32_t)slot, p.div_si);
            const int rem = slot - img * SI;
            const int r = (int)fdiv((uint32_t)rem, p.div_sw);
            const int c = rem - r * p.SW;
            const int n = n0 + img, hs = h0 + org_h + r, ws = w0 + org_w + c;
            const bool ok = slot < S && n < p.N && (unsigned)hs < (unsigned)p.Hs && (unsigned)ws < (unsigned)p.Ws;
            if constexpr (D3) {
                const int smp = (int)fdiv((uint32_t)n, p.div_dd);
                const uint32_t z = (uint32_t)(n - smp * p.Dd);
                if constexpr (kPacked) hz[i / 2] |= z << 16 * (i % 2);
                else hz[i] = z;
                if (ok) hoff[i] = (uint32_t)(((smp * p.Ds * p.Hs + hs) * p.Ws + ws) * p.cp + 16 * sc);
            } else {
                if (ok) hoff[i] = (uint32_t)(((n * p.Hs + hs) * p.Ws + ws) * p.cp + 16 * sc);
            }
        }
    }
    v4i rh[kMaxUnits];
    auto fetch_halo = [&](int kci) {
        if constexpr (D3) {
            const int kd = (int)fdiv((uint32_t)kci, p.div_nkc), kc = kci - kd * p.nkc_frame;
            const bool kok = kci < nkc && kc * kKc + 16 * sc < p.cp;
            const uint32_t frame = (uint32_t)(p.Hs * p.Ws * p.cp);
            if constexpr (kPacked) asm volatile("" : "+v"(hz[0]), "+v"(hz[1]), "+v"(hz[2]), "+v"(hz[3]));   // (unpacked ahead of the loop they would spill)
#pragma unroll
            for (int i = 0; i < kMaxUnits; ++i)
                if (i < p.units) {   // uniform
                    const int z = (int)(kPacked ? hz[i / 2] >> 16 * (i % 2) & 0xFFFFu : hz[kPacked ? 0 : i]);
                    const int t = p.fwd ? (z << p.sD_log2) + kd * p.dD - p.pD : z + p.pD - kd * p.dD;
                    const int zs = p.fwd ? t : t >> p.sD_log2;   // arithmetic shift: a negative t stays negative
                    const bool zok = (unsigned)zs < (unsigned)p.Ds && (p.fwd || (zs << p.sD_log2) == t);
                    rh[i] = buffer_load16(rs_src, kok && zok && hoff[i] != kOob ? hoff[i] + (uint32_t)zs * frame : kOob, (uint32_t)(kc * kKc));
                }
            return;
        }
        const bool kok = kci < nkc && kci * kKc + 16 * sc < p.cp;
#pragma unroll
        for (int i = 0; i < kMaxUnits; ++i)
            if (i < p.units) rh[i] = buffer_load16(rs_src, kok ? hoff[i] : kOob, (uint32_t)(kci * kKc));
    };
    auto stage_halo = [&](int buf) {
        int8_t* H = lds + buf * halo_bytes;
#pragma unroll
        for (int i = 0; i < kMaxUnits; ++i) {
            const int slot = (tid >> 2) + SPT * i;
            if (i < p.units && slot < S) *reinterpret_cast<v4i*>(H + slot * kPitch + 16 * sc) = rh[i];
        }
    };

    // ---- filter fragments: tile (x, sub) of this wave is 1 KiB at ((row block)*2 + sub)*1024, lane*16 inside ----
    uint32_t aoff[2][2];
#pragma unroll
    for (int x = 0; x < NX; ++x)
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
            const int rb = (row0 + wr * RW) / 32 + x;
            aoff[x][sub] = rb < p.RB ? (uint32_t)((rb * 2 + sub) * 1024 + lane * 16) : kOob;
        }
    v4i ra[kRingA][2][2];   // [ring slot][x][sub]
    int f_j = 0, f_kc = 0, f_s = 0;
    auto fetch_a = [&](int slot) {
        const bool live = f_s < NS;
        const int id = p.tap_id[phase][live ? f_j : 0];
        // a dead prefetch is sent out of range through the VECTOR offset, the one the hardware checks against the extent
        const uint32_t base = live ? (uint32_t)(((f_kc * p.T + id) * p.RB) * 2048) : 0u;
#pragma unroll
        for (int x = 0; x < NX; ++x)
#pragma unroll
            for (int sub = 0; sub < 2; ++sub) ra[slot][x][sub] = buffer_load16(rs_w, live ? aoff[x][sub] : kOob, base);
        ++f_s;
        if (++f_j == taps) { f_j = 0; ++f_kc; }
    };

    // ---- pixel fragments: destination pixel q of the tile -> slot of its window origin ----
    int bslot[BF];
#pragma unroll
    for (int y = 0; y < BF; ++y) {
        const int q = wp * PXW + 32 * y + l32;
        const int img = (int)fdiv((uint32_t)q, p.div_thw);
        const int rem = q - img * p.TH * p.TW;
        const int th = (int)fdiv((uint32_t)rem, p.div_tw);
        const int tw = rem - th * p.TW;
        bslot[y] = (img < NI) ? img * SI + th * p.SW + tw : 0;
    }

    v16i acc[2][BF];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < BF; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;

    if constexpr (TAPS == 1) {
        // 1 x 1 filters: a step is a chunk, and every chunk needs a new window.  With the window requested only one
        // step ahead each chunk would wait out a full memory latency; here window registers and filter tiles both
        // sit in rings of kRing1 chunks (slot = chunk % kRing1), requested kRing1 - 1 chunks before their use.
        constexpr int kRing1 = 4, kU1 = PX / 64;   // kU1: 16-byte window units per thread (no halo: at most PX slots)
        v4i ra1[kRing1][2][2], rw[kRing1][kU1];
        auto fetch_1 = [&](int slot, int kc) {
            const bool live = kc < nkc;
            const uint32_t base = live ? (uint32_t)((kc * p.RB) * 2048) : 0u;
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) ra1[slot][x][sub] = buffer_load16(rs_w, live ? aoff[x][sub] : kOob, base);
            const bool kok = live && kc * kKc + 16 * sc < p.cp;
#pragma unroll
            for (int i = 0; i < kU1; ++i)
                if (i < p.units) rw[slot][i] = buffer_load16(rs_src, kok ? hoff[i] : kOob, (uint32_t)(kc * kKc));
        };
        auto stage_1 = [&](int buf, int slot) {
            int8_t* H = lds + buf * halo_bytes;
#pragma unroll
            for (int i = 0; i < kU1; ++i) {
                const int sl = (tid >> 2) + SPT * i;
                if (i < p.units && sl < S) *reinterpret_cast<v4i*>(H + sl * kPitch + 16 * sc) = rw[slot][i];
            }
        };
        int bbyte[BF];
#pragma unroll
        for (int y = 0; y < BF; ++y) bbyte[y] = bslot[y] * kPitch + 16 * lh;
#pragma unroll
        for (int c = 0; c < kRing1 - 1; ++c) fetch_1(c, c);
        stage_1(0, 0);
        __syncthreads();
        for (int base = 0; base < nkc; base += kRing1) {
#pragma unroll
            for (int u = 0; u < kRing1; ++u) {
                const int kc = base + u;
                if (kc >= nkc) break;   // uniform
                fetch_1((u + kRing1 - 1) % kRing1, kc + kRing1 - 1);
                const int8_t* H = lds + (kc & 1) * halo_bytes;
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) {
                    v4i b[BF];
#pragma unroll
                    for (int y = 0; y < BF; ++y) b[y] = *reinterpret_cast<const v4i*>(H + bbyte[y] + 32 * sub);
#pragma unroll
                    for (int x = 0; x < NX; ++x)
#pragma unroll
                        for (int y = 0; y < BF; ++y)
                            acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ra1[u][x][sub], b[y], acc[x][y], 0, 0, 0);
                }
                if (kc + 1 < nkc) {
                    stage_1((kc + 1) & 1, (u + 1) % kRing1);
                    __syncthreads();
                }
            }
        }
    } else if constexpr (TAPS > 0) {
        // tap tables: loop invariant, indexed with constants after unrolling
        int t_id[TAPS], t_off[TAPS];
#pragma unroll
        for (int t = 0; t < TAPS; ++t) {
            t_id[t] = p.tap_id[0][t];
            t_off[t] = p.tap_slot[0][t] * kPitch;
        }
        int bbyte[BF];
#pragma unroll
        for (int y = 0; y < BF; ++y) bbyte[y] = bslot[y] * kPitch + 16 * lh;
        v4i rt[TAPS][2][2];   // [tap][x][sub]
        auto fetch_t = [&](int t, int kc) {
            const bool live = kc < nkc;
            const uint32_t base = live ? (uint32_t)(((kc * p.T + t_id[t]) * p.RB) * 2048) : 0u;
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int sub = 0; sub < 2; ++sub) rt[t][x][sub] = buffer_load16(rs_w, live ? aoff[x][sub] : kOob, base);
        };
        v4i bq[2][2][BF];     // [set][sub][y]
        auto read_b = [&](int set, int buf, int t) {
            const int8_t* H = lds + (DB ? buf * halo_bytes : 0) + t_off[t];
#pragma unroll
            for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                for (int y = 0; y < BF; ++y)
                    bq[set][sub][y] = *reinterpret_cast<const v4i*>(H + bbyte[y] + 32 * sub);
        };
        fetch_halo(0);
#pragma unroll
        for (int t = 0; t < TAPS - 1; ++t) fetch_t(t, 0);
        stage_halo(0);
        __syncthreads();
        read_b(0, 0, 0);
        for (int kc = 0; kc < nkc; ++kc) {
            if (DB && kc + 1 < nkc) fetch_halo(kc + 1);
#pragma unroll
            for (int t = 0; t < TAPS; ++t) {
                // the tile of the step TAPS - 1 ahead: the previous tap's slot, of the next chunk unless t == 0
                fetch_t((t + TAPS - 1) % TAPS, t == 0 ? kc : kc + 1);
                if (t + 1 < TAPS) read_b((t + 1) & 1, kc & 1, t + 1);
#pragma unroll
                for (int sub = 0; sub < 2; ++sub)
#pragma unroll
                    for (int x = 0; x < NX; ++x)
#pragma unroll
                        for (int y = 0; y < BF; ++y)
                            acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(rt[t][x][sub], bq[t & 1][sub][y], acc[x][y], 0, 0, 0);
            }
            if (DB && kc + 1 < nkc) {
                stage_halo((kc + 1) & 1);
                __syncthreads();
                read_b(0, (kc + 1) & 1, 0);
            }
        }
    } else {
        if (NS > 0) {
            fetch_halo(0);
    #pragma unroll
            for (int d = 0; d < kRingA - 1; ++d) fetch_a(d);
            stage_halo(0);
            __syncthreads();
        }

        // flat loop over steps (chunk outer, live tap inner), unrolled by the ring depth so that ring slots are constants
        int j = 0, kci = 0;
        for (int base = 0; base < NS; base += kRingA) {
    #pragma unroll
            for (int u = 0; u < kRingA; ++u) {
                if (base + u < NS) {   // uniform
                    fetch_a((u + kRingA - 1) % kRingA);                          // filter tiles of step s + kRingA - 1
                    if (DB && j == 0 && kci + 1 < nkc) fetch_halo(kci + 1);      // uniform; staged at the chunk's last tap
                    const int8_t* H = lds + (DB ? (kci & 1) * halo_bytes : 0) + 16 * lh;
                    const int ts = p.tap_slot[phase][j];
    #pragma unroll
                    for (int sub = 0; sub < 2; ++sub) {
                        v4i b[BF];
    #pragma unroll
                        for (int y = 0; y < BF; ++y)
                            b[y] = *reinterpret_cast<const v4i*>(H + (bslot[y] + ts) * kPitch + 32 * sub);
    #pragma unroll
                        for (int x = 0; x < NX; ++x)
    #pragma unroll
                            for (int y = 0; y < BF; ++y)
                                acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ra[u][x][sub], b[y], acc[x][y], 0, 0, 0);
                    }
                    if (j + 1 == taps) {
                        if (DB && kci + 1 < nkc) {
                            stage_halo((kci + 1) & 1);
                            __syncthreads();
                        }
                        j = 0;
                        ++kci;
                    } else {
                        ++j;
                    }
                }
            }
        }
    }

    // epilogue: register r of tile (x, y) is row 32x + 8*(r/4) + 4*lh + r%4, destination pixel q = wp*PXW + 32y + l32
    // (Copies of the fields: behind a store the compiler takes p, a reference, for changed, and would fetch a field again and wait for
    // it before each of the next stores: 1 x 1 stride 2 with odd rows, 258 -> 193 at 19 x 15, batch 9, 9.5 us against 8.7.)
    const int Hd = p.Hd, Wd = p.Wd, Crow = p.Crow, N = p.N, TH = p.TH, TW = p.TW, bf16 = p.bf16, nt = p.nt;
    const FastDiv div_thw = p.div_thw, div_tw = p.div_tw;
    float* const out = p.out;
    int32_t* const acc_out = p.acc_out;
    const int rowbase = row0 + wr * RW + 4 * lh;
    const int HWd = Hd * Wd;
    const int CS = D3 ? p.Dd * HWd : HWd;   // elements from a result channel to the next
    const bool full_rows = row0 + ROWS <= Crow;
    if (ST == 2 && zfill && !bf16 && !acc_out && (Wd & 1) == 0) {   // uniform
        // Strided 1 x 1 layers, even rows: a pixel's 2 x 2 block leaves as (value, 0) and (0, 0), 8 bytes each.  The
        // result is four times the class image, so the lines a wave has touched but not yet completed outgrow the
        // L2 when its pixel fragments are written one after the other; here the fragments of one row (channel) are
        // written back to back instead, and the lines they share complete within a few instructions.
        float* o[BF];
        bool ok[BF], h1[BF];
#pragma unroll
        for (int y = 0; y < BF; ++y) {
            const int q = wp * PXW + 32 * y + l32;
            const int img = (int)fdiv((uint32_t)q, div_thw);
            const int rem = q - img * TH * TW;
            const int th = (int)fdiv((uint32_t)rem, div_tw);
            const int tw = rem - th * TW;
            const int n = n0 + img, h = (h0 + th) * ST, w = (w0 + tw) * ST;
            ok[y] = !(img >= NI || n >= N || h >= Hd || w >= Wd);
            h1[y] = h + 1 < Hd;
            o[y] = out + (((int64_t)n * Crow + rowbase) * HWd + h * Wd + w);
        }
#pragma unroll
        for (int x = 0; x < NX; ++x)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int dr = 32 * x + 8 * (r >> 2) + (r & 3);
                if (rowbase + dr >= Crow) continue;
#pragma unroll
                for (int y = 0; y < BF; ++y) {
                    if (!ok[y]) continue;
                    float* z = o[y] + (int64_t)dr * CS;
                    *reinterpret_cast<float2*>(z) = make_float2((float)acc[x][y][r] * scale, 0.0f);
                    if (h1[y]) *reinterpret_cast<float2*>(z + Wd) = make_float2(0.0f, 0.0f);
                }
            }
        return;
    }
#pragma unroll
    for (int y = 0; y < BF; ++y) {
        const int q = wp * PXW + 32 * y + l32;
        const int img = (int)fdiv((uint32_t)q, div_thw);
        const int rem = q - img * TH * TW;
        const int th = (int)fdiv((uint32_t)rem, div_tw);
        const int tw = rem - th * TW;
        const int n = n0 + img, h = (h0 + th) * ST + pa, w = (w0 + tw) * ST + pb;
        if (img >= NI || n >= N || h >= Hd || w >= Wd) continue;
        int64_t pix = ((int64_t)n * Crow + rowbase) * HWd + h * Wd + w;
        if constexpr (D3) {
            const int smp = (int)fdiv((uint32_t)n, p.div_dd);
            pix = ((int64_t)smp * Crow + rowbase) * CS + (int64_t)(n - smp * p.Dd) * HWd + h * Wd + w;
        }
        if (bf16) {   // uniform: the narrow result, same walk over the tile
            uint16_t* ob = reinterpret_cast<uint16_t*>(out) + pix;
            if (ST == 1 && (TW & 1) == 0 && (Wd & 1) == 0) {   // uniform
                // Even tile and image widths: lanes 2k and 2k+1 hold pixels w (even) and w+1 of one row, both inside the
                // image or both outside.  They trade values so that the even lane stores the pair of row dr and the odd
                // lane the pair of row dr+1, each as one aligned dword: half the store instructions, twice the bytes each.
                const bool odd = l32 & 1;
#pragma unroll
                for (int x = 0; x < NX; ++x)
#pragma unroll
                    for (int r = 0; r < 16; r += 2) {
                        const uint32_t v0 = bf16_bits((float)acc[x][y][r] * scale), v1 = bf16_bits((float)acc[x][y][r + 1] * scale);
                        const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? v0 : v1), 0xB1, 0xF, 0xF, false);
                        const uint32_t word = odd ? (got | (v1 << 16)) : (v0 | (got << 16));
                        const int dr = 32 * x + 8 * (r >> 2) + (r & 3) + (odd ? 1 : 0);
                        if (rowbase + dr < Crow)
                            *reinterpret_cast<uint32_t*>(ob + (int64_t)dr * CS - (odd ? 1 : 0)) = word;
                    }
                continue;
            }
            const bool w1 = w + 1 < Wd, h1 = h + 1 < Hd;
            const bool pairs = (Wd & 1) == 0;   // even rows: (value, 0) and (0, 0) go out as aligned 4-byte stores
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 32 * x + 8 * (r >> 2) + (r & 3);
                    if (rowbase + dr >= Crow) continue;
                    uint16_t* z = ob + (int64_t)dr * CS;
                    const uint32_t v = bf16_bits((float)acc[x][y][r] * scale);
                    if (ST == 2 && zfill && pairs) {
                        *reinterpret_cast<uint32_t*>(z) = v;   // little endian: the value first, then the zero
                        if (h1) *reinterpret_cast<uint32_t*>(z + Wd) = 0u;
                    } else {
                        z[0] = (uint16_t)v;
                        if (ST == 2 && zfill) {
                            if (w1) z[1] = 0;
                            if (h1) z[Wd] = 0;
                            if (h1 && w1) z[Wd + 1] = 0;
                        }
                    }
                }
            continue;
        }
        float* o = out + pix;
        if (ST == 2 && zfill && (Wd & 1) == 0) {
            // written below together with the zeros of the 2 x 2 block
        } else if (full_rows && nt) {
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    __builtin_nontemporal_store((float)acc[x][y][r] * scale, &o[(32 * x + 8 * (r >> 2) + (r & 3)) * CS]);
        } else if (full_rows) {
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[(32 * x + 8 * (r >> 2) + (r & 3)) * CS] = (float)acc[x][y][r] * scale;
        } else {
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 32 * x + 8 * (r >> 2) + (r & 3);
                    if (rowbase + dr < Crow) o[dr * CS] = (float)acc[x][y][r] * scale;
                }
        }
        if (acc_out) {
            int32_t* ao = acc_out + pix;
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 32 * x + 8 * (r >> 2) + (r & 3);
                    if (rowbase + dr < Crow) ao[dr * CS] = acc[x][y][r];
                }
        }
        if (ST == 2 && zfill) {
            // the three neighbours of this pixel in its 2 x 2 block receive no tap at all
            const bool w1 = w + 1 < Wd, h1 = h + 1 < Hd;
            const bool pairs = (Wd & 1) == 0;   // even rows: (value, 0) and (0, 0) go out as aligned 8-byte stores
#pragma unroll
            for (int x = 0; x < NX; ++x)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 32 * x + 8 * (r >> 2) + (r & 3);
                    if (rowbase + dr >= Crow) continue;
                    float* z = o + (int64_t)dr * CS;
                    if (pairs) {
                        *reinterpret_cast<float2*>(z) = make_float2((float)acc[x][y][r] * scale, 0.0f);
                        if (h1) *reinterpret_cast<float2*>(z + Wd) = make_float2(0.0f, 0.0f);
                    } else {
                        if (w1) z[1] = 0.0f;
                        if (h1) z[Wd] = 0.0f;
                        if (h1 && w1) z[Wd + 1] = 0.0f;
                    }
                    if (acc_out) {
                        int32_t* za = acc_out + pix + (int64_t)dr * CS;
                        if (w1) za[1] = 0;
                        if (h1) za[Wd] = 0;
                        if (h1 && w1) za[Wd + 1] = 0;
                    }
                }
        }
    }
}

template <int WR, bool DB, int ST, int WAVES, int TAPS = 0, int NX = 2, int PX = kPxWg, bool D3 = false>
__global__ __launch_bounds__(64 * WAVES, (TAPS == 1 || NX == 1 || PX < kPxWg) ? 2 : 1) void k_conv_halo(HaloArgs p) {
    halo_role<WR, DB, ST, WAVES, TAPS, NX, PX, D3>(p, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// 1 x 1 data gradient (and forward pass) at unit stride with a short contraction axis (at most 256 channels: for the
// data gradient the projection layers of MobileNetV2 and the 1 x 1 layers of ResNet-50 that reduce to 64 - 256 channels).  Such a layer is a few
// multiplies per 32 x 32 block of its result and is bound by that fp32 result; as a tile kernel (one to four steps
// per workgroup) it spent as long in set-up as in stores.  Here a wave streams: it keeps the filter fragments of
// two 32-row blocks of the result in registers (16 bytes per lane and 32-byte contraction step, from the
// fragment-order copy) and walks over groups of 32 consecutive pixels with a stride - the pixel fragments are 16
// bytes per lane straight from the NHWC gradient (coalesced, no LDS; the next group's are requested before the
// current group's multiplies), then 2 x KS v_mfma_i32_32x32x32_i8 and 32 stores of 128-byte runs per group.
// Waves of a workgroup hold neighbouring row blocks of the same pixel groups.
// ---------------------------------------------------------------------------------------------
struct StreamArgs {
    // What a block finds its place by fills the first 64 bytes, what it loads and stores by the next: arguments arrive in lines of that size,
    // 0.25 us each when one is asked for behind another (64 -> 64 at 42 x 42, batch 14: 5.30 us with the dealing's fields in a third line).
    int main_blocks;
    uint32_t deal, dealt;   // blocks that an XCD takes in a row; the blocks dealt out that way, whole turns of the XCDs
    FastDiv div_deal;
    FastDiv div_rp;
    int RP, S;            // pairs of row blocks; pixel-group phases, a multiple of four (a wave takes groups s, s + S, ...)
    int cp, Crow, RB, HW;
    int bf16;             // the result is bfloat16 storage
    const int8_t* src;    // NHWC gradient, [pixels][cp]
    const int8_t* wfrag;  // filter in fragment order (one tap): [cp/64][RB][2][1024]
    uint32_t src_bytes, wfrag_bytes;
    uint32_t total_px, groups;
    const float* s_a;
    const float* s_b;
    float* out;
    uint32_t out_bytes;   // STORE 1 and 2
    FastDiv div_hw;
    int32_t* acc_out;
    DwTail tail;          // tail.blocks > 0: that many workgroups behind the first main_blocks finish a deferred filter gradient
};

static_assert(offsetof(StreamArgs, src) == 64 && offsetof(StreamArgs, out_bytes) <= 124, "a block's place in the first line, its operands in the second");

// KS = 32-byte contraction steps (cp <= 32 * KS)
// STORE: how the results leave.  1 (fp32) and 2 (bfloat16, even planes): through a buffer descriptor, an offset past its extent
// for pixels and rows that do not exist, so that every group issues the same number of stores with no branch between them.
// Loads and stores retire in order, and only with that number known can the compiler wait for the next group's pixel
// fragments alone; behind branches it waits for everything, i.e. for the group's own stores to reach memory.
// (ResNet-50, batch 64, backward of the layer: 256 -> 64 at 56 x 56 114 -> 105 us, 256 -> 128 at 56 x 56 167 -> 140,
// 512 -> 256 at 28 x 28 100 -> 93.)  0: any result (accumulators too, bfloat16 on odd planes, 2 GiB and more).
template <int KS, int STORE, bool NT>
__global__ __launch_bounds__(256) void k_dx_1x1_stream(StreamArgs p) {
    __shared__ int32_t l_role[256];
    if ((int)blockIdx.x >= p.main_blocks) {   // uniform
        dw_reduce_role(p.tail, (int)blockIdx.x - p.main_blocks, l_role);
        return;
    }
    const int lane = threadIdx.x % kWave, l32 = lane & 31, lh = lane >> 5;
    // the four waves of a workgroup take four neighbouring pixel groups of one pair of row blocks: together they
    // write 512 consecutive bytes of each of the pair's 64 planes
    uint32_t at = blockIdx.x;
    if (at < p.dealt) {   // uniform: stream_deal
        const uint32_t i = at / kXcd, turn = fdiv(i, p.div_deal);
        at = (turn * (kXcd - 1) + at % kXcd) * p.deal + i;
    }
    const uint32_t quad = fdiv(at, p.div_rp);
    const int rp = (int)(at - quad * (uint32_t)p.RP);
    const uint32_t s = quad * 4u + threadIdx.x / kWave;
    if (s >= (uint32_t)p.S) return;   // uniform per wave
    // (a wave takes groups s, s + S, ...: all waves together advance through the pixels as one window.  Giving every
    // workgroup a contiguous range of its own instead measured 13 % slower over ResNet-50's 17 such layers.)
    const __amdgpu_buffer_rsrc_t rs_src = __builtin_amdgcn_make_buffer_rsrc((void*)p.src, 0, (int)p.src_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void*)p.wfrag, 0, (int)p.wfrag_bytes, 0x00020000);
    const float scale = (*p.s_a / 127.0f) * (*p.s_b / 127.0f);
    const __amdgpu_buffer_rsrc_t rs_out = __builtin_amdgcn_make_buffer_rsrc((void*)p.out, 0, (int)p.out_bytes, 0x00020000);
    const bool rows_full = 64 * rp + 64 <= p.Crow;   // uniform

    v4i A[2][KS];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int rb = 2 * rp + j;
            const bool live = rb < p.RB && 32 * ks < p.cp;
            A[j][ks] = buffer_load16(rs_w, live ? (uint32_t)((((ks >> 1) * p.RB + rb) * 2 + (ks & 1)) * 1024 + lane * 16) : kOob, 0);
        }
    // contraction bytes 32*ks + 16*lh .. +15 of the lane's pixel; bytes past the channel pitch belong to the next pixel
    auto fetch = [&](uint32_t grp, v4i (&B)[KS]) {
        const uint32_t P = grp * 32u + (uint32_t)l32;
        const bool valid = grp < p.groups && P < p.total_px;
        const uint32_t boff = P * (uint32_t)p.cp + 16u * lh;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) B[ks] = buffer_load16(rs_src, (valid && 32 * ks + 16 * lh < p.cp) ? boff : kOob, 32u * ks);
    };
    v4i B[KS];
    fetch(s, B);
    // the loop is entered with nothing on its way, so that its head waits as its own back edge needs
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    for (uint32_t grp = s; grp < p.groups; grp += (uint32_t)p.S) {
        v4i Bn[KS];
        fetch(grp + (uint32_t)p.S, Bn);
        v16i acc[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = 0;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[j][ks], B[ks], acc[j], 0, 0, 0);
        }
        const uint32_t P = grp * 32u + (uint32_t)l32;
        if constexpr (STORE != 0) {
            const uint32_t n = fdiv(P < p.total_px ? P : 0u, p.div_hw);
            const uint32_t r0 = P - n * (uint32_t)p.HW;
            constexpr uint32_t EB = STORE == 1 ? 4 : 2;
            const uint32_t row_bytes = (uint32_t)p.HW * EB;
            const bool odd = l32 & 1;
            const int lane_row = 64 * rp + 4 * lh + (STORE == 2 && odd ? 1 : 0);   // bfloat16: see below
            const uint32_t at = ((n * (uint32_t)p.Crow + (uint32_t)lane_row) * (uint32_t)p.HW + r0 - (STORE == 2 && odd ? 1u : 0u)) * EB;
            const uint32_t voff = P < p.total_px ? at : kOob;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 16; r += STORE) {
                    const int dr = 32 * j + 8 * (r >> 2) + (r & 3);
                    const uint32_t v = (rows_full | (lane_row + dr < p.Crow)) ? voff : kOob;
                    if constexpr (STORE == 1) {
                        const int w = __builtin_bit_cast(int, (float)acc[j][r] * scale);
                        __builtin_amdgcn_raw_buffer_store_b32(w, rs_out, (int)v, (int)((uint32_t)dr * row_bytes), NT ? 2 : 0);   // 2: streaming
                    } else {
                        // lanes 2k and 2k+1 hold pixels r0 (even) and r0 + 1 of one plane: they trade values, and the even
                        // lane stores the pair of row dr, the odd lane that of row dr + 1, one aligned dword each
                        const uint32_t v0 = bf16_bits((float)acc[j][r] * scale), v1 = bf16_bits((float)acc[j][r + 1] * scale);
                        const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? v0 : v1), 0xB1, 0xF, 0xF, false);
                        const int w = (int)(odd ? (got | (v1 << 16)) : (v0 | (got << 16)));
                        __builtin_amdgcn_raw_buffer_store_b32(w, rs_out, (int)v, (int)((uint32_t)dr * row_bytes), NT ? 2 : 0);   // 2: streaming
                    }
                }
        } else if (P < p.total_px) {
            const uint32_t n = fdiv(P, p.div_hw);
            const uint32_t r0 = P - n * (uint32_t)p.HW;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int rowbase = 32 * (2 * rp + j) + 4 * lh;
                const int64_t at = ((int64_t)n * p.Crow + rowbase) * p.HW + r0;
                if (p.bf16) {   // uniform
                    uint16_t* ob = reinterpret_cast<uint16_t*>(p.out) + at;
                    if ((p.HW & 1) == 0) {
                        // Even planes: lanes 2k and 2k+1 hold pixels r0 (even) and r0 + 1 of one plane.  They trade values so
                        // that the even lane stores the pair of row dr and the odd lane the pair of row dr + 1, each as one
                        // aligned dword: half the store instructions, twice the bytes each.
                        const bool odd = l32 & 1;
#pragma unroll
                        for (int r = 0; r < 16; r += 2) {
                            const uint32_t v0 = bf16_bits((float)acc[j][r] * scale), v1 = bf16_bits((float)acc[j][r + 1] * scale);
                            const uint32_t got = (uint32_t)__builtin_amdgcn_mov_dpp((int)(odd ? v0 : v1), 0xB1, 0xF, 0xF, false);
                            const uint32_t word = odd ? (got | (v1 << 16)) : (v0 | (got << 16));
                            const int dr = 8 * (r >> 2) + (r & 3) + (odd ? 1 : 0);
                            if (rowbase + dr < p.Crow) {
                                uint32_t* z = reinterpret_cast<uint32_t*>(ob + (int64_t)dr * p.HW - (odd ? 1 : 0));
                                if (NT) __builtin_nontemporal_store(word, z);
                                else *z = word;
                            }
                        }
                    } else {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int dr = 8 * (r >> 2) + (r & 3);
                            if (rowbase + dr < p.Crow) ob[(int64_t)dr * p.HW] = (uint16_t)bf16_bits((float)acc[j][r] * scale);
                        }
                    }
                    continue;
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int dr = 8 * (r >> 2) + (r & 3);
                    if (rowbase + dr >= p.Crow) continue;
                    float* z = p.out + at + (int64_t)dr * p.HW;
                    if (NT) __builtin_nontemporal_store((float)acc[j][r] * scale, z);
                    else *z = (float)acc[j][r] * scale;
                    if (p.acc_out) p.acc_out[at + (int64_t)dr * p.HW] = acc[j][r];
                }
            }
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) B[ks] = Bn[ks];
    }
}

// Workgroups of one row tile: one per pixel tile, times the parity classes of a strided data gradient.
int64_t blocks_per_row_tile(const HaloArgs& a) {
    return (int64_t)a.groups * a.tiles_h * a.tiles_w * (a.stride > 1 && !a.zfill ? a.stride * a.stride : 1);
}

// Taps of the parity class that has most.
int max_taps(const HaloArgs& a) { return *std::max_element(a.ph_taps, a.ph_taps + a.stride * a.stride); }

// floor division for possibly negative numerators
int floor_div(int a, int b) { return a >= 0 ? a / b : -((-a + b - 1) / b); }

struct Geometry {
    bool ok;
    HaloArgs a;
    size_t lds_bytes;
    int rows;
    int px;   // destination pixels per workgroup
};

// 1 x 1 filters with several contraction chunks, on 64-row tiles: the form with rings of chunks.  Unit stride, or
// stride 2 without padding (one live parity class whose workgroups also write the zeros of the other three: the
// contraction loop is the same, only the block decoding and the epilogue know about the stride).
bool ring1_applies(const Geometry& g) {
    const HaloArgs& a = g.a;
    return (a.stride == 1 || a.zfill) && a.T == 1 && a.ph_taps[0] == 1 && a.tap_slot[0][0] == 0 && a.double_buffer &&
           a.units <= g.px / 64 && g.rows == 64;
}

// backward: destination (h, w) of parity class (pa, pb), h = 2*th + pa, reads source row th + (pa + pad - kh*dil)/stride
// for every kh that makes the quotient exact.  forward (unit stride): source row = h - pad + kh*dil.
Geometry plan(bool backward, int N, int Hs, int Ws, int cp, int Hd, int Wd, int Crow, int kH, int kW, int sH, int sW,
              int pH, int pW, int dH, int dW, int px = kPxWg, bool depth = false) {
    Geometry g{};
    g.px = px;
    HaloArgs& a = g.a;
    if (sH != sW || (sH != 1 && !(sH == 2 && backward)) || kH * kW > kMaxTaps) return g;
    // strided 1x1: three of four parity classes are empty; served when the live one is class (0, 0) (no padding),
    // whose workgroups then write the zeros of the other three next to their own results
    if (kH * kW == 1 && sH != 1 && (pH != 0 || pW != 0)) return g;
    a.zfill = (kH * kW == 1 && sH == 2) ? 1 : 0;
    const int s = sH;
    a.stride = s;
    a.T = kH * kW;
    int span_h = 0, span_w = 0;
    struct Tap { int oh, ow, id; };
    for (int ph = 0; ph < s * s; ++ph) {
        const int pa = ph / s, pb = ph % s;
        Tap taps[kMaxTaps];
        int nt = 0, mn_h = 1 << 30, mx_h = -(1 << 30), mn_w = 1 << 30, mx_w = -(1 << 30);
        for (int kh = 0; kh < kH; ++kh)
            for (int kw = 0; kw < kW; ++kw) {
                int oh, ow;
                if (backward) {
                    const int th = pa + pH - kh * dH, tw = pb + pW - kw * dW;
                    if (((th % s) + s) % s || ((tw % s) + s) % s) continue;
                    oh = floor_div(th, s);
                    ow = floor_div(tw, s);
                } else {
                    oh = kh * dH - pH;
                    ow = kw * dW - pW;
                }
                taps[nt++] = Tap{oh, ow, kh * kW + kw};
                mn_h = std::min(mn_h, oh); mx_h = std::max(mx_h, oh);
                mn_w = std::min(mn_w, ow); mx_w = std::max(mx_w, ow);
            }
        a.ph_taps[ph] = nt;
        a.ph_org_h[ph] = nt ? mn_h : 0;
        a.ph_org_w[ph] = nt ? mn_w : 0;
        if (nt) {
            span_h = std::max(span_h, mx_h - mn_h);
            span_w = std::max(span_w, mx_w - mn_w);
        }
        for (int t = 0; t < nt; ++t) {
            // slot offsets are filled in below, once the window width is known
            a.tap_slot[ph][t] = ((taps[t].oh - a.ph_org_h[ph]) << 8) | (taps[t].ow - a.ph_org_w[ph]);
            a.tap_id[ph][t] = taps[t].id;
        }
    }
    if (span_h > 255 || span_w > 255) return g;
    // tile of one parity class: best coverage of the class image by 256-pixel tiles whose window fits
    const int PH = (int)ceil_div(Hd, s), PW = (int)ceil_div(Wd, s);
    double best = 0.0;
    int bTH = 0, bTW = 0, bNI = 0;
    if (PH * PW <= px) {
        bTH = PH; bTW = PW; bNI = px / (PH * PW);
        if ((int64_t)bNI * (bTH + span_h) * (bTW + span_w) > 64 * kMaxUnits) bNI = (64 * kMaxUnits) / ((bTH + span_h) * (bTW + span_w));
        if (bNI < 1) return g;
    } else {
        // widest tile among the best covers: the result is stored in runs of TW pixels
        for (int tw = std::min(PW, 128); tw >= 4; --tw) {
            const int th = std::min(px / tw, PH);
            if (th < 1) continue;
            if ((int64_t)(th + span_h) * (tw + span_w) > 64 * kMaxUnits) continue;
            const double eff = (double)PH * PW / ((double)ceil_div(PH, th) * ceil_div(PW, tw) * px);
            if (eff > best + 0.02) { best = eff; bTH = th; bTW = tw; }
        }
        bNI = 1;
        if (bTH == 0) return g;
    }
    a.TH = bTH; a.TW = bTW; a.NI = bNI;
    a.SH = bTH + span_h; a.SW = bTW + span_w;
    for (int ph = 0; ph < s * s; ++ph)
        for (int t = 0; t < a.ph_taps[ph]; ++t) {
            const int v = a.tap_slot[ph][t];
            a.tap_slot[ph][t] = (v >> 8) * a.SW + (v & 255);
        }
    const int S = a.NI * a.SH * a.SW;
    a.units = (int)ceil_div(S, 64);   // for four waves; the eight-wave form of 128-row tiles halves it at launch
    if (a.units > kMaxUnits) return g;
    a.N = N; a.Hs = Hs; a.Ws = Ws; a.cp = cp; a.Hd = Hd; a.Wd = Wd; a.Crow = Crow;
    a.RB = (int)ceil_div(Crow, 32);
    a.tiles_h = (int)ceil_div(PH, a.TH);
    a.tiles_w = (int)ceil_div(PW, a.TW);
    a.groups = (int)ceil_div(N, a.NI);
    a.double_buffer = cp > kKc || depth;   // (depth: the 3-D forms exist with two window buffers only)
    g.lds_bytes = (size_t)(a.double_buffer ? 2 : 1) * S * kPitch;
    if (g.lds_bytes > 150 * 1024) return g;
    // Tiles of 64 rows, two workgroups to a CU; of 128 rows, one to a CU, only for a single chunk by parity classes, where they fill the chip (384 <- 16
    // at 59 x 59, batch 78: 130 us and 163 on 64 rows; elsewhere the other way round, up to 1.7 times: 192 <- 110, 5 x 5, 26 x 26, batch 53, 46.6 and 28.5).
    const int64_t blocks128 = (int64_t)a.groups * a.tiles_h * a.tiles_w * (a.zfill ? 1 : s * s) * ceil_div(Crow, 128);
    g.rows = Crow > 64 && blocks128 >= 256 && px == kPxWg && s == 2 && !a.double_buffer ? 128 : 64;
    a.div_tw = make_fastdiv((uint32_t)a.TW);
    a.div_thw = make_fastdiv((uint32_t)(a.TH * a.TW));
    a.div_sw = make_fastdiv((uint32_t)a.SW);
    a.div_si = make_fastdiv((uint32_t)(a.SH * a.SW));
    a.div_tiles_w = make_fastdiv((uint32_t)a.tiles_w);
    a.div_tiles_hw = make_fastdiv((uint32_t)(a.tiles_h * a.tiles_w));
    const int64_t pt = blocks_per_row_tile(a);
    // room for the workgroups of a deferred filter-gradient reduction (at most 4096, dw_tail_worthwhile) is kept here,
    // so that the grid-size test of the launch cannot fail once an entry point has started launching
    if (pt * ceil_div(Crow, 64) >= ((int64_t)1 << 31) - 4096) return g;
    a.row_tiles = (int)ceil_div(Crow, g.rows);
    a.div_row_tiles = make_fastdiv((uint32_t)a.row_tiles);
    g.ok = true;
    return g;
}

// Profile labels, one per kernel form (they are different instantiations with different bounds): the tile kernel with
// a run-time tap list at unit stride, by parity classes at stride 2, on 128-row tiles, and the two constant-tap forms.
struct HaloNames { const char *dyn, *s2, *r128, *k1, *k9; };
constexpr HaloNames kBwdNames{"conv_bwd_data_halo", "conv_bwd_data_halo_s2", "conv_bwd_data_halo_r128", "conv_bwd_data_halo_1x1",
                              "conv_bwd_data_halo_3x3"};
constexpr HaloNames kFwdNames{"conv_fwd_halo", "conv_fwd_halo", "conv_fwd_halo_r128", "conv_fwd_halo_1x1", "conv_fwd_halo_3x3"};

// The ring form holds two workgroups per CU.  A layer whose 256-pixel tiles give far fewer than that (the late 1 x 1
// layers of a classification network: few pixels, long contraction) is cut into 128-pixel tiles instead.  Measured
// on ResNet-50's last stages, N = 64: 512 -> 2048 at 7 x 7 (104 tiles) 23.3 -> 17.2 us, 256 -> 1024 at 14 x 14 (256
// tiles) 14.6 -> 14.5 us cold and 12.4 -> 11.6 us warm, 2048 -> 512 at 7 x 7 (416 tiles) 14.0 -> 15.1 us: not there.
// The constant-tap 3 x 3 form takes 128-pixel tiles where 256-pixel tiles are fewer than the CUs: 512 -> 512 at 7 x 7, batch 128 (208 tiles),
// 25.6 -> 23.5 us; 256 -> 256 at 14 x 14, batch 48 (192), 15.7 -> 15.1; batch 64 (256) 14.4 -> 14.9: not there.
bool taps9_applies(const Geometry& g) {
    const HaloArgs& a = g.a;
    return a.stride == 1 && a.ph_taps[0] == 9 && a.double_buffer && g.rows == 64;
}

template <typename Plan>
Geometry plan_small(Geometry g, Plan replan) {
    if (!g.ok) return g;
    const int64_t blocks = blocks_per_row_tile(g.a) * ceil_div(g.a.Crow, 64);
    if (ring1_applies(g) && blocks < 384) {
        Geometry s = replan(128);
        return s.ok && ring1_applies(s) ? s : g;
    }
    if (taps9_applies(g) && blocks < 256) {
        Geometry s = replan(128);
        return s.ok && taps9_applies(s) ? s : g;
    }
    return g;
}

daq_status launch(Geometry& g, hipStream_t st, const HaloNames& names) {
    const HaloArgs& a = g.a;
    const char* name = g.rows == 128 ? names.r128 : a.stride == 2 ? names.s2 : names.dyn;
    const int64_t ptiles = blocks_per_row_tile(a);
    const int64_t blocks = ptiles * ceil_div(a.Crow, g.rows) + a.tail.blocks;
    if (blocks >= ((int64_t)1 << 31)) return DAQ_ERR_UNSUPPORTED;
    g.a.main_blocks = (int)(blocks - a.tail.blocks);
    if (a.tail.blocks > 0) g.lds_bytes = std::max<size_t>(g.lds_bytes, 8 * kWave * sizeof(int32_t));   // the role's scratch
    const dim3 grid((unsigned)blocks);
    // Layers with several contraction chunks and 3 x 3 filters at unit stride: the form with a constant tap count.  (With a single chunk the
    // kernel is all prologue and epilogue, and the dynamic form, which needs fewer registers, lets more workgroups overlap theirs.)
    // 1 x 1 filters with several contraction chunks: the form with rings of chunks
    const bool ring1 = ring1_applies(g);
    if (g.px != kPxWg && !ring1 && !taps9_applies(g)) return DAQ_ERR_UNSUPPORTED;   // small tiles exist in these two forms only (see plan_small)
    if (ring1) {
        if (g.px != kPxWg && tiles_by_rows(a.TH, a.TW, a.tiles_h, a.tiles_w, a.stride, a.Hd, a.Wd, a.bf16 ? 2 : 4, ptiles, a.row_tiles)) {
            g.a.by_rows = 1;
            g.a.row_tiles = (int)ptiles;
            g.a.div_row_tiles = make_fastdiv((uint32_t)ptiles);
        }
        if (g.px == kPxWg && a.stride == 1 && tiles_spread(a.TH, a.TW, a.tiles_h, a.tiles_w, a.Hd, a.Wd, a.bf16 ? 2 : 4, ptiles, a.row_tiles))
            g.a.spread = (int)(ptiles / kXcd * kXcd * a.row_tiles);
        const bool wide = wide_waves1(g.a.main_blocks, a.stride, a.Wd);
        auto kern = a.stride == 2 ? (g.px != kPxWg ? k_conv_halo<1, true, 2, 4, 1, 2, 128> : wide ? k_conv_halo<2, true, 2, 4, 1, 1> : k_conv_halo<1, true, 2, 4, 1>)
                                  : (g.px != kPxWg ? k_conv_halo<1, true, 1, 4, 1, 2, 128> : wide ? k_conv_halo<2, true, 1, 4, 1, 1> : k_conv_halo<1, true, 1, 4, 1>);
        if (!allow_lds((const void*)kern, g.lds_bytes))
            return DAQ_ERR_HIP;
        DAQ_LAUNCH(names.k1, st, hipLaunchKernelGGL(kern, grid, dim3(256), g.lds_bytes, st, a));
        return DAQ_OK;
    }
    if (taps9_applies(g)) {
        auto kern = g.px == kPxWg ? k_conv_halo<2, true, 1, 4, 9, 1> : k_conv_halo<2, true, 1, 4, 9, 1, 128>;
        if (!allow_lds((const void*)kern, g.lds_bytes))
            return DAQ_ERR_HIP;
        DAQ_LAUNCH(names.k9, st, hipLaunchKernelGGL(kern, grid, dim3(256), g.lds_bytes, st, a));
        return DAQ_OK;
    }
    if (g.rows == 128) {
        HaloArgs a8 = g.a;   // eight waves stage the window in half as many passes
        a8.units = (int)ceil_div((int64_t)g.a.NI * g.a.SH * g.a.SW, 128);
        auto kern = k_conv_halo<2, false, 2, 8>;
        if (!allow_lds((const void*)kern, g.lds_bytes)) return DAQ_ERR_HIP;
        DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, grid, dim3(512), g.lds_bytes, st, a8));
    } else if (a.Crow <= 32) {
#define DAQ_HALO_NARROW(DBV)                                                                                         \
    {                                                                                                                \
        auto kern = a.stride == 2 ? k_conv_halo<1, DBV, 2, 4, 0, 1> : k_conv_halo<1, DBV, 1, 4, 0, 1>;               \
        if (!allow_lds((const void*)kern, g.lds_bytes))                                                                                              \
            return DAQ_ERR_HIP;                                                                                      \
        DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, grid, dim3(256), g.lds_bytes, st, a));                         \
    }
        if (a.double_buffer) DAQ_HALO_NARROW(true) else DAQ_HALO_NARROW(false)
#undef DAQ_HALO_NARROW
    } else {
        // (many workgroups: waves of 32 rows x 128 pixels, as above)
        const bool wide = wide_waves(g.a.main_blocks, (int)ceil_div(a.cp, kKc), max_taps(a));
        auto kern = wide ? (a.double_buffer ? (a.stride == 2 ? k_conv_halo<2, true, 2, 4, 0, 1> : k_conv_halo<2, true, 1, 4, 0, 1>)
                                            : (a.stride == 2 ? k_conv_halo<2, false, 2, 4, 0, 1> : k_conv_halo<2, false, 1, 4, 0, 1>))
                         : (a.double_buffer ? (a.stride == 2 ? k_conv_halo<1, true, 2, 4> : k_conv_halo<1, true, 1, 4>)
                                            : (a.stride == 2 ? k_conv_halo<1, false, 2, 4> : k_conv_halo<1, false, 1, 4>));
        if (!allow_lds((const void*)kern, g.lds_bytes)) return DAQ_ERR_HIP;
        DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, grid, dim3(256), g.lds_bytes, st, a));
    }
    return DAQ_OK;
}

Geometry plan_bwd(const daq_conv_desc& d) {
    daq_layout Lg;
    daq_wpack_layout Lw;
    Geometry g{};
    if (d.groups != 1 || daq_layout_qg(&d, &Lg) != DAQ_OK || daq_layout_qw(&d, &Lw) != DAQ_OK) return g;
    if (Lg.kind != DAQ_LAYOUT_NHWC || Lg.bytes >= ((int64_t)1 << 31) || Lw.bytes - Lw.off_bwd_frag >= ((int64_t)1 << 31)) return g;
    auto make = [&](int px) {
        return plan(true, d.N, Lg.H, Lg.W, Lg.c_pitch, d.Hin, d.Win, d.Cin, d.kH, d.kW, d.strideH, d.strideW, d.padH, d.padW,
                    d.dilH, d.dilW, px);
    };
    g = plan_small(make(kPxWg), make);
    g.a.src_bytes = (uint32_t)Lg.bytes;
    g.a.wfrag_bytes = (uint32_t)(Lw.bytes - Lw.off_bwd_frag);
    return g;
}

Geometry plan_fwd(const daq_conv_desc& d) {
    daq_layout Lx;
    daq_wpack_layout Lw;
    Geometry g{};
    if (d.groups != 1 || daq_layout_qx_nhwc(&d, &Lx) != DAQ_OK || daq_layout_qw(&d, &Lw) != DAQ_OK) return g;
    if (Lx.bytes >= ((int64_t)1 << 31) || Lw.off_bwd_frag - Lw.off_fwd_frag >= ((int64_t)1 << 31)) return g;
    auto make = [&](int px) {
        return plan(false, d.N, d.Hin, d.Win, Lx.c_pitch, daq_out_h(&d), daq_out_w(&d), d.Cout, d.kH, d.kW, d.strideH,
                    d.strideW, d.padH, d.padW, d.dilH, d.dilW, px);
    };
    g = plan_small(make(kPxWg), make);
    g.a.src_bytes = (uint32_t)Lx.bytes;
    g.a.wfrag_bytes = (uint32_t)(Lw.off_bwd_frag - Lw.off_fwd_frag);
    return g;
}

// ---------------------------------------------------------------------------------------------
// Both gradients of a small layer in one launch.  They do not depend on each other, and a layer whose two kernels together
// have no more workgroups than the chip has CUs gains nothing from running them one after the other: each is a chain of
// latencies (prologue, a few chunks, combine, stores; 6 to 10 us), most CUs idle, and a launch between them - unless the filter
// gradient needs more CUs than the data gradient leaves it (bwd_filter_beside).  The first
// w_blocks workgroups work on the filter gradient, those from x_first on (a multiple of eight, so that either part's own
// mapping to the XCDs holds) on the data gradient, with the first four of their eight waves.  All are resident at once: at
// most 256, each with a CU's LDS to itself.
// (Backward step, quantizer included: 16 -> 16 3 x 3 at 16 x 16, batch 4, 24.8 -> 18.3 us; 100 -> 70 3 x 3 at 29 x 31, batch
// 5, 28.7 -> 22.4; 53 -> 592 1 x 1 stride 2 at 53 x 53, batch 3, 32 -> 23.)
// ---------------------------------------------------------------------------------------------
enum BothForm { kBothRing1, kBothTaps9, kBothOneChunk, kBothNarrow, kBothRing1S2, kBothNone };   // of the tile kernel
constexpr int kBothBlocks = 256;

template <bool K11, int FORM>
__global__ __launch_bounds__(512, 1) void k_bwd_both(int w_blocks, int x_first, Dw32Args w, HaloArgs x) {
    asm volatile("" ::"s"(w_blocks), "s"(w.part), "s"(w.x_frame), "s"(x.main_blocks));   // the first lines of arguments of either part, asked for at once
    const int b = (int)blockIdx.x;
    if (b < x_first) {   // uniform
        if (b >= w_blocks) return;
        if constexpr (K11) dw11_role<1, 1, 8, 3, 1, true>(w, b);
        else dw32_ring_role<false>(w, b);
        return;
    }
    if (threadIdx.x >= 256) return;   // (a barrier waits for the waves that are still there)
    const uint32_t bid = (uint32_t)(b - x_first);
    if constexpr (FORM == kBothRing1) halo_role<1, true, 1, 4, 1, 2, 128, false>(x, bid);
    else if constexpr (FORM == kBothTaps9) halo_role<2, true, 1, 4, 9, 1, 128, false>(x, bid);
    else if constexpr (FORM == kBothOneChunk) halo_role<1, false, 1, 4, 0, 2, kPxWg, false>(x, bid);
    else if constexpr (FORM == kBothNarrow) halo_role<1, false, 1, 4, 0, 1, kPxWg, false>(x, bid);
    else halo_role<1, true, 2, 4, 1, 2, 128, false>(x, bid);
}

BothForm both_form(const Geometry& g) {
    const HaloArgs& a = g.a;
    if (!g.ok || g.rows != 64) return kBothNone;
    if (ring1_applies(g)) return g.px != 128 ? kBothNone : a.stride == 2 ? kBothRing1S2 : kBothRing1;
    if (taps9_applies(g)) return g.px == 128 ? kBothTaps9 : kBothNone;
    if (g.px != kPxWg || a.double_buffer || a.stride != 1) return kBothNone;
    return a.Crow <= 32 ? kBothNarrow : kBothOneChunk;
}

// ---------------------------------------------------------------------------------------------
// 3-D layers (forms D3 of the tile kernel).  The filter of such a layer is stored [tap][row][contraction, a multiple of 16]
// with tap = (kd*kH + kh)*kW + kw; a lane of the tile kernel would collect its fragment from 32 rows a pitch apart, a
// quarter of the rate of one contiguous KiB, and every workgroup reads the whole filter.  So the filter is put into
// fragment order first, in the workspace: a few hundred KiB, once per call (64 -> 64, 3 x 3 x 3: 221 KiB, about 2 us).
// One thread per 16-byte unit; units of padded rows and contraction bytes are zeros.
__global__ __launch_bounds__(256) void k_frag3(const int8_t* __restrict__ src, int rows, int kp, int taps, int RB, int nkc_frame,
                                               uint32_t units, v4i* __restrict__ dst) {
    const uint32_t u = blockIdx.x * 256u + threadIdx.x;
    if (u >= units) return;
    const int r32 = (int)(u & 31u), kg = (int)((u >> 5) & 1u), sub = (int)((u >> 6) & 1u);
    uint32_t v = u >> 7;
    const int rb = (int)(v % (uint32_t)RB);
    v /= (uint32_t)RB;
    const int tap = (int)(v % (uint32_t)taps), kci = (int)(v / (uint32_t)taps);
    const int kd = kci / nkc_frame, kc = kci - kd * nkc_frame;
    const int row = 32 * rb + r32, k = kKc * kc + 32 * sub + 16 * kg;
    v4i w = {0, 0, 0, 0};
    if (row < rows && k < kp) w = *reinterpret_cast<const v4i*>(src + ((int64_t)(kd * taps + tap) * rows + row) * kp + k);
    dst[u] = w;
}

struct Plan3 {
    bool ok;
    Geometry g;
    int rows, kp;          // rows and padded contraction length of the filter copy the direction uses
    int64_t frag_bytes;
};

Plan3 plan3(bool backward, const daq_conv3d_desc& d) {
    Plan3 pl{};
    const int Do = daq_conv3d_out_d(&d), Ho = daq_conv3d_out_h(&d), Wo = daq_conv3d_out_w(&d);
    if (d.groups != 1 || d.kH * d.kW == 1 || d.strideD > 2 || (!backward && (d.strideH != 1 || d.strideW != 1))) return pl;
    const int kc = backward ? d.Cout : d.Cin, rows = backward ? d.Cin : d.Cout;
    const int Ds = backward ? Do : d.Din, Hs = backward ? Ho : d.Hin, Ws = backward ? Wo : d.Win;
    const int Dd = backward ? d.Din : Do, Hd = backward ? d.Hin : Ho, Wd = backward ? d.Win : Wo;
    pl.kp = (int)round_up(kc, 16);
    pl.rows = rows;
    const int64_t src_bytes = round_up((int64_t)d.N * Ds * Hs * Ws * pl.kp, 256);
    const int nkc_frame = (int)ceil_div(pl.kp, kKc), taps = d.kH * d.kW;
    pl.frag_bytes = (int64_t)d.kD * nkc_frame * taps * ceil_div(rows, 32) * 2048;
    if (src_bytes >= ((int64_t)1 << 31) || pl.frag_bytes >= ((int64_t)1 << 31) || (int64_t)d.N * Dd >= ((int64_t)1 << 31) || Dd > 65535) return pl;
    auto make = [&](int px) {
        return plan(backward, d.N * Dd, Hs, Ws, pl.kp, Hd, Wd, rows, d.kH, d.kW, d.strideH, d.strideW, d.padH, d.padW, d.dilH, d.dilW, px,
                    true);
    };
    Geometry g = plan_small(make(kPxWg), make);
    if (!g.ok || g.a.zfill) return pl;
    HaloArgs& a = g.a;
    a.src_bytes = (uint32_t)src_bytes;
    a.wfrag_bytes = (uint32_t)pl.frag_bytes;
    a.Dd = Dd; a.Ds = Ds; a.kD = d.kD; a.sD_log2 = d.strideD - 1; a.pD = d.padD; a.dD = d.dilD; a.fwd = backward ? 0 : 1;
    a.nkc_frame = nkc_frame;
    a.div_dd = make_fastdiv((uint32_t)Dd);
    a.div_nkc = make_fastdiv((uint32_t)nkc_frame);
    pl.g = g;
    pl.ok = true;
    return pl;
}

daq_status launch3(Plan3& pl, const int8_t* filter, void* frag, const char* name, hipStream_t st) {
    HaloArgs a = pl.g.a;
    const uint32_t units = (uint32_t)(pl.frag_bytes / 16);
    DAQ_LAUNCH("frag_w3", st, hipLaunchKernelGGL(k_frag3, dim3((unsigned)ceil_div(units, 256)), dim3(256), 0, st, filter, pl.rows, pl.kp, a.T, a.RB,
                                                 a.nkc_frame, units, (v4i*)frag));
    a.wfrag = (const int8_t*)frag;
    const int64_t blocks = blocks_per_row_tile(a) * ceil_div(a.Crow, 64);
    a.main_blocks = (int)blocks;
    const bool wide = wide_waves(blocks, 1, 1);
    auto kern = a.stride == 2 ? (a.Crow <= 32 ? k_conv_halo<1, true, 2, 4, 0, 1, kPxWg, true> : k_conv_halo<1, true, 2, 4, 0, 2, kPxWg, true>)
                : a.Crow <= 32 && pl.g.px == kPxWg ? k_conv_halo<1, true, 1, 4, 0, 1, kPxWg, true>
                : taps9_applies(pl.g) ? (pl.g.px == kPxWg ? k_conv_halo<2, true, 1, 4, 9, 1, kPxWg, true> : k_conv_halo<2, true, 1, 4, 9, 1, 128, true>)
                : wide                ? k_conv_halo<2, true, 1, 4, 0, 1, kPxWg, true>
                                      : k_conv_halo<1, true, 1, 4, 0, 2, kPxWg, true>;
    if (!allow_lds((const void*)kern, pl.g.lds_bytes)) return DAQ_ERR_HIP;
    DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(256), pl.g.lds_bytes, st, a));
    return DAQ_OK;
}

// The streaming form serves: 1 x 1, unit stride, no padding, dense, at most 256 output channels.
bool stream_applies(const daq_conv_desc& d, const daq_layout& Lg) {
    return d.groups == 1 && d.kH == 1 && d.kW == 1 && d.strideH == 1 && d.strideW == 1 && d.padH == 0 && d.padW == 0 &&
           Lg.kind == DAQ_LAYOUT_NHWC && Lg.c_pitch <= 256 && (int64_t)d.N * d.Hin * d.Win < ((int64_t)1 << 31) - 64 &&
           ceil_div(std::max(d.Cin, d.Cout), 64) <= 4096;
}

// src: the NHWC operand (layout Ls); wfrag: the fragment-order filter copy whose rows are the result's `rows` channels
daq_status launch_stream(const char* name, const daq_conv_desc& d, const daq_layout& Ls, const int8_t* src,
                         const int8_t* wfrag, int64_t wfrag_bytes, int rows, const float* s_a, const float* s_b, float* out,
                         int32_t* acc, hipStream_t st, const DwTail* tail, bool bf16 = false) {
    StreamArgs a{};
    a.src = src;
    a.wfrag = wfrag;
    a.src_bytes = (uint32_t)Ls.bytes;
    a.wfrag_bytes = (uint32_t)wfrag_bytes;
    a.cp = Ls.c_pitch;
    a.Crow = rows;
    a.RB = (int)ceil_div(rows, 32);
    a.HW = d.Hin * d.Win;
    a.total_px = (uint32_t)((int64_t)d.N * a.HW);
    a.groups = (uint32_t)ceil_div((int64_t)a.total_px, 32);
    a.RP = (int)ceil_div(a.RB, 2);
    const int ks = (int)ceil_div(a.cp, 32);
    // waves the chip holds at this form's register count; a wave should get several groups for its filter fragments
    const int64_t target = ks <= 2 ? 8192 : ks <= 4 ? 4096 : 2048;
    a.S = (int)round_up(std::max<int64_t>(1, std::min<int64_t>(ceil_div((int64_t)a.groups, 2), target / a.RP)), 4);
    a.div_rp = make_fastdiv((uint32_t)a.RP);
    a.div_hw = make_fastdiv((uint32_t)a.HW);
    a.s_a = s_a; a.s_b = s_b;
    a.out = out; a.acc_out = acc;
    a.bf16 = bf16 ? 1 : 0;
    const int64_t wgs = (int64_t)a.RP * ceil_div(a.S, 4);
    if (tail) a.tail = *tail;
    a.main_blocks = (int)wgs;
    const dim3 grid((unsigned)(wgs + a.tail.blocks));
    const int64_t out_bytes = (int64_t)d.N * rows * a.HW * (bf16 ? 2 : 4);
    const int64_t deal = stream_deal(out_bytes, (int64_t)a.HW * (bf16 ? 2 : 4), a.cp, a.RP, wgs);
    a.deal = (uint32_t)std::max<int64_t>(deal, 1);
    a.dealt = (uint32_t)(deal ? wgs / (kXcd * deal) * (kXcd * deal) : 0);
    a.div_deal = make_fastdiv(a.deal);
    const int store = acc || out_bytes >= ((int64_t)1 << 31) || (bf16 && (a.HW & 1)) ? 0 : bf16 ? 2 : 1;
    const bool nt = stream_result(out_bytes, (int64_t)a.HW * (bf16 ? 2 : 4));
    a.out_bytes = store ? (uint32_t)out_bytes : 0u;
#define DAQ_STREAM(KSV)                                                                                                          \
    {                                                                                                                            \
        auto kern = store == 1 ? (nt ? k_dx_1x1_stream<KSV, 1, true> : k_dx_1x1_stream<KSV, 1, false>)                          \
                    : store == 2 ? (nt ? k_dx_1x1_stream<KSV, 2, true> : k_dx_1x1_stream<KSV, 2, false>)                        \
                                 : (nt ? k_dx_1x1_stream<KSV, 0, true> : k_dx_1x1_stream<KSV, 0, false>);                       \
        DAQ_LAUNCH(name, st, hipLaunchKernelGGL(kern, grid, dim3(256), 0, st, a));                                               \
    }
    if (ks <= 1) DAQ_STREAM(1)
    else if (ks <= 2) DAQ_STREAM(2)
    else if (ks <= 4) DAQ_STREAM(4)
    else DAQ_STREAM(8)
#undef DAQ_STREAM
    return DAQ_OK;
}

}  // namespace

static OtherKernel as_other(const Geometry& g) {
    const HaloArgs& a = g.a;
    const int taps = max_taps(a);
    const TileForm form = ring1_applies(g) ? TileForm::kRing1 : taps9_applies(g) ? TileForm::kTaps9 : a.Crow <= 32 ? TileForm::kNarrow : TileForm::kTaps;
    return OtherKernel{form, a.stride > 1, blocks_per_row_tile(a) * ceil_div(a.Crow, 64), taps * (int)ceil_div(a.cp, kKc)};
}

bool bwd_data_halo_supported(const daq_conv_desc& d) { return plan_bwd(d).ok; }

int product_direct_waves(bool backward, const daq_conv_desc& d, bool bf16) {
    daq_layout L;
    if ((backward ? daq_layout_qg(&d, &L) : daq_layout_qx_nhwc(&d, &L)) != DAQ_OK) return 0;
    const Geometry g = backward ? plan_bwd(d) : plan_fwd(d);
    if (g.ok) return stream_applies(d, L) ? 0 : direct_waves(backward, d, as_other(g), bf16);
    return !backward && fwd_mfma_supported(d) ? direct_waves(false, d, fwd_nhwc_as_other(d), bf16) : 0;
}

daq_status conv_bwd_data_halo(const daq_conv_desc& d, const int8_t* qg, const float* s_g, const int8_t* qw,
                              const float* s_w, float* dX, int32_t* acc, hipStream_t st, const DwTail* tail, bool bf16) {
    Geometry g = plan_bwd(d);
    if (tail) g.a.tail = *tail;
    g.a.bf16 = bf16 ? 1 : 0;
    daq_wpack_layout Lw;
    if (!g.ok || daq_layout_qw(&d, &Lw) != DAQ_OK) return DAQ_ERR_UNSUPPORTED;
    daq_layout Lg;
    if (daq_layout_qg(&d, &Lg) == DAQ_OK && stream_applies(d, Lg))
        return launch_stream("conv_bwd_data_stream", d, Lg, qg, qw + Lw.off_bwd_frag, Lw.bytes - Lw.off_bwd_frag, d.Cin, s_w, s_g, dX, acc,
                             st, tail, bf16);
    daq_status rc;
    if (conv_direct(true, d, as_other(g), qg, qw, s_w, s_g, dX, acc, st, tail, bf16, rc)) return rc;
    g.a.src = qg;
    g.a.wfrag = qw + Lw.off_bwd_frag;
    g.a.s_a = s_w; g.a.s_b = s_g;
    g.a.out = dX; g.a.acc_out = acc;
    g.a.nt = !bf16 && stream_result((int64_t)d.N * d.Cin * d.Hin * d.Win * 4, (int64_t)d.Hin * d.Win * 4);
    return launch(g, st, kBwdNames);
}

// The time of the data gradient's part, from which the filter gradient's split follows.  (3 x 3: with 5 and 1.0 us, as waves of 64 x 32 took, 112 <- 80 at 11 x 11,
// batch 26, 13.0 us, 10.9 now; 147 layers 1.010 times the speed, worst 0.993.)
double beside_data_us(bool nine_taps, int chunks) { return nine_taps ? 4.0 + 0.8 * chunks : 4.5 + 0.35 * chunks; }

bool conv_bwd_both_small(const daq_conv_desc& d, const Plan32& plan_w, const int8_t* qx, const float* s_x, const int8_t* vq, const float* s_chan, float* dW,
                         int32_t* dW_acc, const int8_t* qg, const float* s_g, const int8_t* qw, const float* s_w, float* dX, int32_t* dX_acc,
                         void* ws, hipStream_t st, daq_status& rc) {
    Geometry g = plan_bwd(d);
    const BothForm form = both_form(g);
    if (form == kBothNone) return false;
    const int64_t x_blocks = blocks_per_row_tile(g.a) * ceil_div(g.a.Crow, 64);
    if (x_blocks > kBothBlocks - 8) return false;
    // The data gradient by itself may be one for the kernel without staging; that is not asked.  Of 150 drawn layers that both would serve this
    // launch is the faster for 145, 1.43 times the speed over all; level or up to 1.14 times slower from twelve chunks of a 3 x 3 filter on
    // (16 <- 864 channels of 10 x 10, batch 6: 22.7 us here, 20.0 in two launches; 32 <- 786 of 14 x 14, batch 18: 22.0 and 22.7).
    const double x_us = beside_data_us(form == kBothTaps9, (int)ceil_div(g.a.cp, kKc));
    daq_layout Lg;
    const bool streams = daq_layout_qg(&d, &Lg) == DAQ_OK && stream_applies(d, Lg);
    DwBeside w;
    if (!bwd_filter_beside(d, plan_w, qx, s_x, vq, s_chan, dW, dW_acc, ws, kBothBlocks - (int)x_blocks, x_us, streams, w)) return false;
    daq_wpack_layout Lw;
    if (daq_layout_qw(&d, &Lw) != DAQ_OK) return false;
    HaloArgs& a = g.a;
    a.src = qg;
    a.wfrag = qw + Lw.off_bwd_frag;
    a.s_a = s_w;
    a.s_b = s_g;
    a.out = dX;
    a.acc_out = dX_acc;
    a.main_blocks = (int)x_blocks;
    const int x_first = (int)round_up(w.blocks, kXcd);
    const dim3 grid((unsigned)(x_first + x_blocks));
    const size_t lds = std::max(w.lds_bytes, g.lds_bytes);
    auto run = [&]() -> daq_status {
#define DAQ_BOTH(K, F)                                                                                                \
    if (w.k11 == K && form == F) {                                                                                   \
        auto kern = k_bwd_both<K, F>;                                                                                \
        if (!allow_lds((const void*)kern, lds)) return DAQ_ERR_HIP;                                                  \
        DAQ_LAUNCH("conv_bwd_both", st, hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, w.blocks, x_first, w.a, a)); \
        return w.tail.blocks > 0 ? launch_dw_reduce(w.tail, 1, st) : DAQ_OK;                                         \
    }
        DAQ_BOTH(false, kBothTaps9) DAQ_BOTH(false, kBothOneChunk) DAQ_BOTH(false, kBothNarrow)
        DAQ_BOTH(true, kBothRing1) DAQ_BOTH(true, kBothOneChunk) DAQ_BOTH(true, kBothNarrow) DAQ_BOTH(true, kBothRing1S2)
#undef DAQ_BOTH
        return DAQ_ERR_UNSUPPORTED;
    };
    rc = run();
    return rc != DAQ_ERR_UNSUPPORTED;   // nothing was launched
}

bool fwd_halo_supported(const daq_conv_desc& d) { return plan_fwd(d).ok; }

daq_status conv_fwd_halo(const daq_conv_desc& d, const int8_t* qx, const int8_t* qw, const float* s_x, const float* s_w,
                         float* Y, int32_t* acc, hipStream_t st) {
    Geometry g = plan_fwd(d);
    daq_wpack_layout Lw;
    if (!g.ok || daq_layout_qw(&d, &Lw) != DAQ_OK) return DAQ_ERR_UNSUPPORTED;
    daq_layout Lx;
    if (daq_layout_qx_nhwc(&d, &Lx) == DAQ_OK && stream_applies(d, Lx))   // thin 1 x 1 layers: the streaming kernel, rows = Cout
        return launch_stream("conv_fwd_stream", d, Lx, qx, qw + Lw.off_fwd_frag, Lw.off_bwd_frag - Lw.off_fwd_frag, d.Cout, s_x, s_w, Y,
                             acc, st, nullptr);
    daq_status rc;
    if (conv_direct(false, d, as_other(g), qx, qw, s_x, s_w, Y, acc, st, nullptr, false, rc)) return rc;
    g.a.src = qx;
    g.a.wfrag = qw + Lw.off_fwd_frag;
    g.a.s_a = s_x; g.a.s_b = s_w;
    g.a.out = Y; g.a.acc_out = acc;
    g.a.nt = stream_result((int64_t)d.N * d.Cout * daq_out_h(&d) * daq_out_w(&d) * 4, (int64_t)daq_out_h(&d) * daq_out_w(&d) * 4);
    return launch(g, st, kFwdNames);
}

// Whether a layer takes these kernels.  The dot4 kernels need one launch instead of two, and a thread of theirs walks the
// taps and 16-channel records one after the other, about 0.45 us each: short walks over small layers stay there (27 taps,
// 32 channels, 4 x 16 x 16: level), long ones do not (128 channels, 4 x 8 x 8: 95 against 16 us).
static bool mfma3_worthwhile(bool backward, const daq_conv3d_desc& d) {
    const int64_t taps = (int64_t)d.kD * d.kH * d.kW, kc = backward ? d.Cout : d.Cin;
    const int64_t macs = (int64_t)d.N * d.Cout * (d.Cin / d.groups) * taps * daq_conv3d_out_d(&d) * daq_conv3d_out_h(&d) * daq_conv3d_out_w(&d);
    return macs >= ((int64_t)40 << 20) || taps * ceil_div(kc, 16) >= 64;
}

size_t conv3d_halo_ws_bytes(bool backward, const daq_conv3d_desc& d) {
    if (!mfma3_worthwhile(backward, d)) return 0;
    const Plan3 pl = plan3(backward, d);
    return pl.ok ? (size_t)round_up(pl.frag_bytes, 256) : 0;
}

daq_status conv3d_bwd_data_halo(const daq_conv3d_desc& d, const int8_t* qg, const float* s_g, const int8_t* w_bwd, const float* s_w, float* dX,
                                int32_t* acc, void* frag, hipStream_t st) {
    Plan3 pl = plan3(true, d);
    if (!pl.ok) return DAQ_ERR_UNSUPPORTED;
    HaloArgs& a = pl.g.a;
    a.src = qg;
    a.s_a = s_w; a.s_b = s_g;
    a.out = dX; a.acc_out = acc;
    a.nt = (int64_t)a.N * d.Cin * d.Hin * d.Win * 4 >= kStreamBytes;
    return launch3(pl, w_bwd, frag, "conv3d_bwd_data_halo", st);
}

daq_status conv3d_fwd_halo(const daq_conv3d_desc& d, const int8_t* qx, const int8_t* w_fwd, const float* s_x, const float* s_w, float* Y,
                           int32_t* acc, void* frag, hipStream_t st) {
    Plan3 pl = plan3(false, d);
    if (!pl.ok) return DAQ_ERR_UNSUPPORTED;
    HaloArgs& a = pl.g.a;
    a.src = qx;
    a.s_a = s_x; a.s_b = s_w;
    a.out = Y; a.acc_out = acc;
    a.nt = (int64_t)a.N * d.Cout * daq_conv3d_out_h(&d) * daq_conv3d_out_w(&d) * 4 >= kStreamBytes;
    return launch3(pl, w_fwd, frag, "conv3d_fwd_halo", st);
}

}  // namespace daq
