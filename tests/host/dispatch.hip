// Rules of the dispatch at sizes where an earlier one cost time: each line a call that was measured slower than another form of it.
#include <cstdio>
#include <cstring>

#include "daq_internal.h"
#include "dw32_role.h"

static int fails = 0;
#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); ++fails; } \
    } while (0)

using namespace daq;

static void resident_quantizer() {
    auto pays = [](int C, int64_t units, const char* kind) {                // p: padded planes, t: not whole units, s: stochastic codes
        return resident_pays(C, units, std::strchr(kind, 'p'), std::strchr(kind, 't'), std::strchr(kind, 's'));
    };
    EXPECT(!pays(16, 22 * 703, "pts"));                                     // 22 images of 53 x 53, 16 channels
    EXPECT(!pays(4, 8 * 1561, "pts") && !pays(30, 60 * 160, "s"));
    EXPECT(!pays(96, 66 * 200, "pts"));                                     // 66 images of 114 x 7
    EXPECT(pays(85, 102 * 64, "s") && pays(97, 84 * 169, "s"));
    EXPECT(!pays(268, 83 * 144, "s"));                                      // a second round of twelve workgroups
    EXPECT(pays(16, 5000, "pts") && pays(128, 9460, "pts") && pays(512, 12544, "s") && pays(300, 14000, "pts"));
    EXPECT(pays(16, 9 * 729, "") && pays(25, 3 * 2475, "") && pays(12, 14 * 578, ""));   // frames of 27 x 27, 30 x 30 and 34 x 34
    EXPECT(pays(4, 8000, "p") && pays(4, 8000, "t") && pays(32, 8000, "pt") && !pays(16, 9460, "pt") && !pays(4, 14272, ""));
    EXPECT(!fold_in_packing(672 * 25) && fold_in_packing(192 * 4));         // depthwise: 672 channels of 38 x 38, batch 34
    auto is = [](int C, int64_t units, int nu, int waves) {
        const ResidentForm f = resident_form(C, units);
        return f.nu == nu && f.waves == waves;
    };
    EXPECT(is(546, 44 * 324, 16, 16) && is(328, 38 * 361, 16, 16));         // not 14 waves
    EXPECT(is(678, 108 * 49, 8, 12) && is(1024, 5289, 8, 12));              // not 6 waves of 16 units
    EXPECT(is(1240, 2401, 8, 8));                                           // five of eight units in use, not four of four on 12 waves
    EXPECT(is(2048, 2795, 4, 12) && is(2048, 7998, 16, 8) && is(256, 7998, 8, 16) && is(700, 9460, 16, 12));
    for (int C : {1, 3, 200, 257, 700, 3000})
        for (int64_t units = 1; units <= 16 * 1024; ++units) {
            const ResidentForm f = resident_form(C, units);
            EXPECT((int64_t)f.nu * f.waves * kWave >= units && f.waves >= 1 && f.waves <= 16 && (f.waves <= 4 || f.waves % 4 == 0));
        }
}

// The resident launch that writes the global copy too: every workgroup reads the whole tensor.
static void resident_both_copies() {
    auto pays = [](int C, int64_t M) { return resident_all_pays(C, M, ceil_div(M, 4)); };
    EXPECT(!pays(8192, 8) && !pays(5120, 16) && !pays(2048, 40) && !pays(1536, 1));   // up to six times the two launches
    EXPECT(!pays(1024, 49) && !pays(640, 128) && !pays(512, 160) && !pays(264, 256));
    EXPECT(pays(16, 1024) && pays(80, 1024) && pays(256, 256) && pays(384, 160) && pays(520, 64) && pays(768, 16) && pays(1024, 16));
    for (int C = 1; C <= 12000; ++C)
        for (int64_t M : {1, 2, 3, 5, 16, 49, 100, 300, 1000, 1024, 1025, 5000})
            if (pays(C, M)) EXPECT(ceil_div(M, 4) <= 2 * 8 * kWave && ceil_div(C, 256) * C * M <= 120 * 1024);   // units of the launch's threads
}

// The packing launch behind an early copy: its workgroups mostly return at once, and their number does not follow the row length.
static void early_packing() {
    EXPECT(early_pack_blocks(72 * 143) == 3 && early_pack_blocks(131 * 49) == 2 && early_pack_blocks(49) == 1);
    EXPECT(early_pack_blocks(32 * 3136) == 16 && early_pack_blocks(4096) == 1 && early_pack_blocks(4097) == 2);
}

// From which size on the counting sweep writes both copies: calls that got slower with them.
static void early_copy() {
    const int64_t mi = 1 << 20;
    enum { kNearest = 1, kPadded = 2, kBf16 = 4, kGiven = 8, kChannelMajor = 16 };
    auto from = [](int flags, int vector, int W) {
        return early_copy_from({bool(flags & kGiven), bool(flags & kNearest), bool(flags & kPadded), bool(flags & kBf16), bool(flags & kChannelMajor), vector, W});
    };
    EXPECT(from(kNearest, 4, 56) > 5 * mi && from(kNearest | kPadded, 4, 56) > 7 * mi && from(kNearest | kPadded, 0, 49) > 7 * mi);
    EXPECT(from(kNearest | kPadded | kBf16, 4, 56) > 7 * mi && from(kNearest | kPadded | kBf16, 0, 49) > 5 * mi);
    EXPECT(from(kNearest | kPadded | kGiven, 0, 31) > 12 * mi && from(kNearest | kChannelMajor | kPadded, 0, 7) > 100 * mi);
    for (int vector : {0, 2, 4}) EXPECT(from(0, vector, 56) == 4 * mi && from(kPadded | kBf16, vector, 56) == 4 * mi);
    EXPECT(from(kNearest, 2, 26) == 4 * mi && from(kNearest, 0, 49) == 4 * mi && from(kNearest | kPadded, 2, 26) == 8 * mi);
    EXPECT(from(kGiven, 0, 49) == 3 * mi && from(kGiven | kNearest, 0, 49) == 3 * mi && from(kGiven | kPadded, 0, 49) == 3 * mi);
    for (int flags : {0, (int)kNearest, (int)kPadded, kNearest | kPadded}) EXPECT(from(flags | kGiven, 2, 26) == 0 && from(flags | kGiven, 4, 56) == 0);
    EXPECT(from(kChannelMajor | kPadded, 0, 7) == 4 * mi && from(kChannelMajor | kPadded | kNearest, 0, 49) == 4 * mi && from(kChannelMajor | kNearest | kGiven, 0, 7) == 3 * mi);
}

// The counting pass: blocks of channels by the size of the tensor, and what its kernel and its buffers take for granted.
static void counting_pass() {
    auto width = [](int C, int N, int HW) { return plan_count(C, N, HW).width; };
    EXPECT(width(80, 40, 3136) == 4 && width(74, 99, 26 * 26) == 4);        // not workgroups of five waves
    EXPECT(width(240, 14, 3136) == 8 && width(400, 16, 3136) == 8 && width(400, 80, 3136) != 5);
    EXPECT(width(144, 20, 3136) == 8 && width(3000, 37, 143) == 8 && width(1216, 107, 81) == 8);   // not 9 or 12 waves a CU
    EXPECT(width(880, 9, 27 * 29) == 4 && width(128, 12, 3136) == 4);       // under two rounds
    EXPECT(width(112, 14, 3136) == 7 && width(144, 128, 3136) == 9 && width(96, 128, 12544) == 6 && width(792, 37, 59 * 63) == 10);
    // the sizes of test_counting_pass_wide_blocks: width, and channel groups of the last block
    auto is = [](int C, int N, int HW, int width, int last) {
        const CountPlan p = plan_count(C, N, HW);
        return p.width == width && p.groups(C, p.blocks - 1) == last && p.tiles > 2 * p.cgroups * (p.waves / p.groups(C, 0));   // and several turns
    };
    EXPECT(is(112, 4, 140 * 139, 7, 7) && is(240, 3, 112 * 112, 8, 7) && is(200, 20, 45 * 49, 8, 5) && is(272, 11, 55 * 57, 8, 1));
    EXPECT(is(208, 20, 101 * 103, 7, 6) && is(270, 16, 99 * 101, 9, 8) && is(400, 35, 56 * 56, 9, 7) && is(186, 73, 56 * 56, 12, 12));
    for (int C = 1; C <= 9000; C += C < 420 ? 1 : 37)
        for (int N : {1, 3, 16, 128, 700})
            for (int HW : {1, 2, 3, 4, 49, 143, 784, 3136, 12544, 50176}) {
                if ((int64_t)C * N * HW >= (int64_t)1 << 29) continue;
                for (int given : {0, 4, 8}) {
                    const CountPlan p = plan_count(C, N, HW, given);
                    const int G = (C + 15) / 16;
                    EXPECT(p.width <= p.waves && p.waves <= kCountMaxWaves && (p.blocks - 1) * p.width < G && p.blocks * p.width >= G);
                    EXPECT(1 <= p.cgroups_last && p.cgroups_last <= p.cgroups && p.cgroups <= kCountGroups);
                    EXPECT(p.tile_dwords(C) * 8 <= 48 << 10);               // two tiles of LDS, no more than a launch has without asking
                    if (given) EXPECT(p.tile_dwords(C) <= CountPlan::most_tile_dwords(given));   // the forward's, whose LDS is of a fixed size
                    for (int b = 0; b < 2; ++b)
                        for (uint32_t i = 0, gb = (uint32_t)p.groups(C, b ? p.blocks - 1 : 0); i < 64 * kCountMaxWaves; ++i)
                            EXPECT(i * p.by_groups[b] >> 16 == i / gb);
                }
            }
}

// The forward sweep that writes both copies: records in blocks of 128 channels from 24 Mi elements on (the sizes of test_forward_wide_blocks).
static void forward_blocks() {
    EXPECT(forward_waves(384, 55, 71 * 70, 48) == 8 && forward_waves(384, 60, 58 * 58, 48) == 8);                       // slower in pieces of 64 bytes
    EXPECT(forward_waves(64, 128, 112 * 112, 48) == 4 && forward_waves(256, 16, 3136, 48) == 4 && forward_waves(8192, 2048, 3, 48) == 4);
    EXPECT(forward_waves(80, 101, 3136, 48) == 8 && forward_waves(100, 79, 57 * 57, 48) == 8 && forward_waves(129, 59, 58 * 58, 48) == 8);
    EXPECT(forward_waves(208, 25, 71 * 70, 48) == 8 && forward_waves(400, 77, 27 * 31, 48) == 8 && forward_waves(72, 23400, 15, 48) == 8);
    EXPECT(forward_waves(768, 37, 37 * 37, 256) == 8 && forward_waves(864, 60, 37 * 37, 512) == 4 && forward_waves(2677, 296, 36, 168) == 4);   // many workgroups for the filter
}

static daq_conv_desc layer(int n, int ci, int h, int w, int co, int k, int s) { return daq_conv_desc{n, ci, h, w, co, k, k, s, s, k / 2, k / 2, 1, 1, 1}; }

static void filter_gradient() {
    auto splits = [](daq_conv_desc d) { return make_plan32(d).splits; };
    EXPECT(splits(layer(11, 54, 7, 59, 56, 3, 2)) > 1 && splits(layer(5, 10, 39, 39, 386, 3, 2)) > 1);
    EXPECT(splits(layer(10, 16, 13, 13, 314, 3, 1)) > 1 && splits(layer(9, 26, 5, 32, 67, 3, 1)) > 1);
    EXPECT(splits(layer(43, 434, 8, 46, 689, 1, 1)) == 2);                  // not three
    EXPECT(splits(layer(4, 16, 16, 16, 16, 3, 1)) >= 1);
    EXPECT(splits(layer(16, 384, 14, 14, 64, 1, 1)) == 1 && splits(layer(16, 64, 14, 14, 384, 1, 1)) == 1);   // a launch more for 1.3 us
    EXPECT(splits(layer(16, 96, 56, 56, 24, 1, 1)) > 1);
    for (const daq_conv_desc& d : {layer(90, 513, 77, 6, 193, 3, 1), layer(38, 707, 9, 53, 321, 3, 1), layer(15, 649, 16, 19, 750, 3, 1)}) {
        const Plan32 pl = make_plan32(d);                                   // rectangles may not cost a round over an XCD's CUs
        const int64_t most = pl.bands_m ? (int64_t)pl.band_m * pl.band_n : ceil_div((int64_t)pl.tiles_m * pl.tiles_n * pl.splits, kXcd);
        EXPECT(ceil_div(most, 32) <= ceil_div((int64_t)pl.tiles_m * pl.tiles_n * pl.splits, 256));
    }
    EXPECT(make_plan32(layer(30, 7, 99, 12, 106, 3, 1)).splits_tail > 32 && make_plan32(layer(79, 53, 18, 18, 303, 1, 1)).splits_tail > 32);
    EXPECT(make_plan32(layer(4, 16, 16, 16, 16, 3, 1)).splits_tail <= 6);   // six chunks
    auto beside = [](daq_conv_desc d, int blocks_left, double other_us, bool streams) {
        DwBeside out;
        return bwd_filter_beside(d, make_plan32(d), nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, reinterpret_cast<void*>(256), blocks_left,
                                 other_us, streams, out);
    };
    EXPECT(!beside(layer(26, 4, 33, 33, 395, 3, 1), 22, 12.0, false) && !beside(layer(61, 6, 34, 12, 105, 3, 1), 12, 7.0, false));
    EXPECT(!beside(layer(6, 62, 59, 59, 10, 1, 1), 150, 4.9, true));
    EXPECT(beside(layer(4, 16, 16, 16, 16, 3, 1), 240, 6.0, false) && beside(layer(5, 100, 29, 31, 70, 3, 1), 200, 7.0, false));
    EXPECT(beside(layer(33, 431, 8, 8, 190, 1, 2), 200, 5.6, false));
    auto beside_splits = [](daq_conv_desc d, int blocks_left, double other_us) {
        DwBeside out;
        const bool ok = bwd_filter_beside(d, make_plan32(d), nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, reinterpret_cast<void*>(256),
                                          blocks_left, other_us, false, out);
        return ok ? out.a.splits : 0;
    };
    EXPECT(beside_splits(layer(4, 16, 16, 16, 16, 3, 1), 252, 4.9) == 1);   // six chunks: no reduction's launch for them
    EXPECT(beside_splits(layer(4, 12, 25, 20, 20, 3, 1), 240, 4.9) > 1);    // 32 and more: shared out
}

// Products without staging: what goes back to the tile kernel, and the waves to a tile of the layers of test_products_of_few_tiles.
static void products() {
    auto fwd = [](daq_conv_desc d) { return product_direct_waves(false, d, false); };
    auto bwd = [](daq_conv_desc d) { return product_direct_waves(true, d, false); };
    EXPECT(!fwd(layer(37, 871, 34, 34, 16, 1, 1)) && !fwd(layer(16, 1219, 63, 50, 16, 1, 1)) && !fwd(layer(10, 1397, 51, 51, 6, 1, 1)));   // a source beyond the L2s
    EXPECT(!fwd(layer(71, 7, 135, 135, 4, 3, 1)) && !bwd(layer(101, 5, 123, 123, 10, 5, 2)));                                            // hundreds of tiles a CU
    EXPECT(fwd(layer(6, 768, 5, 5, 52, 5, 1)) && fwd(layer(23, 3, 16, 16, 96, 7, 2)) && fwd(layer(39, 3, 133, 133, 96, 3, 2)));
    EXPECT(fwd(layer(26, 1173, 14, 14, 37, 1, 1)) && bwd(layer(20, 649, 5, 5, 985, 1, 1)));
    auto both = [&](daq_conv_desc d, int f, int b) {
        if (fwd(d) != f || bwd(d) != b) { std::printf("FAILED: %d and %d waves, not %d and %d\n", fwd(d), bwd(d), f, b); ++fails; }
    };
    both(layer(1, 1, 1, 1, 1, 3, 1), 2, 2);
    both(layer(2, 16, 9, 11, 33, 5, 1), 4, 8);
    both(layer(3, 40, 7, 9, 65, 3, 1), 4, 8);
    both(daq_conv_desc{2, 70, 13, 5, 31, 1, 7, 1, 1, 3, 3, 1, 1, 1}, 8, 2);
    both(layer(3, 3, 17, 15, 40, 7, 2), 8, 8);
    both(layer(4, 50, 14, 13, 60, 3, 2), 8, 2);
    both(layer(3, 130, 9, 8, 20, 1, 2), 2, 1);
    both(daq_conv_desc{2, 33, 15, 14, 40, 3, 3, 2, 2, 2, 2, 2, 2, 1}, 4, 2);
    both(layer(2, 20, 14, 16, 40, 3, 3), 4, 0);
    both(layer(41, 20, 64, 65, 40, 5, 2), 1, 0);
    both(layer(19, 80, 35, 41, 5, 5, 1), 8, 1);
    both(layer(12, 96, 32, 33, 64, 3, 2), 8, 0);
}

int main() {
    resident_quantizer();
    resident_both_copies();
    early_packing();
    early_copy();
    counting_pass();
    forward_blocks();
    filter_gradient();
    products();
    std::printf("%d failures\n", fails);
    return fails != 0;
}
