// Which form of a kernel a call takes, at sizes where the other one was measured slower.
#include <cstdio>

#include "daq_internal.h"
#include "dw32_role.h"

static int fails = 0;
#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); ++fails; } \
    } while (0)

using namespace daq;

static daq_conv_desc layer(int N, int cin, int H, int W, int cout, int k, int stride) {
    return daq_conv_desc{N, cin, H, W, cout, k, k, stride, stride, k / 2, k / 2, 1, 1, 1};
}

// 1 x 1 filter gradients of many chunks to a workgroup.
static void long_filter_gradients() {
    auto is_long = [](const daq_conv_desc& d) {
        const Plan32 pl = make_plan32(d);
        return pl.ok && pl.k11 && dw11_long(ceil_div(pl.nchunks, pl.splits));
    };
    EXPECT(is_long(layer(128, 512, 7, 7, 2048, 1, 1)) && is_long(layer(128, 2048, 7, 7, 512, 1, 1)) && is_long(layer(128, 1024, 14, 14, 512, 1, 1)));
    EXPECT(is_long(layer(128, 512, 28, 28, 1024, 1, 2)) && is_long(layer(122, 1472, 13, 13, 136, 1, 1)));
    EXPECT(!is_long(layer(3, 32, 70, 70, 1312, 1, 2)) && !is_long(layer(64, 64, 14, 14, 384, 1, 1)) && !is_long(layer(64, 512, 7, 7, 2048, 1, 1)));
}

// Streaming 1 x 1 products: the blocks that an XCD takes in a row.
static void dealt_blocks() {
    auto deal = [](int N, int rows, int H, int W, int cp, int64_t blocks) {
        return stream_deal((int64_t)N * rows * H * W * 4, (int64_t)H * W * 4, cp, (int)ceil_div(rows, 64), blocks);
    };
    EXPECT(deal(50, 1499, 43, 43, 64, 2064) == 0 && deal(122, 1015, 22, 22, 16, 2048) == 0 && deal(44, 512, 22, 22, 16, 672) == 0);   // a multiple of eight pairs
    EXPECT(deal(53, 1936, 20, 18, 48, 2046) == 0 && deal(106, 1952, 29, 28, 32, 2046) == 0);                                       // nearly
    EXPECT(deal(18, 1776, 24, 26, 128, 1036) == 0 && deal(2, 1880, 72, 72, 128, 1020) == 0);                                       // whole lines, many pairs
    EXPECT(deal(12, 1368, 75, 75, 192, 528) == 2 * 22 && deal(51, 1304, 50, 51, 192, 525) == 2 * 21);                              // few blocks
    EXPECT(deal(65, 480, 50, 51, 256, 512) == 2 * 8 && deal(84, 240, 45, 44, 256, 512) == 8 * 4 && deal(10, 2048, 13, 14, 160, 256) == 0);
    EXPECT(deal(34, 320, 61, 61, 16, 2000) == 8 * 5 && deal(64, 512, 28, 28, 256, 512) == 4 * 8 && deal(64, 448, 28, 28, 256, 504) == 4 * 7);
    EXPECT(deal(110, 311, 27, 23, 48, 1000) == 8 * 5 && deal(128, 384, 14, 14, 64, 1024) == 128 && deal(86, 48, 45, 45, 16, 1024) == 128);
}

// 1 x 1 products on 128-pixel tiles: one by one where no two tiles share a line of the result.
static void order_of_tiles() {
    EXPECT(tiles_by_rows(7, 7, 1, 1, 1, 7, 7, 4, 64, 8) && tiles_by_rows(7, 7, 1, 1, 1, 7, 7, 2, 64, 8));          // whole images: 512 <- 2048, batch 128
    EXPECT(!tiles_by_rows(7, 7, 1, 1, 1, 7, 7, 4, 41, 15) && tiles_by_rows(7, 7, 1, 1, 1, 7, 7, 4, 4, 28));        // many tiles, no multiple of eight
    EXPECT(tiles_by_rows(2, 48, 24, 1, 1, 48, 48, 4, 96, 4) && !tiles_by_rows(2, 47, 24, 1, 1, 47, 47, 4, 96, 4)); // whole rows, on lines and off them
    EXPECT(tiles_by_rows(8, 16, 8, 4, 1, 64, 64, 4, 160, 4) && !tiles_by_rows(8, 12, 8, 4, 1, 64, 48, 4, 160, 4)); // pieces of rows
    EXPECT(!tiles_by_rows(9, 14, 2, 1, 1, 14, 14, 4, 128, 1) && tiles_by_rows(4, 28, 7, 1, 2, 56, 56, 4, 56, 8) && !tiles_by_rows(1, 56, 56, 1, 1, 56, 56, 2, 56, 8));
    EXPECT(tiles_spread(16, 16, 3, 3, 48, 48, 4, 522, 8) && tiles_spread(16, 16, 3, 3, 48, 48, 4, 558, 4) && tiles_spread(16, 16, 3, 3, 48, 48, 4, 216, 2));
    EXPECT(!tiles_spread(12, 20, 2, 1, 20, 20, 4, 38, 16) && !tiles_spread(3, 74, 25, 1, 74, 74, 4, 144, 7) && tiles_spread(14, 14, 1, 1, 14, 14, 4, 128, 16));
}

// The tile kernel with a run-time tap list, and of 1 x 1 filters.
static void waves_of_tiles() {
    EXPECT(wide_waves(4932, 1, 25) && wide_waves(513, 2, 9) && wide_waves(3920, 3, 2) && wide_waves(4320, 1, 49));
    EXPECT(wide_waves1(396, 2, 11) && wide_waves1(2049, 1, 56) && !wide_waves1(2048, 1, 11) && !wide_waves1(520, 2, 40));
    EXPECT(!wide_waves(512, 1, 25) && !wide_waves(1428, 3, 25) && !wide_waves(912, 3, 25) && !wide_waves(888, 6, 25) && !wide_waves(1053, 4, 7));
}

// Products of few tiles: the kernel without staging or the tile kernel, as that is now.
static void few_tiles() {
    auto fwd = [](const daq_conv_desc& d) { return product_direct_waves(false, d, false) > 0; };
    auto bwd = [](const daq_conv_desc& d) { return product_direct_waves(true, d, false) > 0; };
    EXPECT(!bwd(layer(2, 208, 27, 27, 637, 3, 1)) && !bwd(layer(9, 32, 35, 35, 288, 3, 1)) && !bwd(layer(4, 112, 23, 23, 240, 3, 1)));   // 1.15 to 1.35 times the time
    EXPECT(bwd(layer(8, 896, 29, 29, 16, 7, 1)) && bwd(layer(64, 272, 9, 9, 129, 7, 1)) && bwd(layer(3, 168, 56, 56, 960, 3, 2)));        // 1.1 to 1.45 the other way
    EXPECT(!bwd(layer(17, 1280, 7, 7, 824, 5, 1)) && !bwd(layer(6, 976, 64, 64, 765, 3, 2)));                                              // large ones, 1.05 to 1.3
    EXPECT(!bwd(layer(128, 512, 7, 7, 2048, 1, 1)) && !product_direct_waves(true, layer(128, 512, 7, 7, 2048, 1, 1), true) && !bwd(layer(64, 320, 7, 7, 1280, 1, 1)));   // twice
    EXPECT(fwd(layer(16, 224, 12, 12, 400, 5, 1)) && fwd(layer(13, 176, 11, 11, 480, 5, 1)) && fwd(layer(1, 368, 6, 6, 808, 3, 1)));
}

// Both gradients in one launch: the filter gradient's splits by the time of the data gradient's part as it is now.
static void joint_launch() {
    auto splits = [](const daq_conv_desc& d, int blocks_left, int chunks) {
        DwBeside w;
        const Plan32 pl = make_plan32(d);
        if (!bwd_filter_beside(d, pl, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, reinterpret_cast<void*>(256), blocks_left, beside_data_us(true, chunks), false, w)) return 0;
        return w.a.splits;
    };
    EXPECT(splits(layer(26, 112, 11, 11, 80, 3, 1), 204, 2) > 1 && splits(layer(8, 16, 17, 17, 80, 3, 1), 238, 2) > 1 && splits(layer(4, 36, 28, 28, 128, 3, 1), 224, 2) > 1);
}

int main() {
    long_filter_gradients();
    dealt_blocks();
    order_of_tiles();
    waves_of_tiles();
    few_tiles();
    joint_launch();
    std::printf("%d failures\n", fails);
    return fails != 0;
}
