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

int main() {
    long_filter_gradients();
    std::printf("%d failures\n", fails);
    return fails != 0;
}
