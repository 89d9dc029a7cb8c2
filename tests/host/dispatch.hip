// Rules of the dispatch at sizes where an earlier one cost time: each line a call that was measured slower than another form of it.
#include <cstdio>

#include "daq_internal.h"

static int fails = 0;
#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) { std::printf("FAILED line %d: %s\n", __LINE__, #cond); ++fails; } \
    } while (0)

using namespace daq;

static void resident_quantizer() {
    EXPECT(!resident_pays(16, 22 * 703));                                   // 22 images of 53 x 53, 16 channels
    EXPECT(!resident_pays(4, 8 * 1561) && !resident_pays(30, 60 * 160));
    EXPECT(!resident_pays(96, 66 * 200));                                   // 66 images of 114 x 7
    EXPECT(!resident_pays(268, 83 * 144));                                  // a second round of twelve workgroups
    EXPECT(resident_pays(16, 5000) && resident_pays(128, 9460) && resident_pays(512, 12544) && resident_pays(300, 14000));
    EXPECT(!fold_in_packing(672 * 25) && fold_in_packing(192 * 4));         // depthwise: 672 channels of 38 x 38, batch 34
    auto is = [](int C, int64_t units, int nu, int waves) {
        const ResidentForm f = resident_form(C, units);
        return f.nu == nu && f.waves == waves;
    };
    EXPECT(is(546, 44 * 324, 16, 16) && is(328, 38 * 361, 16, 16));         // not 14 waves
    EXPECT(is(678, 108 * 49, 8, 12) && is(1024, 5289, 8, 12));              // not 6 waves of 16 units
    EXPECT(is(2048, 2795, 4, 12) && is(2048, 7998, 16, 8) && is(256, 7998, 8, 16) && is(700, 9460, 16, 12));
    for (int C : {1, 3, 200, 257, 700, 3000})
        for (int64_t units = 1; units <= 16 * 1024; ++units) {
            const ResidentForm f = resident_form(C, units);
            EXPECT((int64_t)f.nu * f.waves * kWave >= units && f.waves >= 1 && f.waves <= 16 && (f.waves <= 4 || f.waves % 4 == 0));
        }
}

int main() {
    resident_quantizer();
    std::printf("%d failures\n", fails);
    return fails != 0;
}
