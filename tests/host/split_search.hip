// cheapest_split against the search over every count, and the number of costs it looks at: planning is host time of every call.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "daq_internal.h"

int main() {
    using namespace daq;
    std::srand(7);
    auto pick = [](int lo, int hi) { return lo + std::rand() % (hi - lo + 1); };
    int bad = 0, most = 0;
    for (int i = 0; i < 100000; ++i) {
        const int64_t tiles = i % 2 ? pick(1, 20) : pick(1, 1200), n = i % 3 ? pick(1, 300) : pick(1, 40000);
        SplitModel m{n, tiles, 1024 / tiles, 0.01 * pick(5, 400), 4.0, i % 5 ? 0.0 : (double)pick(0, 20), 5.0, i % 4 ? 1e-3 * pick(1, 40) * (double)tiles : 0.0};
        int want = 1, tried = 0;
        double best = 0.0;
        for (int64_t s = 1; s <= n && (s == 1 || s <= m.limit); ++s) {
            double c = (double)ceil_div(tiles * s, 256) * std::max((double)ceil_div(n, s) * m.t_step + m.t_fixed, m.t_floor);
            if (s > 1) c += m.t_reduce + m.t_part * (double)s;
            if (s == 1 || c < best) { best = c; want = (int)s; }
        }
        const int got = cheapest_split(m, &tried);
        most = std::max(most, tried);
        if (got != want && ++bad <= 5)
            std::printf("n %lld tiles %lld step %g floor %g part %g: %d, cheapest %d\n", (long long)n, (long long)tiles, m.t_step, m.t_floor, m.t_part, got, want);
    }
    std::printf("%d bad, at most %d costs looked at\n", bad, most);
    return bad != 0 || most > 64;
}
