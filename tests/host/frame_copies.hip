// The filter gradient of a 3-D layer reads its operands from copies in the caller's workspace (dw3_plan).  Replays, on the
// host, what a workgroup of the 2-D kernel stages for the last depth tap, channel and chunk and compares it with the
// size that daq_conv3d_workspace_bytes reports, over random layers.  Nothing is launched.
#include "conv_mfma_dw32.hip"
#include "conv3d.hip"

#include <cstdio>
#include <cstdlib>

int main() {
    using namespace daq;
    std::srand(20210204);
    auto pick = [](int lo, int hi) { return lo + std::rand() % (hi - lo + 1); };
    int plans = 0, at_the_end = 0, bad = 0;
    for (int i = 0; i < 200000; ++i) {
        const int k = pick(0, 3) ? 3 : 1, s = k == 1 ? 2 : pick(1, 2);   // (1 x 1 frames at unit stride are 2-D problems)
        const int kD = pick(1, 5), dD = pick(1, 3), sD = pick(0, 2) ? 1 : pick(2, 3), pD = pick(0, 4);
        const int channels = i % 2 ? pick(1, 96) : 16 * pick(4, 20);
        const daq_conv3d_desc d = {pick(1, 16), channels, pick(1, 12), pick(3, 60), pick(3, 60), pick(16, 160), kD, k, k, sD, s, s,
                                   pD, k / 2, k / 2, dD, 1, 1, 1};
        daq_conv_desc cx, cg;
        if (daq_conv3d_carriers(&d, &cx, &cg) != 0) continue;
        const Dw3Plan p = dw3_plan(d);
        if (!p.ok) continue;
        ++plans;
        const Plan32 pl = make_plan32(p.frames, kD);
        const int64_t staged = (int64_t)(pl.nchunks - 1) * kKC + (pl.k11 ? kKC : 16 * pl.b_units);   // of one operand row
        const int64_t frame = (int64_t)p.Lx.img_rows * p.Lx.row_pitch;
        int64_t end = 0;
        for (int kd = 0; kd < kD; ++kd) {
            const int64_t base = (int64_t)(kd * dD % sD) * p.Lx.bytes + (int64_t)(kd * dD / sD) * frame;
            end = std::max(end, base + (int64_t)(d.Cin - 1) * p.Lx.chan_pitch + (pl.s2 ? 3 : 0) * p.Lx.plane_pitch + staged);
        }
        const int64_t ws = (int64_t)daq_conv3d_workspace_bytes(DAQ_OP_CONV_BWD_FILTER, &d);
        const bool g_ok = (int64_t)pl.nchunks * kKC == p.Lg.plane_pitch && p.off_g + p.Lg.bytes <= p.off_x;
        if (end > p.Lx.bytes * sD) ++at_the_end;   // more than the copy itself
        if (p.off_x + end > ws || !g_ok) {
            if (++bad <= 5)
                std::printf("N %d Cin %d D %d H %d W %d Cout %d k %d %d stride %d %d pad %d dil %d: %lld bytes past the workspace\n", d.N, d.Cin, d.Din,
                            d.Hin, d.Win, d.Cout, kD, k, sD, s, pD, dD, (long long)(p.off_x + end - ws));
        }
    }
    std::printf("%d plans, %d read past the copy, %d past the workspace\n", plans, at_the_end, bad);
    return bad == 0 && plans > 10000 && at_the_end > 100 ? 0 : 1;
}
