// plane_lists.hpp -- which plane segments of a batch share a launch
// (k_plane.hip).  Host code without HIP: plain integers in and out.
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace pk {

// planes of one shape: LDS and threads of a plane, planes (workgroups) of all
// problems
struct PlaneSeg {
    size_t lds;
    int threads;
    long planes;
};

// workgroups of this LDS and thread count that one compute unit holds
inline int planes_per_cu(size_t lds, int threads)
{
    const long by_lds = (long)(160 * 1024 / lds), by_waves = 2048 / threads;
    return (int)std::max(1L, std::min(by_lds, by_waves));
}

// The launches, each a list of indices into `segs` in their order (the largest
// problems first, whose workgroups are dealt out first: 10 of 64x128x95 ahead of 6
// of 96x96x35, FP64 forward, 42 us, behind them 47).  Every workgroup of a launch
// gets the LDS of its largest plane, so much smaller planes gain from a launch of
// their own, with more of them per compute unit; but launches run one after the
// other, and each costs about the time of one plane.
inline std::vector<std::vector<int>> plane_launches(const std::vector<PlaneSeg> &segs, int max_seg)
{
    std::vector<std::vector<int>> out;
    long rest = 0, held = 0;
    for (const PlaneSeg &s : segs) rest += s.planes;
    size_t most = 0, least = 0;  // LDS of the last launch's planes
    const int n = (int)segs.size();
    for (int i = 0; i < n; ++i) {
        const PlaneSeg &s = segs[i];
        // workgroup slots that planes [from, to) lose to an allotment of `lds`
        auto lost = [&](int from, int to, size_t own, size_t lds) {
            double slots = 0.0;
            for (int k = from; k < to; ++k)
                slots += (double)segs[k].planes * (1.0 / planes_per_cu(lds, segs[k].threads) -
                                                   1.0 / planes_per_cu(own, segs[k].threads));
            return slots;
        };
        bool cut = out.empty() || (int)out.back().size() == max_seg;
        if (!cut && 5 * s.lds < 3 * most) {
            // much smaller planes from here on: both sides have to fill the
            // device, the smaller planes twice -- or nearly once where each
            // side is one shape and gets the kernel of that shape.  Graph
            // loops, us, always split -> one launch -> this rule:
            //   one problem of each of 7 shapes, FP64: 150 -> 102 -> 101
            //   24 of 64^3, 24 of 96x96x48, 16 of 128x128x64, FP32 + refinement:
            //     922 -> 981 -> 922
            //   11 of 96x128x84, 10 of 48x128x34, the same: 420 -> 438 -> 420
            // The larger planes may be fewer where the others lose 300 slots.
            cut = (held >= 256 && rest >= (n == 2 ? 320 : 512)) ||
                  lost(i, n, s.lds, most) >= 300.0;
        } else if (!cut && 5 * least < 3 * s.lds) {
            // much larger planes (of fewer points).  16 of 64x64x96, 8 of
            // 128x128x16: FP64 one launch 190 us, two 165; FP32 + refinement 352
            // and 310
            cut = lost(out.back()[0], i, most, s.lds) >= 300.0;
        }
        if (cut) {
            out.emplace_back();
            held = 0;
            most = 0;
            least = s.lds;
        }
        out.back().push_back(i);
        held += s.planes;
        rest -= s.planes;
        most = std::max(most, s.lds);
        least = std::min(least, s.lds);
    }
    return out;
}

}  // namespace pk
