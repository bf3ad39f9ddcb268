// plane_lists.hpp -- which plane segments of a batch share a launch
// (k_plane.hip).  Host code without HIP: plain integers in and out.
#pragma once
#include <algorithm>
#include <cstddef>
#include <numeric>
#include <vector>

namespace pk {

// planes of one shape: LDS of a plane, planes (workgroups) of all problems
struct PlaneSeg {
    size_t lds;
    long planes;
};

// The launches, each a list of indices into `segs`.  Every workgroup of a
// launch gets the LDS of its largest plane, so much smaller planes have a
// launch of their own, with more of them per compute unit.  The launches run
// one after the other, so a split pays only where the larger planes occupy
// half of the 256 compute units and the smaller ones all of them twice.
// Graph loops, us, always split -> one launch -> this rule:
//   one problem of each of 7 shapes, FP64: 154 -> 102 -> 100
//   16 of 64x64x96 and 8 of 128x128x16, FP64 169 -> 176 -> 165, FP32 + refinement
//     314 -> 338 -> 309
//   24 of 64^3, 24 of 96x96x48, 16 of 128x128x64, FP32 + refinement 910 -> 987 -> 908
// Sorted by LDS, so that the rule sees every pair whichever shape comes first
// (in the batch's order, by points, 64x64x96 comes before 128x128x16: its planes
// were given four times the LDS they need, 188 and 353 us).
inline std::vector<std::vector<int>> plane_launches(const std::vector<PlaneSeg> &segs, int max_seg)
{
    constexpr long HELD = 128, REST = 512;
    std::vector<int> order(segs.size());
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(),
                     [&](int a, int b) { return segs[a].lds > segs[b].lds; });
    long rest = 0, held = 0;
    for (const PlaneSeg &s : segs) rest += s.planes;
    std::vector<std::vector<int>> out;
    for (int i : order) {
        const PlaneSeg &s = segs[i];
        const bool full = !out.empty() && (int)out.back().size() == max_seg;
        const bool small = !out.empty() && 5 * s.lds < 3 * segs[out.back()[0]].lds &&
                           held >= HELD && rest >= REST;
        if (out.empty() || full || small) {
            out.emplace_back();
            held = 0;
        }
        out.back().push_back(i);
        held += s.planes;
        rest -= s.planes;
    }
    return out;
}

}  // namespace pk
