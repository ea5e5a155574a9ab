// cb_rules.h -- how a call's work is cut into workgroups: host rules on sizes,
// free of the HIP runtime so that they can be checked on the CPU.
#pragma once
#include <algorithm>
#include <cstdint>

namespace cb {

// Token tiles of the single-layer application, in 32-token sub-blocks: a
// source block's `sub` sub-blocks go to workgroups of the returned count each,
// at most 256 (8192 tokens).  A compute unit holds `resident` workgroups.
// Loading its maps and filling its ring costs a workgroup as much as kFixed
// sub-blocks (4 measured the same or slower); those of one round pay it
// together, so w workgroups per compute unit take about
//     ceil(w / resident) (per + kFixed)
// sub-block times, but no less than the compute unit's share of the memory
// rate allows, w per `rate` (a workgroup alone reaches it at about 10 KB per
// sub-block, source and target rows together).  The cheapest count of tiles is
// taken, among 32 from the fewest on and those that give every compute unit
// one, two, three or four workgroups.
// Measured, 1,024 maps (640 source blocks), tiles of at least 256 tokens and
// about 16 workgroups per compute unit, after a pass that split the maps -> now,
// us: 32 tokens 114 -> 22, 200 135 -> 43, 777 260 -> 114, 3,000 510 -> 355,
// 8,000 962 -> 817; 320 maps of 96 and 128, 777 tokens 70 -> 32.  Few source
// blocks, the same start -> the 32 counts from the fewest on alone -> now, us: one
// of 128 and 128, 32,768 tokens 17.2 -> 26.9 -> 11.4, 131,072 30.8 -> 66.1 -> 20.5;
// four, 131,072 102 -> 68 -> 58; one of 64 and 64, 131,072 15.3 -> 54.6 -> 11.9;
// sixteen (three workgroups per compute unit) 130 -> 151 -> 109.
constexpr int64_t kApplyFixed = 8, kApplyMaxSub = 256;

inline double apply_cost(int64_t sub, int64_t per, int64_t groups, int64_t n_cu, int64_t resident, double rate) {
    const int64_t w = (groups * ((sub + per - 1) / per) + n_cu - 1) / n_cu;
    return std::max((double)((w + resident - 1) / resident * (per + kApplyFixed)), rate * (double)(w * per + kApplyFixed));
}

inline int64_t choose_apply_sub_blocks(int64_t sub, int64_t groups, int64_t n_cu, int64_t resident,
                                       int64_t bytes_per_sub_block) {
    const double rate = std::min(1.0, (double)bytes_per_sub_block / 10240.0);
    const int64_t fewest = (sub + kApplyMaxSub - 1) / kApplyMaxSub;
    int64_t best = std::min(sub, kApplyMaxSub);
    double cost = -1.0;
    auto look = [&](int64_t tiles) {
        const int64_t per = (sub + tiles - 1) / tiles;
        const double c = apply_cost(sub, per, groups, n_cu, resident, rate);
        if (cost >= 0.0 && c >= cost) return;
        cost = c;
        best = per;
    };
    for (int64_t t = fewest; t <= std::min(sub, fewest + 31); ++t) look(t);
    for (int64_t w = 1; w <= 4; ++w) {
        const int64_t t = std::min(sub, w * n_cu / std::max<int64_t>(groups, 1));
        if (t > fewest + 31) look(t);
    }
    return best;
}

}  // namespace cb
