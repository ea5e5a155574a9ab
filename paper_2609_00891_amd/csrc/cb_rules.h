// cb_rules.h -- how a call's work is cut into workgroups: host rules on sizes,
// free of the HIP runtime so that they can be checked on the CPU.
#pragma once
#include <algorithm>
#include <cstdint>

namespace cb {

// Work units of a call: each item's token tiles (KT tokens of one sequence)
// are cut into n_chunks chunks of chunk_tiles tiles.  Enough (item, chunk)
// units to give every compute unit `per_cu` of them, at most 2048 tiles (64Ki
// tokens) per fp32 partial, and never more chunks than the plan's workspace
// holds (max_chunks <= 0: no such limit).
inline void choose_chunks(int64_t tiles, int n_items, int n_cu, int max_chunks, int *n_chunks, int *chunk_tiles,
                          int per_cu = 8) {
    if (tiles <= 0) {
        *n_chunks = 0;
        *chunk_tiles = 1;
        return;
    }
    const int64_t target_units = (int64_t)per_cu * n_cu;
    int64_t nc = (target_units + n_items - 1) / n_items;
    nc = std::max<int64_t>(nc, (tiles + 2047) / 2048);
    nc = std::min<int64_t>(nc, tiles);
    if (max_chunks > 0) nc = std::min<int64_t>(nc, max_chunks);
    nc = std::max<int64_t>(nc, 1);
    const int64_t ct = (tiles + nc - 1) / nc;
    *chunk_tiles = (int)ct;
    *n_chunks = (int)((tiles + ct - 1) / ct);
}

// Squared rounding error that `tiles` tiles summed in chunks of ct leave in a
// moment of slowly growing sums, in units of the last place of the result: a
// tile adds four products to the chunk's fp32 sum, which grows to ct / tiles of
// the whole, and every chunk is one addition to the whole.
inline double stats_error2(int64_t tiles, int64_t ct) {
    return 4.0 * (double)ct * (double)ct / (3.0 * (double)tiles) + (double)tiles / (3.0 * (double)ct);
}

// The moments' chunks.  One workgroup runs per compute unit, so a call takes
// about ceil(units / compute units) rounds of a chunk's tiles plus a fixed part
// (ring fill and drain, about 5 tiles' time), and every unit's partial is written
// and read again, `unit_tiles` tiles' bytes.  The cheapest count is taken among
// eight units per compute unit and fewer, longer chunks (of at most 2048 tiles)
// whose sums are surely no less precise: stats_error2, which leaves out what else
// rounds, a quarter below.  Many short chunks may grow; long ones may not: 1,024
// maps over 2,048-token sequences keep 4 chunks of 16 tiles a call (G and C of four
// calls 1.2e-7 from 64 bits, 500 us a call; one chunk of 64 left 2.3e-7 and took
// 335, and sums of 16 tiles that a chunk of 64 adds to its partial in memory take
// 500 too: it is the partials' traffic).
// Measured, one call, eight units per compute unit -> this rule, us: 128 maps of
// 128 and 128, 4 x 2,048 tokens 380 -> 181 (32 chunks per item -> 8), about means
// 417 -> 187; 4 maps of 64 and 64, 4 x 256 tokens 40 -> 17 (32 -> 16), about means
// 53 -> 19; two maps of 128 and 128, 65,536 tokens 3,120 -> 116 (2,048 -> 171).
inline void choose_stats_chunks(int64_t tiles, int n_items, int n_cu, int max_chunks, double unit_tiles, int *n_chunks,
                                int *chunk_tiles) {
    choose_chunks(tiles, n_items, n_cu, max_chunks, n_chunks, chunk_tiles);
    const int64_t most = *n_chunks, even = *chunk_tiles;
    const double limit = 0.75 * stats_error2(tiles, even);
    double best = -1.0;
    for (int64_t nc = 1, ct = tiles, next; ct > 0 && nc <= most; nc = next) {
        ct = (tiles + nc - 1) / nc;
        next = ct > 1 ? (tiles + ct - 2) / (ct - 1) : most + 1;     // the first count with shorter chunks
        if (ct != even && (ct > 2048 || stats_error2(tiles, ct) > limit)) continue;
        const int64_t units = nc * n_items;
        const double cost = (double)((units + n_cu - 1) / n_cu) * (double)(ct + 5) + (double)units * unit_tiles / n_cu;
        if (best >= 0.0 && cost >= best) continue;
        best = cost;
        *n_chunks = (int)nc;
        *chunk_tiles = (int)ct;
    }
}

// The most chunks that choose_stats_chunks takes for any call of up to `tiles`
// tiles: at most choose_chunks's, whose count before rounding grows with them.  Calls of many short
// sequences can have more tiles than the plan's tokens fill; they are held to it.
inline int32_t most_stats_chunks(int64_t tiles, int n_items, int n_cu) {
    const int64_t per_cu8 = (8LL * n_cu + n_items - 1) / n_items;
    return (int32_t)std::min(tiles, std::max(per_cu8, (tiles + 2047) / 2048));
}

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
