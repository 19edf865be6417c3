// How a call of 3 to 64 tokens splits K over blocks, for the kernel and for the size of its workspace (host code only).
#ifndef FBQ_SPLIT_PLAN_H
#define FBQ_SPLIT_PLAN_H

#include "fbq_internal.h"

namespace fbq {

constexpr int kSplitCus = 256;           // (the workspace is sized without a device)
constexpr int kSplitTapCost = 5;         // a tile of 16 taps in tiles of 16 rows: fp16 against codes of 3 or 4 bits

struct FewSplitRuns { int tap_blocks, taps, row_blocks, units; };        // per segment: blocks for A^T, their tiles of 16 taps, blocks for rows, their units of rows

inline int few_split_unit_rows(int sets) { return sets <= 2 ? 16 : 32; }

// `slots` blocks of one segment, dealt out to A^T and rows so that the longest run is short.
inline FewSplitRuns few_split_runs(int sets, int N, int r, int slots)
{
    const int tap_tiles = ceil_div(r, 16), unit_tiles = few_split_unit_rows(sets) / 16, units = ceil_div(N, 16 * unit_tiles);
    const int even = ceil_div(units * unit_tiles + kSplitTapCost * tap_tiles, slots) / kSplitTapCost;   // tiles of taps a block in an even division
    FewSplitRuns best{0, 0, 1, units};
    int best_cost = 1 << 30;
    for (int taps = std::max(1, std::min(even, tap_tiles)); taps <= std::max(1, std::min(even + 1, tap_tiles)); ++taps) {
        const int tap_blocks = ceil_div(tap_tiles, taps), left = std::max(1, slots - tap_blocks), each = ceil_div(units, left);
        const int cost = std::max(tap_tiles ? taps * kSplitTapCost : 0, each * unit_tiles) + (tap_blocks >= slots ? taps * kSplitTapCost : 0);
        if (cost < best_cost) { best_cost = cost; best = {tap_blocks, tap_tiles ? taps : 0, ceil_div(units, each), each}; }
    }
    return best;
}

// Of the layer and the number of sets alone, so that a layer of a grouped call gets exactly what a call of its own gives it.  As few segments as
// the registers for a segment's activations allow, or one or two more where that divides the work better: the time of a block (its activations at 100
// KB per us, its codes at a CU's part of the memory's rate), and the partial sums, written and read.
inline FewSplit few_split(int sets, int N, int K, int r, int bits)
{
    const int G = K / kGroup, most = sets <= 2 ? 4 : 2, least = ceil_div(G, 8 * most);
    FewSplit best{least, ceil_div(G, 8 * least)};
    double best_us = 1e300;
    for (int segments = least; segments <= least + 2; ++segments) {
        const FewSplit f{segments, ceil_div(G, 8 * segments)};
        if (ceil_div(G, 8 * f.share) != segments) continue;      // (a segment would be empty)
        // A unit half empty costs what a full one does: 2560 -> 28000 INT4, 64 tokens, in three segments with one group a wave 43.0 us, in two with two 33.6; 10240 -> 5120 INT4, 32 tokens,
        // five with two 20.6, four with three 19.7.  (Groups dealt out evenly over segments and waves, up to 16 % fewer to the longest, are no better with three and four sets, and with fewer
        // worse: 8320 -> 8192, 32 tokens, 1.05 of the time of the sets instead of 0.86.)
        if (2 * f.share <= most && segments > least) continue;
        const FewSplitRuns runs = few_split_runs(sets, N, r, std::max(1, kSplitCus / segments));
        const double rounds = ceil_div(segments * (runs.tap_blocks + runs.row_blocks), kSplitCus);
        const double tile_bytes = 16.0 * 8 * f.share * (16.0 * bits + 4);
        const double stream_us = std::max(runs.units * few_split_unit_rows(sets) / 16, kSplitTapCost * runs.taps) * tile_bytes / 21000.0;
        const double x_us = 16.0 * sets * 8 * f.share * 256 / 100000.0;
        const double us = rounds * (stream_us + x_us) + 2.0 * segments * sets * 64.0 * N / 5e6;
        if (us < best_us) { best_us = us; best = f; }
    }
    return best;
}

// Bytes of partial sums.
inline size_t few_split_bytes(const FewSplit &f, int sets, int N, int r) { return (size_t)f.segments * sets * (ceil_div(N, 16) + ceil_div(r, 16)) * 1024; }

}  // namespace fbq

#endif
