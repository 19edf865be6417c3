// How K and rows of a call are split over blocks (csrc/fbq_split_plan.h): one line on stdout for each line "sets N K r bits slots" on stdin,
// "segments share tap_blocks taps row_blocks units bytes".
#include <cstdio>
#include <iostream>

#include "fbq_split_plan.h"

int main()
{
    int sets, N, K, r, bits, slots;
    while (std::cin >> sets >> N >> K >> r >> bits >> slots) {
        const fbq::FewSplit f = fbq::few_split(sets, N, K, r, bits);
        const fbq::FewSplitRuns u = fbq::few_split_runs(sets, N, r, slots > 0 ? slots : std::max(1, fbq::kSplitCus / f.segments));
        printf("%d %d %d %d %d %d %zu\n", f.segments, f.share, u.tap_blocks, u.taps, u.row_blocks, u.units, fbq::few_split_bytes(f, sets, N, r));
    }
    return 0;
}
