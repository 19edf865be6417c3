// How a launch of the streaming kernel for few tokens deals rows out to blocks (host code only).
#ifndef FBQ_STREAM_PLAN_H
#define FBQ_STREAM_PLAN_H

#include "fbq_internal.h"

namespace fbq {

// Blocks run one per CU, in dispatch order: every layer's preparing blocks first (its down-projection), then rows; a grid row is a
// layer, and the layers' blocks of equal index start one after the other.  The first `early` blocks of a layer's rows find a CU at once and own
// `rows` of them; those that start when preparing blocks are done own `late_rows`, as many less as a CU streams in that time.
struct StreamPlan {
    int rows, late_rows;
    int early[kMaxSmallGroup], late[kMaxSmallGroup];   // blocks with rows, by layer
};

// n layers of N[i] rows with preparing[i] preparing blocks; behind: rows that a CU streams while these run; passes over K.
inline StreamPlan plan_stream(const int *N, const int *preparing, int n, int behind, int passes, int cus)
{
    StreamPlan p{};
    long total = 0;
    int prep = 0;
    for (int i = 0; i < n; ++i) { total += N[i]; prep += preparing[i]; }
    // Row blocks of all layers with the plan's rows and late_rows: early, and late.
    auto deal = [&]() {
        int owners[kMaxSmallGroup];
        for (int i = 0; i < n; ++i) owners[i] = ceil_div(N[i], p.rows);
        int each = cus / n, spare = 0;                      // blocks of every grid row that find a CU at once (as long as it has more); CUs left over
        for (;;) {
            int open = 0;
            spare = cus;
            for (int i = 0; i < n; ++i) {
                spare -= std::min(each, preparing[i] + owners[i]);
                open += preparing[i] + owners[i] > each;
            }
            if (open == 0 || spare < open) break;
            each += spare / open;
        }
        int blocks = 0;
        for (int i = 0; i < n; ++i) {
            p.early[i] = std::max(0, std::min(owners[i], each - preparing[i]));
            if (spare > 0 && preparing[i] + owners[i] > each) {   // the next ones in order
                --spare;
                if (each >= preparing[i]) ++p.early[i];
            }
            p.late[i] = ceil_div(std::max(0, N[i] - p.early[i] * p.rows), p.late_rows);
            blocks += p.early[i] + p.late[i];
        }
        return blocks;
    };
    p.rows = (int)((total + (long)prep * behind + cus - 1) / cus);
    if (prep == 0 || p.rows <= behind) {                    // everything that starts late would find nothing left: nobody does
        const int free_cus = std::max({cus - prep, cus / 2, n});
        for (p.rows = std::max(1, (int)((total + free_cus - 1) / free_cus));; ++p.rows) {
            int blocks = 0;
            for (int i = 0; i < n; ++i) blocks += p.early[i] = ceil_div(N[i], p.rows);
            if (blocks <= free_cus) break;
        }
        p.late_rows = p.rows;
        return p;
    }
    // Every layer rounds up, so the division alone can leave more blocks than CUs.  The ones too many would start when all others end
    // (three sets of 28672 -> 5120, INT4, r = 64: 258 blocks with rows 79.0 us, 256 58.2; of 8192 -> 8192 32.1 / 27.2), and with few rows per late
    // block there are hundreds (of 4096 -> 4593, INT3, r = 64: 195 early blocks of 70 rows and 129 late ones of a single row 17.2, as here 12.5).
    for (;; ++p.rows) {
        p.late_rows = p.rows - behind;
        if (deal() <= cus) break;
    }
    // where the activations are loaded anew for every round of four tiles: no round for a few rows
    const int whole = 64 * ceil_div(p.late_rows, 64);
    if (passes > 1 && p.rows > whole && prep < cus) {
        const StreamPlan kept = p;
        p.rows = whole;
        for (p.late_rows = std::max(1, (int)((total - (long)(cus - prep) * whole + prep - 1) / prep)); p.late_rows <= whole; ++p.late_rows)
            if (deal() <= cus) return p;
        p = kept;
    }
    return p;
}

}  // namespace fbq

#endif
