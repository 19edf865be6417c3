// How a launch of the streaming kernel for few tokens deals rows out to blocks (host code only).
#ifndef FBQ_STREAM_PLAN_H
#define FBQ_STREAM_PLAN_H

#include "fbq_internal.h"

namespace fbq {

// Blocks run one per CU, in dispatch order: every layer's preparing blocks first (its down-projection), then rows.  The first `early`
// blocks of a layer's rows find a CU at once and own `rows` of them; those that start when preparing blocks are done own `late_rows`, as many
// less as a CU streams in that time.
//
// Layers that are alike are the columns of a grid: their blocks of equal index start one after the other.  Of layers that are not, the
// narrower ones would leave empty blocks in it, and as blocks go to the XCDs round-robin, a layer's blocks to only four of them (two
// layers) or two (four): an XCD with more blocks than CUs takes twice as long.  So these are in line: all preparing blocks, then the rows' blocks, layer
// after layer, and nothing in between.  That is not done for all, because a block in line learns its layer, and with it the address
// of its parameters, from the kernel's arguments: a second round trip to them.  us, in a grid / in line: {28672, 14336} x 13824, INT3, 16 tokens
// 149 / 84.6; {12000, 11008, 16000, 10240} x 4096, INT4, 4 tokens 40.1 / 25.8; but two of 11008 x 4096, INT3, 8 tokens 16.1 / 16.3, three sets of
// 4096 x 4096 11.2 / 12.0.
struct StreamPlan {
    int rows, late_rows;
    int early[kMaxSmallGroup], late[kMaxSmallGroup];   // blocks with rows, by layer
};

// What a CU would stream in, in bytes at 23 KB per us, while it runs a block of a down-projection over `slice` activations: 5 us, and as a wave
// has an eighth of the slice and asks for 128 activations at once, 1.7 more for every further 1024 of
// a slice.  Two layers of 11008 x 4096 at 8 tokens, by the bytes allowed for: 40000 17.4 us, 70000 15.3, 100000 14.8, 130000 15.6;
// 10240 x 32768, r = 200, slices of 8192: INT4, 8 tokens 60.2 us without the longer slices' time and 54.1 with it, INT3, 16 tokens 65.5 / 58.4
// (slices of 4096, i.e. twice the blocks, 53.7 and 58.2, but two sets of 28672 -> 8192, r = 128, 80.5 instead of 60.7).
inline int stream_down_bytes(int slice) { return 115000 + (slice - 1024) / 1024 * 40000; }
// ... and a block of the other kernel, three tiles of rows up to K = 4096, two beyond.
inline int stream_burst_bytes(int K) { return K <= 4096 ? 60000 + 35 * K : 35000 + ceil_div(K, 4096) * 120000; }

// Whether the layers of a launch are dealt out in line.
inline bool stream_in_line(const int *N, const int *preparing, int n)
{
    for (int i = 1; i < n; ++i)
        if (N[i] != N[0] || preparing[i] != preparing[0]) return true;
    return false;
}

// n layers of N[i] rows with preparing[i] preparing blocks; behind: rows that a CU streams while these run; passes over K.
inline StreamPlan plan_stream(const int *N, const int *preparing, int n, int behind, int passes, int cus)
{
    StreamPlan p{};
    long total = 0;
    int prep = 0;
    for (int i = 0; i < n; ++i) { total += N[i]; prep += preparing[i]; }
    const bool in_line = stream_in_line(N, preparing, n);
    // Row blocks of all layers with the plan's rows and late_rows: early, and late.
    auto deal = [&]() {
        int at_once = std::max(0, cus - prep), blocks = 0;
        for (int i = 0; i < n; ++i) {
            p.early[i] = std::min(in_line ? at_once : std::max(0, cus / n - preparing[i]), ceil_div(N[i], p.rows));
            at_once -= p.early[i];
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
