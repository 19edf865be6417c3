// Deals rows of streamed layers out to blocks (plan_stream, csrc/fbq_stream_plan.h): one line on stdout for each line "cus passes slice
// row_bytes N preparing [N preparing ..]" on stdin, "behind in_line rows late_rows early late [early late ..]"; after the plan a walk over the
// blocks as the kernel indexes them, which ends with an error where a row is owned by no block or by two.
#include <cstdio>
#include <cstdlib>
#include <iostream>
#include <sstream>
#include <string>

#include "fbq_stream_plan.h"

using namespace fbq;

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        int cus, passes, slice, row_bytes, N[kMaxSmallGroup], preparing[kMaxSmallGroup], n = 0;
        in >> cus >> passes >> slice >> row_bytes;
        while (n < kMaxSmallGroup && in >> N[n] >> preparing[n]) ++n;
        const int behind = std::max(1, stream_down_bytes(slice) / row_bytes);
        const StreamPlan p = plan_stream(N, preparing, n, behind, passes, cus);
        printf("%d %d %d %d", behind, stream_in_line(N, preparing, n), p.rows, p.late_rows);
        for (int i = 0; i < n; ++i) {
            int next = 0;
            for (int block = 0; block < p.early[i] + p.late[i]; ++block) {
                const int row0 = std::min(block < p.early[i] ? block * p.rows : p.early[i] * p.rows + (block - p.early[i]) * p.late_rows, N[i]);
                const int end = std::min(N[i], row0 + (block < p.early[i] ? p.rows : p.late_rows));
                if (row0 != next || end <= row0) return fprintf(stderr, "%s: layer %d, block %d owns %d..%d, expected from %d\n", line.c_str(), i, block, row0, end, next), 1;
                next = end;
            }
            if (next != N[i]) return fprintf(stderr, "%s: layer %d ends at row %d\n", line.c_str(), i, next), 1;
            printf(" %d %d", p.early[i], p.late[i]);
        }
        printf("\n");
    }
    return 0;
}
