"""Layers on either side of every line between the ways that 3 to 64 tokens can take: N, K, r, M and the way, "burst" or "stream" (the two few-token kernels), "sets" (sets of 16
side by side), "sets+gemv" (one or two tokens left over go through the GEMV), "split" (K split over blocks) or "gemm".  test_launch_order.py keeps the ways up to date, on the CPU;
test_gpu_edges.py runs the layers."""

# sets of 16, the split or the GEMM
SETS_OR_GEMM_CASES = [
    # the shortest rows that two and four sets take beyond the GEMM's old line and one group of 128 less, which is split, up to 44000 rows
    (40001, 3072, 40, 17, "sets"), (40001, 2944, 40, 17, "split"), (44001, 2944, 40, 17, "gemm"),
    # the longest ones, and one group more
    (20001, 8192, 0, 32, "sets"), (20001, 8320, 0, 32, "split"),
    (8543, 8192, 72, 64, "sets"), (8545, 8320, 72, 64, "split"),
    # either side of 70 million codes at four sets; three sets; a rank above 128
    (17089, 4096, 136, 50, "sets"), (17091, 4096, 136, 50, "split"), (35001, 4096, 136, 50, "gemm"),
    (28673, 8192, 16, 18, "sets"), (28673, 8192, 16, 33, "split"), (46001, 4096, 16, 33, "gemm"),
    # one or two tokens left over as a set, beside two sets, and in rows of several passes
    (5121, 5120, 24, 33, "sets+gemv"), (5121, 5120, 24, 34, "sets"), (2601, 8320, 96, 49, "sets"),
    # the GEMM at the shortest rows, at rows that fill little of two segments, and where a split is one segment
    (40001, 1920, 40, 33, "gemm"), (19001, 2176, 24, 50, "gemm"), (30001, 2048, 136, 64, "gemm"), (25001, 2176, 0, 48, "gemm"),
    # long rows that a first form of the rule split, and four sets of which one has one token
    (2048, 14336, 8, 3, "burst"), (2049, 14464, 0, 8, "burst"), (10239, 16384, 40, 9, "burst"), (3001, 8448, 72, 17, "sets+gemv"), (28001, 2176, 40, 49, "gemm"), (4097, 14336, 96, 49, "split"),
]

SPLIT_CASES = [
    # and the way without room for partial sums.  One to four sets, a token more or less than whole ones; last segments of one group; odd numbers of scales; a row more than whole
    # tiles and units; no sub-branch, ranks on both sides of 16, 32 and 128; the shortest and the longest rows
    (2048, 16512, 8, 3, "burst"), (2049, 16640, 0, 8, "burst"), (4099, 28672, 200, 16, "burst"), (10239, 16512, 40, 9, "burst"),
    (4601, 8448, 72, 17, "sets"), (2100, 14336, 0, 32, "sets"), (5121, 13824, 136, 33, "sets"), (3001, 8448, 8, 48, "sets"), (4097, 14336, 256, 64, "sets"),
    (28673, 2048, 16, 50, "gemm"), (18001, 2176, 40, 49, "gemm"), (30001, 2176, 0, 20, "gemm"), (1025, 32768, 24, 63, "sets"),
]

# further lines of the rule, on the CPU only
ROUTE_CASES = SETS_OR_GEMM_CASES + [(N, K, r, M, "split") for N, K, r, M, _ in SPLIT_CASES] + [
    (2047, 16512, 8, 3, "burst"), (10240, 16512, 8, 3, "stream"), (4096, 16384, 64, 16, "burst"), (4096, 14336, 64, 8, "burst"), (2048, 16512, 8, 2, "gemv"),
    (4599, 8448, 72, 32, "sets"), (4600, 8448, 72, 32, "split"), (3399, 8448, 72, 18, "sets+gemv"), (3400, 8448, 72, 18, "split"), (3400, 8448, 72, 19, "sets"),
    (2304, 12288, 64, 32, "sets"), (2304, 12416, 64, 32, "split"), (1999, 12416, 64, 32, "sets"), (3000, 8320, 8, 48, "sets"), (3100, 8320, 8, 48, "split"),
    (28000, 2560, 64, 48, "split"), (28000, 2560, 64, 64, "gemm"), (26000, 3072, 64, 64, "split"), (26500, 3072, 64, 64, "gemm"), (28672, 8192, 128, 64, "split"),
    (131072, 4096, 64, 64, "gemm"), (131072, 2048, 64, 20, "gemm"), (52000, 20480, 64, 20, "split"), (5120, 13824, 128, 48, "split"), (28672, 8192, 128, 65, "gemm"),
]
