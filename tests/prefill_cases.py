"""One small layer for every way the prefill launcher cuts a layer into blocks: N, K, r, M and the cut, "<rows of a tile>/<blocks
that split K>" or "<rows>+<rows of the second launch's tiles>", " single" where low tiles have one K group.  test_prefill_cut.py
keeps the cuts up to date and the list complete, test_gpu_edges.py runs them."""

CUT_CASES = [
    # row counts that are no multiple of eight or of a tile, an odd number of groups (the K groups and shares are then unequal) where
    # there is one, ranks on both sides of a multiple of 16 and of 64
    (777, 128, 8, 65, "64 single"),
    (5001, 640, 72, 131, "64 single"),
    (32971, 128, 0, 65, "96 single"),
    (33011, 896, 40, 67, "96 single"),
    (18797, 2304, 0, 849, "96 single"),
    (32771, 384, 8, 97, "128 single"),
    (8001, 1152, 200, 1001, "128 single"),
    (258, 896, 8, 65, "64"),
    (258, 1920, 40, 66, "64/3"),
    (32358, 2176, 0, 66, "96"),
    (6407, 3200, 72, 65, "96/5"),
    (33229, 1664, 8, 97, "128"),
    (259, 9344, 200, 1747, "128/8"),
    (33316, 2176, 40, 130, "192"),
    (11074, 5760, 0, 131, "192/5"),
    (32930, 2176, 64, 198, "256"),
    (10762, 8320, 136, 194, "256/5"),
    (33363, 2176, 16, 297, "128+64"),
    (22143, 3328, 8, 521, "128+96"),
    (21962, 2176, 24, 521, "192+64"),
    (18735, 2176, 8, 773, "192+96"),
    (26526, 2176, 40, 577, "192+128"),
    (33213, 2688, 0, 483, "256+64"),
    (39603, 2688, 72, 463, "256+96"),
    (33355, 2176, 72, 581, "256+128"),
    (32821, 1664, 128, 683, "256+192"),
]

# The order of the down-projection's blocks: N, K, r, M, and the token tiles, K slices and slices dealt out to the XCDs whole.  A ragged last tile,
# more tiles than XCDs and a number of slices that is no multiple of eight wherever slices are; either side of the lines of narrow layers
ORDER_CASES = [
    (300, 20480, 200, 290, (10, 23, 16)),
    (301, 16384, 200, 333, (11, 22, 16)),
    (2049, 13824, 128, 333, (11, 22, 16)),
    (2050, 8320, 200, 289, (10, 22, 16)),
    (300, 28672, 128, 230, (8, 32, 32)),
    (1600, 8320, 200, 289, (10, 22, 0)),
    (300, 13824, 128, 290, (10, 22, 0)),
]
