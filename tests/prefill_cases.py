"""One small layer for every way the prefill launcher cuts a layer into blocks: N, K, r, M and the cut, "<rows of a tile>/<blocks
that split K>" or "<rows>+<rows of the second launch's tiles>", " short" where a block has one K group.  test_prefill_cut.py
keeps the cuts up to date and the list complete, test_gpu_edges.py runs them."""

CUT_CASES = [
    # row counts that are no multiple of eight or of a tile, an odd number of groups (the K groups and shares are then unequal) where
    # there is one, ranks on both sides of a multiple of 16 and of 64
    (777, 128, 8, 65, "64 short"),
    (5001, 640, 72, 131, "64 short"),
    (32783, 128, 0, 65, "96 short"),
    (32783, 768, 40, 67, "96 short"),
    (258, 896, 8, 65, "64"),
    (258, 1920, 40, 66, "64/3"),
    (32814, 896, 0, 67, "96"),
    (4647, 5248, 72, 65, "96/7"),
    (32841, 896, 8, 99, "128"),
    (258, 9344, 200, 1747, "128/8"),
    (32843, 896, 40, 129, "192"),
    (10965, 5760, 0, 137, "192/5"),
    (32843, 896, 64, 195, "256"),
    (11021, 8320, 136, 197, "256/5"),
    (32868, 896, 0, 291, "128+64"),
    (22309, 3328, 8, 530, "128+96"),
    (26577, 896, 24, 515, "192+64"),
    (32845, 896, 0, 411, "192+96"),
    (26323, 1664, 40, 578, "192+128"),
    (32917, 1664, 8, 393, "256+64"),
    (21843, 896, 72, 970, "256+96"),
    (32980, 896, 0, 577, "256+128"),
    (32980, 896, 128, 654, "256+192"),
]
