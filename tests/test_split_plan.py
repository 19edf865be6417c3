"""How a call of 3 to 64 tokens splits K and rows over blocks, on the CPU: every group to one wave of one segment, every row and tap to one
block, no empty ones, what a wave holds within its registers, and the partial sums within the bytes asked for."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_every_group_row_and_tap_once(tmp_path):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP runtime's headers")
    exe = str(tmp_path / "split_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16385_amd", "csrc"), os.path.join(ROOT, "tests", "host", "split_driver.cpp"), "-o", exe], check=True)
    rng = random.Random(5)
    calls = [(rng.randint(1, 4), rng.randint(1, 60000), 128 * rng.randint(1, 256), 8 * rng.randint(0, 32), rng.choice([3, 4]), rng.choice([0, 0, 1, 2, 7, 40]))
             for _ in range(20000)]
    res = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in calls), text=True, capture_output=True, timeout=120, check=True)
    lines = res.stdout.split("\n")
    for (sets, N, K, r, bits, slots), line in zip(calls, lines):
        segments, share, tap_blocks, taps, row_blocks, units, size = map(int, line.split())
        G, unit_rows, tap_tiles = K // 128, 16 if sets <= 2 else 32, -(-r // 16)
        where = (sets, N, K, r, bits, slots, line)
        assert 1 <= share <= (4 if sets <= 2 else 2) and (segments - 1) * 8 * share < G <= segments * 8 * share, where
        assert (row_blocks - 1) * units * unit_rows < N <= row_blocks * units * unit_rows, where
        assert (tap_blocks - 1) * taps < tap_tiles <= tap_blocks * taps if r else tap_blocks == 0, where
        assert size == segments * sets * (-(-N // 16) + tap_tiles) * 1024, where
        if slots == 0 and tap_blocks < 256 // segments:
            assert segments * (tap_blocks + row_blocks) <= 256, where
