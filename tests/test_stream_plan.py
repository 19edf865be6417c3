"""How a launch of the streaming kernel deals rows out to blocks, on the CPU: every row to one block, and no more blocks with rows
than there are CUs - one block too many starts when all others end."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP runtime's headers")
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16385_amd", "csrc"), os.path.join(ROOT, "tests", "host", "plan_driver.cpp"), "-o", exe], check=True)

    def run(calls):
        given = "".join(" ".join(map(str, (cus, passes, behind, *(v for layer in layers for v in layer)))) + "\n" for cus, passes, behind, layers in calls)
        res = subprocess.run([exe], input=given, text=True, capture_output=True, timeout=120)
        assert res.returncode == 0, res.stderr
        return [[int(v) for v in line.split()] for line in res.stdout.split("\n") if line]
    return run


# cus, passes, behind, {rows, preparing blocks} of each layer: three sets of 48 tokens through 28672 -> 5120, r = 64, INT4 and 4096 -> 4593 INT3;
# 13824 -> 5120, r = 128, INT3; two grouped 4096 -> 11008; layers of unequal rows and ranks; preparing blocks on every CU; one layer; no sub-branch
CALLS = [
    (256, 7, 7, [(5120, 68)] * 3), (256, 1, 69, [(4593, 20)] * 3), (256, 4, 20, [(5120, 72)] * 3), (256, 1, 69, [(11008, 20)] * 2),
    (256, 1, 52, [(14336, 80), (10240, 5), (28672, 20), (10241, 0)]), (256, 1, 40, [(4096, 80)] * 4), (256, 1, 26, [(28672, 72)]), (256, 2, 18, [(10245, 0)]),
]


def test_no_more_blocks_than_compute_units(plans):
    for (cus, _, _, layers), (rows, late_rows, *blocks) in zip(CALLS, plans(CALLS)):
        assert sum(blocks) <= cus and 0 < late_rows <= rows, (layers, rows, late_rows, blocks)


def test_random_launches(plans):
    rng = random.Random(1)
    calls = []
    for _ in range(20000):
        n = rng.randint(1, 4)
        rows = [round(10240 * 28 ** rng.random()) for _ in range(n)] if rng.random() < 0.5 else [round(10240 / n * 28 ** rng.random())] * n
        preparing = [rng.choice([0, 2, 5, 20, 40, 72, 80]) for _ in range(n)] if rng.random() < 0.3 else [rng.choice([0, 2, 5, 20, 40, 72, 80])] * n
        calls.append((256, rng.randint(1, 8), round(2 * 400 ** rng.random()), list(zip(rows, preparing))))
    for (cus, _, behind, layers), (rows, late_rows, *blocks) in zip(calls, plans(calls)):
        assert sum(blocks) <= cus and 0 < late_rows <= rows, (behind, layers, rows, late_rows, blocks)
        # and they are dealt out evenly: nobody owns more than 1.3 times the even share, with those that wait owning `behind` rows less,
        # and a round of four tiles
        total, prep = sum(n for n, _ in layers), sum(p for _, p in layers)
        even = max((total + prep * behind) / cus, total / max(cus - prep, cus / 2))
        assert rows <= 1.3 * even + 64, (behind, layers, rows, even)
