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
        given = "".join(" ".join(map(str, (CUS, passes, slice_, row_bytes, *(v for layer in layers for v in layer)))) + "\n" for passes, slice_, row_bytes, layers in calls)
        res = subprocess.run([exe], input=given, text=True, capture_output=True, timeout=120)
        assert res.returncode == 0, res.stderr
        return [[int(v) for v in line.split()] for line in res.stdout.split("\n") if line]
    return run


CUS, XCDS = 256, 8

# passes over K, activations of a down-projection's slice, bytes of a row, {rows, preparing blocks} of each layer: three sets of 48 tokens through
# 28672 -> 5120, r = 64, INT4, 4096 -> 4593, r = 64, INT3 and 13824 -> 5120, r = 128, INT3; two grouped 4096 -> 11008; layers of unequal rows and
# ranks; preparing blocks on every CU; one layer; no sub-branch
CALLS = [
    (7, 1792, 15232, [(5120, 68)] * 3), (1, 1024, 1664, [(4593, 20)] * 3), (4, 1792, 5616, [(5120, 72)] * 3), (1, 1024, 1664, [(11008, 20)] * 2),
    (1, 1024, 2176, [(14336, 80), (10240, 5), (28672, 20), (10241, 0)]), (1, 1024, 2176, [(4096, 80)] * 4), (1, 1024, 4352, [(28672, 72)]),
    (2, 1024, 8704, [(10245, 0)]), (4, 1024, 5616, [(28672, 0), (14336, 0)]),
    # small layers along with a large one: they own no rows here, and have more preparing blocks, with 10240 and 8000 rows more than there are CUs
    (1, 1024, 2176, [(0, 106), (11008, 20)]), (1, 1024, 2176, [(0, 190), (0, 190), (10240, 24)]), (1, 1024, 1664, [(0, 22), (0, 22), (10240, 0)]),
]


def check(layers, plan):
    """No more blocks with rows than CUs, on the whole and - blocks go to the XCDs round-robin, in dispatch order - on any XCD."""
    _, in_line, rows, late_rows, *blocks = plan
    blocks = [e + l for e, l in zip(blocks[::2], blocks[1::2])]
    assert sum(blocks) <= CUS and 0 < late_rows <= rows, (layers, plan)
    if in_line:
        first = sum(p for _, p in layers)
        ids = range(first, first + sum(blocks))
    else:
        assert len(set(layers)) == 1
        ids = [(p + b) * len(layers) + i for i, ((_, p), n) in enumerate(zip(layers, blocks)) for b in range(n)]
    assert max(sum(i % XCDS == x for i in ids) for x in range(XCDS)) <= CUS // XCDS, (layers, plan)


def test_no_more_blocks_than_compute_units(plans):
    for (*_, layers), plan in zip(CALLS, plans(CALLS)):
        check(layers, plan)


def test_random_launches(plans):
    rng = random.Random(1)
    calls = []
    for _ in range(20000):
        n = rng.randint(1, 4)
        rows = [round(10240 * 28 ** rng.random()) for _ in range(n)] if rng.random() < 0.5 else [round(10240 / n * 28 ** rng.random())] * n
        preparing = [rng.choice([0, 2, 5, 20, 40, 72, 80]) for _ in range(n)] if rng.random() < 0.3 else [rng.choice([0, 2, 5, 20, 40, 72, 80])] * n
        calls.append((rng.randint(1, 8), 1024 * rng.choice([1, 1, 2, 4, 8]), round(150 * 100 ** rng.random()), list(zip(rows, preparing))))
    for (*_, layers), plan in zip(calls, plans(calls)):
        check(layers, plan)
        # and they are dealt out evenly: nobody owns more than 1.3 times the even share, with those that wait owning `behind` rows less,
        # and a round of four tiles
        total, prep, behind, rows = sum(n for n, _ in layers), sum(p for _, p in layers), plan[0], plan[2]
        even = max((total + prep * behind) / CUS, total / max(CUS - prep, CUS / 2))
        assert rows <= 1.3 * even + 64, (layers, plan, even)


def test_blocks_behind_long_slices_own_fewer_rows(plans):
    """A down-projection over slices of 8192 activations (K = 32768, r = 200) takes more than twice as long as one over 1024."""
    layer = [(10240, 65)]
    short, long = plans([(8, 1024, 17408, layer), (8, 8192, 17408, layer)])
    assert long[0] >= 3 * short[0] and long[2] - long[3] > short[2] - short[3]
