"""The rule that cuts a prefill layer into blocks, on the CPU: it takes the cases of prefill_cases.py where the GPU tests expect
them, and the cases leave out no kind of cut that calls of ordinary sizes meet."""
import os
import shutil
import subprocess

import pytest

from prefill_cases import CUT_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def cuts(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP runtime's headers")
    exe = str(tmp_path_factory.mktemp("cut") / "cut_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16385_amd", "csrc"), os.path.join(ROOT, "tests", "host", "cut_driver.cpp"), "-o", exe], check=True)
    given = "".join(f"{M} {N} {K}\n" for N, K, _, M, _ in CUT_CASES)
    out = subprocess.run([exe], input=given, text=True, capture_output=True, check=True, timeout=120).stdout.split("\n")
    at = out.index("kinds")
    return out[:at], [line.split(" ", 1) for line in out[at + 1:] if line]


def test_the_cases_are_cut_as_they_say(cuts):
    assert cuts[0] == [cut for *_, cut in CUT_CASES]


def test_every_kind_of_cut_has_a_case(cuts):
    covered = {cut.split("/")[0] + ("/split" if "/" in cut else "") for *_, cut in CUT_CASES}
    met = {kind for _, kind in cuts[1]}
    assert met <= covered, met - covered


def test_short_k_has_low_tiles_of_one_k_group(cuts):
    """Up to six quantization groups a block is mostly start and end; with one block per CU, nothing ran meanwhile."""
    short = [cut for (_, K, _, _, _), cut in zip(CUT_CASES, cuts[0]) if K <= 768]
    assert len(short) >= 4 and set(short) == {"64 short", "96 short"}
