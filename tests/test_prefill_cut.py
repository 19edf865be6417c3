"""The rule that cuts a prefill layer into blocks, on the CPU: it takes the cases of prefill_cases.py where the GPU tests expect
them, and the cases leave out no kind of cut that calls of ordinary sizes meet."""
import os
import re
import shutil
import subprocess

import pytest

from prefill_cases import CUT_CASES, ORDER_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP runtime's headers")
    exe = str(tmp_path_factory.mktemp("cut") / "cut_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2501_16385_amd", "csrc"), os.path.join(ROOT, "tests", "host", "cut_driver.cpp"), "-o", exe], check=True)
    return exe


def run_driver(exe, given):
    out = subprocess.run([exe], input=given, text=True, capture_output=True, check=True, timeout=120).stdout.split("\n")
    at = out.index("kinds")
    return out[:at], [line.split(" ", 1) for line in out[at + 1:] if line]


@pytest.fixture(scope="module")
def cuts(driver):
    return run_driver(driver, "".join(f"{M} {N} {K} {r}\n" for N, K, r, M, _ in CUT_CASES))


def test_the_cases_are_cut_as_they_say(cuts):
    assert cuts[0] == [cut for *_, cut in CUT_CASES]


def test_every_kind_of_cut_has_a_case(cuts):
    covered = {re.sub("/.*", "/split", cut) for *_, cut in CUT_CASES}
    met = {kind for _, kind in cuts[1]}
    assert met <= covered, met - covered


@pytest.mark.parametrize("M,N,K,r", [(922, 14402, 128, 0), (577, 26880, 256, 64), (1166, 20431, 640, 64), (700, 50257, 1024, 16), (65, 151936, 1024, 64),
                                     (2000, 9000, 1536, 64), (849, 18796, 2304, 0)])
def test_many_short_blocks_share_the_compute_units(driver, M, N, K, r):
    """Several blocks per CU and few steps each: one block per CU took 10 to 30 % longer here."""
    assert run_driver(driver, f"{M} {N} {K} {r}\n")[0][0].endswith(" single")


def test_the_down_projections_are_ordered_as_they_say(driver):
    given = "".join(f"{M} {N} {K} {r}\n" for N, K, r, M, _ in ORDER_CASES)
    out = subprocess.run([driver, "order"], input=given, text=True, capture_output=True, check=True, timeout=120).stdout.split("\n")
    assert [tuple(map(int, line.split())) for line in out if line] == [order for *_, order in ORDER_CASES]


@pytest.mark.parametrize("M,N,K,r", [(256, 1024, 8192, 200), (225, 512, 6144, 256), (289, 1024, 6144, 256), (160, 1024, 8192, 256), (1092, 3456, 13952, 128)])
def test_no_order_by_xcd_where_it_is_slower(driver, M, N, K, r):
    """2 to 6 % of the call's time."""
    out = subprocess.run([driver, "order"], input=f"{M} {N} {K} {r}\n", text=True, capture_output=True, check=True, timeout=120).stdout
    assert out.split()[2] == "0"
