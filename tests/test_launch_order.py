"""What a call launches, and what it leaves behind when one of its launches fails, on the CPU: the process's kernel launches go to a recorder
(tests/host/launch_recorder.cpp) that lets the n-th one fail, and nothing runs."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

CHILD = r"""
import ctypes, json, sys
sys.path[:0] = [sys.argv[1], sys.argv[1] + "/tests"]
import paper_2501_16385_amd as fbq
from test_kernel_resources import code_objects
lib = fbq.load()
sizes = {k[".name"]: [a[".size"] for a in k[".args"] if not a[".value_kind"].startswith("hidden")] for k in code_objects()}
launched, fail_at = [], [0]

@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def on_launch(name, args):
    name = name.decode()
    launched.append((name, [ctypes.string_at(args[i], n) for i, n in enumerate(sizes[name])]))
    return len(launched) == fail_at[0]

ctypes.CDLL(None).recorder_set_callback(on_launch)
AT, BT = 0x7A1100000000, 0x7B2200000000          # addresses of the masters: never dereferenced, looked for in the arguments
out = []
for N, K, r, loss in [(700, 1152, 64, 1), (700, 1152, 64, 0), (128, 128, 8, 1), (40000, 256, 256, 0), (40000, 256, 256, 1)]:
    d = fbq.Desc(N, K, r, 4)
    p = lambda i: 0x100000000 * (i + 1)
    def step():
        launched.clear()
        return lib.fbq_train_step(ctypes.byref(d.c()), p(0), p(1), 1.0, AT, BT, 0.1, *(p(i) for i in range(2, 9)), p(9) if loss else None,
                                  p(10), fbq.train_workspace_bytes(d, 1), None)
    fail_at[0] = 0
    assert step() == 0
    whole = list(launched)
    for n in range(1, len(whole) + 1):
        fail_at[0] = n
        assert step() == 6, "a failed launch is reported"
        assert len(launched) == n, "nothing is launched behind a failed launch"
    has = lambda args, v: any(v.to_bytes(8, "little") in a for a in args)
    out.append([[name, has(args, AT), has(args, BT)] for name, args in whole])
print("RESULT " + json.dumps(out))
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP runtime's headers")
    so = str(tmp_path_factory.mktemp("recorder") / "recorder.so")
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "host", "launch_recorder.cpp"), "-o", so, "-ldl"], check=True)
    return so


def test_train_step_moves_both_masters_in_its_last_launch(recorder):
    """A step that reports an error has moved neither master, so it can be made again.  The first launch reads both (it casts
    them to fp16); of the others only the last may know them."""
    import json
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))   # (in front of what is preloaded already)
    res = subprocess.run([sys.executable, "-c", CHILD, ROOT], env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    steps = json.loads(res.stdout.split("RESULT ")[1])
    for launches in steps:
        assert "cast_masters" in launches[0][0] and launches[0][1:] == [True, True]
        assert launches[-1][1:] == [True, True], launches
        assert all(l[1:] == [False, False] for l in launches[1:-1]), launches


GROUP_CHILD = r"""
import ctypes, json, sys
sys.path[:0] = [sys.argv[1]]
import paper_2501_16385_amd as fbq
lib = fbq.load()
launched = []

@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def on_launch(name, args):
    launched.append(name.decode())
    return 0

ctypes.CDLL(None).recorder_set_callback(on_launch)
out = []
for K, r, M, rows in json.loads(sys.argv[2]):
    calls = [fbq.Desc(N, K, r, 4) for N in rows]
    p = lambda i, j: 0x100000000 * (10 * i + j + 2)
    arr = (fbq.fbq._CLayerCall * len(calls))(*(fbq.fbq._CLayerCall(d.c(), 0x100000000, p(i, 0), p(i, 1), p(i, 2), p(i, 3), p(i, 4), p(i, 5), p(i, 6), 1 << 30)
                                               for i, d in enumerate(calls)))
    launched.clear()
    assert lib.fbq_linear_group(arr, len(calls), M, None) == 0
    out.append(list(launched))
print("RESULT " + json.dumps(out))
"""


def test_grouped_layers_share_a_launch(recorder):
    """3 to 16 tokens: one launch for layers of one K on the same activations, also for a few small ones beside a large one (two launches cost 2 to 4 us
    more); two where that is slower; never one for the large ones on their own account."""
    import json
    one = [(4096, 64, 16, [11008, 4096]), (4096, 0, 8, [1024, 10240, 1000]), (12288, 64, 4, [12288, 1024, 1024]), (4096, 64, 16, [4096, 4096, 4096]),
           (4096, 64, 5, [11008, 11008]), (8192, 8, 3, [10240, 20000, 30000, 10241]), (14336, 0, 8, [13000, 1000])]
    two = [(1024, 64, 16, [40000, 1024]), (16384, 64, 16, [16384, 1024]), (8192, 64, 16, [10240, 8192]), (14336, 64, 8, [13000, 1000])]
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))
    res = subprocess.run([sys.executable, "-c", GROUP_CHILD, ROOT, json.dumps(one + two)], env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    launches = json.loads(res.stdout.split("RESULT ")[1])
    for call, names in zip(one + two, launches):
        assert len(names) == (1 if call in one else 2), (call, names)
        assert any("few_stream" in n for n in names) == any(N >= 10240 for N in call[3]), (call, names)


SPLIT_CHILD = r"""
import ctypes, json, sys
sys.path[:0] = [sys.argv[1]]
import paper_2501_16385_amd as fbq
lib = fbq.load()
launched = []

@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def on_launch(name, args):
    launched.append(name.decode())
    return 0

ctypes.CDLL(None).recorder_set_callback(on_launch)
out = []
for M, layers in json.loads(sys.argv[2]):
    p = lambda i, j: 0x100000000 * (10 * i + j + 2)
    arr = (fbq.fbq._CLayerCall * len(layers))(*(fbq.fbq._CLayerCall(fbq.Desc(N, K, r, bits).c(), 0x100000000, p(i, 0), p(i, 1), p(i, 2), p(i, 3), p(i, 4), p(i, 5), at, size)
                                                for i, (N, K, r, bits, at, size) in enumerate(layers)))
    launched.clear()
    rc = lib.fbq_linear_group(arr, len(layers), M, None)
    out.append([rc, [sum(k in n for n in launched) for k in ("few_split_kernel", "few_join_kernel", "small_m", "few_stream", "fbq_gemm_kernel", "fbq_gemv_kernel")], len(launched)])
print("RESULT " + json.dumps(out))
"""


def test_room_for_partial_sums_that_meets_another_workspace_is_not_used(recorder):
    """Workspaces may not overlap in what the layers cannot do without, as ever; where only the room for partial sums would, those layers go unsplit."""
    import json
    BIG, AT = 1 << 30, 0x9000000000
    words = lambda r: 17 * 16 * r * 8
    split, plain = [1, 1, 0, 0], [0, 0, 1, 0]     # few_split, few_join, small_m, few_stream
    cases = [
        # one scratch for two layers that need none; the same for three sets; hand-over areas one behind the other, each with the rest of the arena as its size
        (16, [(8192, 28672, 0, 4, AT, BIG)] * 2, 0, plain), (48, [(5120, 13824, 0, 3, AT, BIG)] * 2, 0, None),
        (8, [(4096, 28672, 64, 4, AT, BIG), (8192, 28672, 64, 4, AT + words(64), BIG - words(64))], 0, plain),
        # a third layer elsewhere keeps its split; a small layer's words inside a split layer's room; one that needs nothing does not count
        (8, [(4096, 28672, 64, 4, AT, BIG), (8192, 28672, 64, 4, AT + words(64), BIG), (2048, 28672, 64, 4, 2 * AT, BIG)], 0, [1, 1, 1, 0]),
        (8, [(4096, 28672, 64, 4, AT, BIG), (1024, 28672, 64, 4, AT + (1 << 20), words(64))], 0, [0, 0, 1, 0]),
        (8, [(4096, 28672, 0, 4, AT, BIG), (1024, 28672, 0, 4, AT, BIG)], 0, [1, 1, 1, 0]),
        # apart: both split, in one launch
        (16, [(8192, 28672, 0, 4, AT, BIG), (8192, 28672, 0, 4, 2 * AT, BIG)], 0, split),
        # and what never went: the same hand-over words, or words that begin inside another layer's
        (16, [(8192, 28672, 64, 4, AT, BIG)] * 2, 5, [0, 0, 0, 0]), (8, [(4096, 28672, 64, 4, AT, BIG), (4096, 28672, 64, 4, AT + words(64) - 16, BIG)], 5, [0, 0, 0, 0]),
    ]
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))
    res = subprocess.run([sys.executable, "-c", SPLIT_CHILD, ROOT, json.dumps([c[:2] for c in cases])], env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    for (M, layers, want_rc, want), (rc, kinds, count) in zip(cases, json.loads(res.stdout.split("RESULT ")[1])):
        assert rc == want_rc, (M, layers, rc)
        assert kinds[:4] == want if want is not None else kinds[0] == 0 and count > 0, (M, layers, kinds)


def test_a_workspace_with_room_for_the_partial_sums_is_used(recorder):
    """What is asked for is what the split kernel writes - hand-over words of four sets, and K segments x 16 tokens a set x rows and taps in fp32 - or what the call needs
    unsplit, if that is more; a byte less is accepted, and goes unsplit."""
    import json
    import paper_2501_16385_amd as fbq
    cases, AT = [], 0x9000000000
    for N, K, r, bits, M, segments in [(8192, 28672, 128, 4, 16, 7), (4096, 28672, 64, 3, 3, 7), (5120, 13824, 128, 3, 48, 7), (2100, 17408, 0, 4, 9, 6)]:
        need = 4 * 17 * 16 * r * 8 + segments * -(-M // 16) * (-(-N // 16) + -(-r // 16)) * 1024
        assert fbq.workspace_bytes(fbq.Desc(N, K, r, bits), M) == need, (N, K, r, bits, M, fbq.workspace_bytes(fbq.Desc(N, K, r, bits), M))
        cases += [(M, [(N, K, r, bits, AT, need)]), (M, [(N, K, r, bits, AT, need - 1)])]
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))
    res = subprocess.run([sys.executable, "-c", SPLIT_CHILD, ROOT, json.dumps(cases)], env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    for i, (rc, kinds, _) in enumerate(json.loads(res.stdout.split("RESULT ")[1])):
        assert rc == 0 and kinds[0] == kinds[1] == (1 - i % 2), (cases[i], rc, kinds)


def test_which_way_a_call_of_few_tokens_takes(recorder):
    import json
    from few_cases import ROUTE_CASES
    AT = 0x9000000000
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))
    for bits in (3, 4):
        calls = [(M, [(N, K, r, bits, AT, 1 << 32)]) for N, K, r, M, _ in ROUTE_CASES]
        res = subprocess.run([sys.executable, "-c", SPLIT_CHILD, ROOT, json.dumps(calls)], env=env, capture_output=True, text=True, timeout=300)
        assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
        for (N, K, r, M, way), (rc, (split, join, small, stream, gemm, gemv), _) in zip(ROUTE_CASES, json.loads(res.stdout.split("RESULT ")[1])):
            few = small + stream
            got = ("split" if split == join == 1 and not few + gemm + gemv else "gemm" if gemm and not few + split + gemv else "gemv" if gemv and not few else
                   "sets" + ("+gemv" if gemv else "") if few == 1 and M > 16 else "stream" if stream else "burst" if small else "?")
            assert rc == 0 and got == way, (N, K, r, M, bits, way, got, rc)


QUANT_CHILD = r"""
import ctypes, json, re, sys
sys.path[:0] = [sys.argv[1]]
import paper_2501_16385_amd as fbq
lib = fbq.load()
launched = []

@ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_char_p, ctypes.POINTER(ctypes.c_void_p))
def on_launch(name, args):
    launched.append(name.decode())
    return 0

ctypes.CDLL(None).recorder_set_callback(on_launch)
p = lambda i: 0x100000000 * (i + 1)
out = []
for step, N, K, r in json.loads(sys.argv[2]):
    d = fbq.Desc(N, K, r, 4)
    launched.clear()
    if step:
        assert lib.fbq_train_step(ctypes.byref(d.c()), p(0), p(1), 1.0, p(2), p(3), 0.0, *(p(i) for i in range(4, 11)), None, p(11), fbq.train_workspace_bytes(d, 1), None) == 0
    else:
        assert lib.fbq_quantize_feedback(ctypes.byref(d.c()), p(0), p(1), p(2), p(3), p(4), p(5), None) == 0
    out += [list(map(int, re.search(r"fbq_quantize_kernelILi4ELb(\d)ELi(\d)ELi(\d)ELb(\d)", n).groups())) for n in launched if "fbq_quantize_kernel" in n]
print("RESULT " + json.dumps(out))
"""


def test_which_instance_of_the_quantizer_a_layer_takes(recorder):
    """With Delta_F, steps of 32 taps, waves a block, in fp64 throughout: a block a CU or less; by rank; eight waves above rank 128 where they fill the GPU, and with Delta_F not
    where they go round once and a little."""
    import json
    want = {(1, 1000, 1024, 64): [1, 2, 4, 1], (1, 2048, 1024, 128): [1, 4, 4, 1], (1, 2049, 1024, 64): [1, 2, 4, 0], (1, 2049, 1024, 72): [1, 4, 4, 0], (1, 1000, 1024, 200): [1, 8, 4, 1],
            (1, 2048, 2048, 200): [1, 8, 8, 0], (1, 2049, 2048, 200): [1, 8, 4, 0], (1, 5000, 1024, 200): [1, 8, 4, 0], (1, 2816, 2048, 200): [1, 8, 8, 0], (1, 1920, 2048, 200): [1, 8, 4, 0],
            (0, 1000, 1024, 64): [0, 2, 4, 0], (0, 5000, 1024, 200): [0, 8, 8, 0], (0, 1000, 1024, 200): [0, 8, 4, 0], (0, 1000, 1024, 0): [0, 2, 4, 0]}
    env = dict(os.environ, LD_PRELOAD=" ".join([recorder] + os.environ.get("LD_PRELOAD", "").split()))
    res = subprocess.run([sys.executable, "-c", QUANT_CHILD, ROOT, json.dumps(list(want))], env=env, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert json.loads(res.stdout.split("RESULT ")[1]) == list(want.values())
