"""CPU-side checks of the C ABI: the library loads, exports what include/fbq.h declares, rejects bad
arguments before any launch, and its host-side fbq_pack writes the documented device layout."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2501_16385_amd as fbq
from oracle import fbq_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "fbq.h")).read()
    declared = sorted(set(re.findall(r"\b(fbq_[a-z_]+)\s*\(", header)))
    assert declared == sorted(fbq.EXPORTED_SYMBOLS)
    lib = fbq.load()
    for name in declared:
        assert getattr(lib, name) is not None


def test_sizes_and_status_strings():
    d = fbq.Desc(4096, 4096, 64, 4)
    assert fbq.packed_bytes(d) == 4096 * 4096 // 2
    assert fbq.packed_bytes(fbq.Desc(4096, 4096, 64, 3)) == 4096 * 4096 * 3 // 8
    assert fbq.workspace_bytes(d, 1) > 0 and fbq.workspace_bytes(fbq.Desc(4096, 4096, 0, 4), 1) == 0
    assert fbq.workspace_bytes(d, 16) >= 16 * 64 * 4
    assert fbq.workspace_bytes(fbq.Desc(4096, 4096, 0, 4), 100) >= 128 * 4096 * 2   # prefill keeps a copy of x
    assert fbq.workspace_bytes(d, 40) == 3 * fbq.workspace_bytes(d, 9)                # 17..64 tokens: the few-token kernel, every 16 tokens with words of their own
    assert fbq.workspace_bytes(d, 64) == 4 * fbq.workspace_bytes(d, 16) and fbq.workspace_bytes(d, 17) == 2 * fbq.workspace_bytes(d, 16)
    assert fbq.workspace_bytes(d, 9) >= 4 * 16 * d.r * 8                               # tagged partial sums of t, one set per K slice
    assert fbq.workspace_bytes(fbq.Desc(4096, 4096, 0, 4), 9) == 0                      # nothing to hand over without a sub-branch
    assert fbq.workspace_bytes(d, 2) == 2 * fbq.workspace_bytes(d, 1)        # one set of tagged words per token
    assert fbq.status_string(0) == "ok"
    assert all(fbq.status_string(c) for c in range(8))


@pytest.mark.parametrize("desc,code", [
    (fbq.Desc(16, 256, 8, 5), 3), (fbq.Desc(16, 256, 8, 4, 64), 3), (fbq.Desc(16, 200, 8, 4), 2),
    (fbq.Desc(0, 256, 8, 4), 2), (fbq.Desc(16, 256, 7, 4), 2), (fbq.Desc(16, 256, 264, 4), 3),
    (fbq.Desc(16, 65536, 8, 4), 3), (fbq.Desc(16, 256, -8, 4), 2)])
def test_bad_descriptors_are_rejected(desc, code):
    lib = fbq.load()
    assert lib.fbq_check_desc(ctypes.byref(desc.c())) == code
    assert fbq.packed_bytes(desc) == 0 and fbq.workspace_bytes(desc, 1) == 0
    # fbq_linear refuses before touching the GPU (bogus but aligned pointers are never dereferenced)
    p = ctypes.c_void_p(0x1000)
    assert lib.fbq_linear(ctypes.byref(desc.c()), 1, p, p, p, p, p, p, p, p, 1 << 20, None) == code


def test_linear_argument_errors_without_launch():
    lib = fbq.load()
    d = fbq.Desc(16, 256, 8, 4)
    ok, odd = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1004)
    call = lambda M, x, ws, wb: lib.fbq_linear(ctypes.byref(d.c()), M, x, ok, ok, ok, ok, ok, ok, ws, wb, None)
    assert call(0, ok, ok, 1 << 20) == 2            # M < 1
    assert call(1, None, ok, 1 << 20) == 1          # null x
    assert call(1, odd, ok, 1 << 20) == 4           # misaligned x
    assert call(1, ok, None, 1 << 20) == 1          # workspace needed but null
    assert call(1, ok, ok, 8) == 5                  # workspace too small
    assert lib.fbq_linear(None, 1, ok, ok, ok, ok, ok, ok, ok, ok, 1 << 20, None) == 1
    # the entry point with the library's own scratch checks the same things, and its token limit, before it touches the GPU
    static = lambda M, x: lib.fbq_linear_static(ctypes.byref(d.c()), M, x, ok, ok, ok, ok, ok, ok, None)
    assert static(0, ok) == 2 and static(17, ok) == 3 and static(1, None) == 1 and static(1, odd) == 4
    assert lib.fbq_linear_static(None, 1, ok, ok, ok, ok, ok, ok, ok, None) == 1
    # the comparator (conventional three-launch sub-branch) validates like fbq_linear and stops at 16 tokens
    unfused = lambda M, x, ws, wb: lib.fbq_linear_unfused(ctypes.byref(d.c()), M, x, ok, ok, ok, ok, ok, ok, ws, wb, None)
    assert unfused(0, ok, ok, 1 << 20) == 2 and unfused(1, None, ok, 1 << 20) == 1 and unfused(1, odd, ok, 1 << 20) == 4
    assert unfused(1, ok, ok, 8) == 5 and unfused(17, ok, ok, 1 << 20) == 3
    assert lib.fbq_unpack_codes(ctypes.byref(d.c()), None, ok, None) == 1
    assert lib.fbq_reconstruct(ctypes.byref(d.c()), ok, ok, ok, None, ok, ok, None) == 1
    assert lib.fbq_quantize_feedback(ctypes.byref(d.c()), ok, ok, ok, odd, ok, ok, None) == 4


def test_group_rejects_overlapping_workspaces_and_the_test_hook_clamps():
    lib = fbq.load()
    d = fbq.Desc(16, 256, 8, 4)
    need = fbq.workspace_bytes(d, 1)
    assert need > 0
    ok = 0x10000
    layer = lambda ws: fbq.fbq._CLayerCall(d.c(), ok, ok, ok, ok, ok, ok, ok, ws, need)
    arr = (fbq.fbq._CLayerCall * 2)(layer(0x20000), layer(0x20000 + need - 16))
    assert lib.fbq_linear_group(arr, 2, 1, None) == 5            # the second workspace starts inside the first
    arr = (fbq.fbq._CLayerCall * 2)(layer(0x20000), layer(0x20000))
    assert lib.fbq_linear_group(arr, 2, 1, None) == 5
    # the poll limit: clamped to the default from above, any negative value means "fall back at once"
    default = lib.fbq_test_set_spin_limit(1 << 30)
    assert default == 1 << 15
    assert lib.fbq_test_set_spin_limit(-7) == 1 << 15            # the huge value was clamped
    assert lib.fbq_test_set_spin_limit(default) == -1
    assert lib.fbq_test_set_spin_limit(default) == default


def test_averages_and_gate_argument_errors_without_launch():
    lib = fbq.load()
    M, d, d2 = 2, fbq.Desc(64, 256, 0, 4), fbq.Desc(32, 256, 0, 4)
    ok, x, y, y2, w, out = 0x10000, 0x20000, 0x30000, 0x40000, 0x50000, 0x60000
    layer = lambda desc, x, y: fbq.fbq._CLayerCall(desc.c(), x, ok, ok, ok, None, None, y, None, 0)

    def call(mix, calls=None, M=M, n=2):
        arr = (fbq.fbq._CLayerCall * 2)(*(calls or [layer(d, x, y), layer(d2, x, y2)]))
        return lib.fbq_linear_group_mix(arr, None if mix is None else (fbq.fbq._CMix * 2)(*[fbq.fbq._CMix(*m) for m in mix]), n, M, None)

    none = (None, None)
    for m in (1, 2, 9, 40, 100):                                 # every kind of kernel behind the call
        if m > 64:
            calls = [fbq.fbq._CLayerCall(dd.c(), x, ok, ok, ok, None, None, yy, wsp, 1 << 28) for dd, yy, wsp in ((d, y, 0x100000000), (d2, y2, 0x200000000))]
        else:
            calls = None
        go = lambda mix: call(mix, calls, m)
        assert go(None) == 1                                     # no mix at all
        assert go([none, (None, out)]) == 1                      # out without with
        assert go([none, (w + 2, out)]) == 4 and go([(w, out + 2), none]) == 4
        size = m * 64 * 2                                        # of the first layer's out, with and y
        assert go([(w, x), none]) == 3                           # out over the activations
        assert go([(w, x + m * 256 * 2 - 16), none]) == 3        # ... over their last sixteen bytes
        assert go([(w, y), none]) == 3                           # out over the layer's own result
        assert go([(w, y2), none]) == 3                          # ... over another layer's
        assert go([(w, y2 - size + 16), none]) == 3
        assert go([(w, w), none]) == 3                           # in place
        assert go([(w, out), (out, 0x70000)]) == 3               # a with that another average writes
        assert go([(w, out), (w, out)]) == 3                     # two averages in one place
        assert go([(y, out), none]) == 3                         # a with that is the layer's own result
        assert go([none, (y + 16, out)]) == 3                    # ... or another layer's
    assert call([none, none], n=0) == 2 and call([none, none], M=0) == 2 and call([none, none], n=65) == 2
    silu = lambda a, b, c, n: lib.fbq_silu_mul(a, b, c, n, None)
    assert silu(None, ok, ok, 8) == 1 and silu(ok, None, ok, 8) == 1 and silu(ok, ok, None, 8) == 1
    assert silu(ok, ok, ok, 0) == 2
    assert silu(ok + 2, ok, ok, 8) == 4 and silu(ok, ok + 8, ok, 8) == 4 and silu(ok, ok, ok + 4, 8) == 4


def test_group_check_takes_time_in_proportion_to_the_layers():
    """Above 64 tokens a workspace size costs a search over tile heights.  The check for overlaps needs each layer's size once,
    not once per pair of layers: 64 layers, refused for their last pair, in the time of a few hundred look-ups, not of 4000."""
    import time
    lib = fbq.load()
    d, M, n, ok = fbq.Desc(4096, 4096, 8, 4), 300, 64, 0x10000
    need = fbq.workspace_bytes(d, M)
    step = (need + 255) // 256 * 256
    ws = [0x10000000 + i * step for i in range(n - 1)]
    arr = (fbq.fbq._CLayerCall * n)(*[fbq.fbq._CLayerCall(d.c(), ok, ok, ok, ok, ok, ok, ok, w, need) for w in ws + ws[-1:]])
    c = d.c()

    def best(fn):
        times = []
        for _ in range(9):
            t = time.perf_counter()
            fn()
            times.append(time.perf_counter() - t)
        return min(times)

    def look_up():
        for _ in range(400):
            lib.fbq_workspace_bytes(ctypes.byref(c), M)

    def group():
        assert lib.fbq_linear_group(arr, n, M, None) == 5

    assert best(group) < best(look_up)


def test_training_argument_errors_without_launch():
    lib = fbq.load()
    d = fbq.Desc(256, 512, 16, 4)
    ok, odd = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1004)
    need = fbq.train_workspace_bytes(d, 100)
    assert need >= 2 * 256 * 512 * 2 and need % 256 == 0
    assert fbq.train_workspace_bytes(fbq.Desc(256, 512, 0, 4), 100) == 0 and fbq.train_workspace_bytes(d, 0) == 0
    assert fbq.train_workspace_bytes(d, 1 << 16) >= 512 * (1 << 16) * 2       # x transposed
    gram = lambda T, X, hs, ws, wb: lib.fbq_gram(ctypes.byref(d.c()), T, X, hs, ok, ws, wb, None)
    assert gram(0, ok, 1.0, ok, need) == 2
    assert gram(100, ok, 0.0, ok, need) == 2         # h_scale must be positive
    assert gram(100, None, 1.0, ok, need) == 1
    assert gram(100, odd, 1.0, ok, need) == 4
    assert gram(100, ok, 1.0, ok, 64) == 5
    step = lambda dd, W, hs, lr, wb: lib.fbq_train_step(ctypes.byref(dd.c()), W, ok, hs, ok, ok, lr, ok, ok, ok, ok, ok, ok, ok, ok,
                                                        ok, wb, None)
    assert step(fbq.Desc(256, 512, 0, 4), ok, 1.0, 0.1, need) == 2      # no branch to train
    assert step(d, ok, 1.0, -1.0, need) == 2
    assert step(d, None, 1.0, 0.1, need) == 1
    assert step(d, odd, 1.0, 0.1, need) == 4
    assert step(d, ok, 1.0, 0.1, 1024) == 5


@pytest.mark.parametrize("bits", [3, 4])
def test_host_pack_writes_the_documented_layout(bits):
    rng = np.random.Generator(np.random.Philox(900 + bits))
    N, K, r = 7, 384, 16
    d = fbq.Desc(N, K, r, bits)
    codes = rng.integers(0, 2 ** bits, (N, K), dtype=np.uint8)
    s = rng.random((N, K // 128)).astype(np.float16)
    z = (rng.random((N, K // 128)) * 8).astype(np.float16)
    A = rng.standard_normal((K, r)).astype(np.float16)
    B = rng.standard_normal((r, N)).astype(np.float16)
    p = fbq.pack(d, codes, s, z, A, B)
    assert np.array_equal(p.qweight, orc.pack(codes, bits))           # same words as the oracle's packer
    assert np.array_equal(orc.unpack(p.qweight, K, bits), codes)      # and the oracle reads them back
    assert np.array_equal(p.scales, s) and np.array_equal(p.zeros, z)
    assert np.array_equal(p.At, A.T) and np.array_equal(p.Bt, B.T)
    bad = codes.copy()
    bad[3, 5] = 2 ** bits
    with pytest.raises(fbq.FbqError) as e:
        fbq.pack(d, bad, s, z, A, B)
    assert e.value.code == 2


def test_loading_the_library_first_still_leaves_one_hip_runtime():
    """The binding hands torch's streams and pointers to the library, so both must sit on the same HIP runtime; torch's
    wheel has a copy of its own.  In a fresh process that touches this package before torch, only one copy may end
    up mapped (with two, every launch on a torch stream failed)."""
    import subprocess
    import sys
    code = (
        "import paper_2501_16385_amd as fbq\n"
        "fbq.load()\n"
        "import torch\n"
        "paths = {line.split()[-1] for line in open('/proc/self/maps') if 'libamdhip64' in line}\n"
        "print(len(paths), sorted(paths))\n"
        "assert len(paths) == 1, paths\n"
    )
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr


def test_native_call_of_linear_hands_over_what_ctypes_would():
    """The compiled call against what fbq_linear is given, with stand-ins for tensors; whatever is not as expected is left to the Python code."""
    from types import SimpleNamespace as NS
    from paper_2501_16385_amd import _fbq_call
    seen = []
    vp = ctypes.c_void_p

    @ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(type(fbq.Desc(1, 1, 0, 4).c())), ctypes.c_int, *[vp] * 8, ctypes.c_size_t, vp)
    def callee(d, M, *rest):
        seen.append(((d[0].N, d[0].K, d[0].r, d[0].bits, d[0].group), M) + rest)
        return 4

    address = ctypes.cast(callee, vp).value
    tensor = lambda p, cuda=True, contiguous=True, shape=(3, 128): NS(is_cuda=cuda, is_contiguous=lambda: contiguous, data_ptr=lambda: p, shape=shape,
                                                                     numel=lambda: 1 << 33, element_size=lambda: 2)
    layer = lambda d=fbq.Desc(8, 128, 16, 3), **more: NS(**{"desc": d, **{n: tensor(0x7F0000000000 + i) for i, n in enumerate(("qweight", "scales", "zeros", "At", "Bt"))}, **more})
    call = lambda l, x=tensor(64), y=tensor(80), ws=tensor(96), stream=1 << 40: _fbq_call.linear(address, l, x, y, ws, stream)
    base = 0x7F0000000000
    assert call(layer()) == 4
    assert seen.pop() == ((8, 128, 16, 3, 128), 3, 64, base, base + 1, base + 2, base + 3, base + 4, 80, 96, 1 << 34, 1 << 40)
    assert call(layer(fbq.Desc(8, 128, 0, 4), At=None, Bt=None), ws=None, stream=0) == 4
    assert seen.pop() == ((8, 128, 0, 4, 128), 3, 64, base, base + 1, base + 2, None, None, 80, None, 0, None)
    for odd in (call(layer(), x=tensor(64, cuda=False)), call(layer(scales=tensor(1, contiguous=False))), call(layer(), y=tensor(2, cuda=False)),
                call(layer(), ws=tensor(2, contiguous=False)), call(layer(At=object())), call(layer(fbq.Desc(-8, 128, 0, 4))), call(layer(fbq.Desc(8.0, 128, 0, 4))),
                call(layer(), x=tensor(64, shape=())), call(layer(), x=tensor(64, shape=(2.5,))), call(layer(), stream=None), call(NS())):
        assert odd is None and not seen
    def fails(e):
        def method():
            raise e
        return method
    assert call(layer(), y=NS(is_cuda=True, is_contiguous=lambda: True, data_ptr=fails(RuntimeError("meta tensor")))) is None
    for e in (KeyboardInterrupt, SystemExit):           # not dropped on the way to the Python code
        with pytest.raises(e):
            call(layer(), y=NS(is_cuda=True, is_contiguous=lambda: True, data_ptr=fails(e())))
    assert not seen
    with pytest.raises(TypeError):
        _fbq_call.linear(address)


def test_linear_refuses_host_tensors_as_before():
    import torch
    layer = fbq.DeviceLayer(fbq.Desc(128, 128, 0, 4), torch.zeros(128, 16, dtype=torch.int32), *[torch.zeros(128, 1, dtype=torch.int16)] * 2, None, None)
    with pytest.raises(ValueError, match="device tensor"):
        fbq.linear(layer, torch.zeros(1, 128).half(), torch.zeros(1, 128).half(), torch.zeros(64, dtype=torch.uint8), stream=type("S", (), {"cuda_stream": 0}))


def test_scratch_of_a_call_is_zero_where_hand_over_words_lie_and_nowhere_else_filled(monkeypatch):
    """Calls without a workspace of their own: partial sums are megabytes that nobody reads before they are written."""
    import torch
    from paper_2501_16385_amd import fbq as binding
    monkeypatch.setattr(torch, "empty", lambda n, **k: torch.full((n,), 0xAB, **k))
    for N, K, r, M in [(8192, 28672, 64, 16), (8192, 28672, 0, 16), (131072, 4096, 64, 40), (5120, 13824, 128, 48), (131072, 4096, 64, 64), (4096, 4096, 64, 16), (4096, 4096, 8, 40),
                       (4096, 4096, 64, 2), (4096, 4096, 0, 2), (4096, 4096, 64, 65)]:
        d = fbq.Desc(N, K, r, 4)
        ws, need, words = binding._scratch(d, M, "cpu"), fbq.workspace_bytes(d, M), 4 * 17 * 16 * r * 8
        assert (ws is None) == (need == 0), (N, K, r, M)
        if ws is None:
            continue
        zeros = need if M <= 2 or M > 64 else min(need, words)
        assert ws.numel() == need and int(ws[:zeros].count_nonzero()) == 0 and bool((ws[zeros:] == 0xAB).all()), (N, K, r, M)
