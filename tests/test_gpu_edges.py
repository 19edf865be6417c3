"""GPU kernels at the sizes where their tiles end: remainders, the smallest and the largest of a range, and the sizes on
either side of a dispatch rule, against the fp64 oracle.  Every array sits inside a buffer of NaN patterns, so that a value
taken from beyond an array shows in the result."""
import numpy as np
import pytest

import fbq_synth
from helpers import assert_matches_oracle, framed_in_nan, framed_layer, gpu_y, make_oracle_layer
from few_cases import SETS_OR_GEMM_CASES, SPLIT_CASES
from oracle import fbq_oracle as orc
from prefill_cases import CUT_CASES, ORDER_CASES

pytestmark = pytest.mark.gpu


def t16(a):
    import torch
    return None if a is None else framed_in_nan(torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda())


# ------------------------------------------------------------------ feedback quantizer: blocks of 64 rows, 16 per wave, taps in tiles of 32

@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r", [(1, 128, 8), (15, 128, 0), (17, 256, 40), (63, 384, 24), (65, 128, 200), (130, 1280, 256), (64, 256, 32)])
def test_quantizer_tile_edges(bits, N, K, r):
    """Codes, scales and zeros are defined in 64 bits; these sums need fewer than 53 bits, so every word must agree."""
    import torch
    import paper_2501_16385_amd as fbq
    L = make_oracle_layer(fbq_synth.LayerSpec("edge", N, K, r, bits), config=41)
    dev = fbq.quantize_feedback(fbq.Desc(N, K, r, bits), t16(L.W), t16(L.A.T) if r else None, t16(L.B.T) if r else None)
    torch.cuda.synchronize()
    assert np.array_equal(dev.scales.cpu().numpy().view(np.float16), L.scales)
    assert np.array_equal(dev.zeros.cpu().numpy().view(np.float16), L.zeros)
    assert np.array_equal(dev.qweight.cpu().numpy().view(np.uint32), L.words)


@pytest.mark.parametrize("bits,N,K,r,kind", [
    (4, 33, 256, 0, "ties"), (3, 33, 256, 8, "ties"), (4, 64, 128, 64, "large branch"), (3, 50, 128, 256, "large branch"), (4, 40, 256, 40, "offset"),
    (3, 40, 256, 16, "subnormal"), (4, 40, 256, 136, "subnormal"), (3, 40, 384, 24, "few values"), (4, 20, 256, 8, "zero branch"),
    (3, 513, 32768, 8, "plain"), (4, 129, 32768, 136, "plain"), (3, 641, 32768, 200, "plain")])
def test_quantizer_where_32_bits_leave_rows_open(bits, N, K, r, kind):
    """Rows whose scale, zero or codes lie on, or within fp32's reach of, a rounding boundary go through fp64; the last three sizes have two
    row tiles a block and blocks of eight waves.  Every word as in 64 bits: sums of dyadic numbers, or of values of one size, need fewer than 53 bits."""
    import torch
    import paper_2501_16385_amd as fbq
    rng = np.random.Generator(np.random.Philox(61 + r + bits))
    W = rng.standard_normal((N, K)) * 0.02
    A, B = rng.standard_normal((K, max(r, 1))) * 0.01, rng.standard_normal((max(r, 1), N)) * 0.01
    if kind == "ties":                                  # scale 1 (or 1/2), zero 0: half the values lie half-way between two codes
        W = rng.integers(0, 2 * (2 ** bits - 1) + 1, (N, K)) / 2.0
        W[:, ::128], W[:, 1::128] = 0.0, 2 ** bits - 1.0
        W[::2] /= 2
        A, B = np.where(np.arange(K)[:, None] % 128 < 2, 0.0, np.round(A * 400) / 16), np.round(B * 400) / 16
    elif kind == "large branch":
        A, B = A * 1000, B * 1000
    elif kind == "offset":
        W += rng.choice([0.5, 3.0, 40.0, -500.0], (N, 1))
    elif kind == "subnormal":
        W, A, B = W * 1e-4, A * np.where(rng.random((K, r)) < 0.5, 1e-4, 1.0), B * np.where(rng.random((r, N)) < 0.5, 1e-4, 1.0)
    elif kind == "few values":
        W = rng.choice([-0.25, 0.25, 0.125, 0.0], (N, K))
    elif kind == "zero branch":
        B *= 0
    W, A, B = (a.astype(np.float16) for a in (W, A, B))
    dev = fbq.quantize_feedback(fbq.Desc(N, K, r, bits), t16(W), t16(A.T) if r else None, t16(B.T) if r else None)
    codes = fbq.unpack_codes(dev).cpu().numpy()
    rows = np.arange(N) if N * K <= 1 << 20 else np.unique(np.r_[0:17, 63:66, 127:130, N - 2:N, rng.integers(0, N, 12)] % N)
    Bs = np.ascontiguousarray(B[:, rows])
    want, s, z = orc.quantize(np.ascontiguousarray(W[rows]), A if r else None, Bs if r else None, bits, 128)
    assert np.array_equal(dev.scales.cpu().numpy().view(np.uint16)[rows], s.view(np.uint16))
    got_z = dev.zeros.cpu().numpy().view(np.float16)[rows]
    assert np.array_equal(got_z, z)
    assert np.array_equal(codes[rows], want)


def quantize_in_64_bits(W, A, B, bits):
    """Scales, zeros and codes of W - B A as include/fbq.h defines them, on the GPU in fp64; s and z as fp16 numbers, rounded once."""
    import torch

    def half_once(d):                                   # by way of an fp32 number rounded to odd
        f = d.float()
        u = f.view(torch.int32)
        u = torch.where(f.double().abs() > d.abs(), u - 1, u)
        return torch.where(f.double() != d, u | 1, u).view(torch.float32).half()
    N, K = W.shape
    qmax = 2 ** bits - 1
    R = (W.double() - B.double() @ A.double()).view(N, K // 128, 128)
    lo, hi = R.amin(2), R.amax(2)
    s = half_once(torch.where(hi > lo, (hi - lo) / qmax, torch.ones_like(hi))).clamp_min(2.0 ** -14)
    while True:
        z = half_once(-lo / s.double())
        off = ~((lo / s.double() + z.double() >= -0.5) & (hi / s.double() + z.double() <= qmax + 0.5)) & (s < 65504)
        if not bool(off.any()):
            return s, z, torch.round(R / s.double()[:, :, None] + z.double()[:, :, None]).clamp_(0, qmax).view(N, K).to(torch.uint8)
        s = torch.where(off, (s.view(torch.int16) + 1).view(torch.float16), s)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("r", [8, 32, 64, 136, 256])
@pytest.mark.parametrize("kind", ["one size", "mixed sizes", "cancelling", "subnormal", "one large", "near"])
def test_codes_where_the_sums_in_32_bits_are_strained(kind, r, bits):
    """The quantizer decides in 32 bits what a bound on the error of its sums allows; the bound rests on how the fp16 matrix instruction rounds (eight products at a time, operands cut 2^-24
    below the largest, subnormals aligned as 2^-14).  Eight million elements a case, the branch as large as the weights or larger, so that hundreds lie within the bound of a rounding
    boundary and as many just outside: products of one size and of sizes 2^24 apart, sums that cancel, subnormal operands, one product far above the rest.  Every word as in 64 bits."""
    import torch
    import paper_2501_16385_amd as fbq
    N, K = 2048, 4096
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * r + bits)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    power = lambda lo, hi, *s: 2.0 ** torch.randint(lo, hi + 1, s, device="cuda", generator=g)
    A, B = rand(r, K) * 0.1, rand(N, r) * 0.1
    if kind == "one size":
        A, B = torch.sign(A) * (1 + torch.rand(r, K, device="cuda", generator=g) * 2.0 ** -9) * 0.1, torch.sign(B) * 0.1
    elif kind == "mixed sizes":
        A, B = A * power(-12, 0, r, K), B * power(-12, 0, N, r)
    elif kind == "cancelling":
        A[1::2], B[:, 1::2] = A[::2] * (1 + rand(r // 2, K) * 2.0 ** -9), -B[:, ::2]
    elif kind == "subnormal":
        A, B = A * power(-18, -10, r, K), B * power(-6, 12, N, r)
    elif kind == "one large":
        A[r // 2] *= 64.0
        B[:, r // 2] *= 64.0
    A, B = A.half(), B.half()
    sigma = B.double() @ A.double()
    W = (sigma + (0.02 if kind == "near" else 1.0) * sigma.std() * rand(N, K)).half()
    d = fbq.Desc(N, K, r, bits)
    dev = fbq.quantize_feedback(d, W, A.view(torch.int16), B.view(torch.int16))
    s, z, q = quantize_in_64_bits(W, A, B, bits)
    assert torch.equal(dev.scales.view(torch.float16), s)
    assert torch.equal(dev.zeros.view(torch.float16), z)
    off = fbq.unpack_codes(dev) != q
    assert not bool(off.any()), (int(off.sum()), off.nonzero()[:5].tolist())


def quantize_group_by_the_book(R, qmax):
    """Scale, zero and codes of one group as include/fbq.h defines them, the scale stepped through every fp16 number: extremes that
    ignore NaN, comparisons that a NaN fails, clamping that turns a NaN into code 0."""
    with np.errstate(all="ignore"):
        lo, hi = np.fmin.reduce(R), np.fmax.reduce(R)
        s = (hi - lo) / qmax
        bits = max(int(np.float16(s if s > 0 else 1.0).view(np.uint16)), 0x0400)
        while True:
            sd = float(np.uint16(bits).view(np.float16))
            z = np.float16(-lo / sd)
            if (lo / sd + float(z) >= -0.5 and hi / sd + float(z) <= qmax + 0.5) or bits >= 0x7bff:
                break
            bits += 1
        q = np.fmin(np.fmax(np.rint(R / sd + float(z)), 0.0), qmax).astype(np.uint8)
    return bits, z, q


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("r", [0, 8])
def test_quantizer_with_weights_that_are_no_numbers(bits, r):
    """NaN and infinite weights: the search for a scale ends where it always ended, and nothing else of the layer changes."""
    import torch
    import paper_2501_16385_amd as fbq
    K, inf, nan = 256, np.inf, np.nan
    rng = np.random.Generator(np.random.Philox(49))
    W = (rng.standard_normal((17, K)) * 0.02).astype(np.float16)
    W[1, 5] = nan                                       # one NaN
    W[2, :128] = nan                                    # a whole group
    W[3, 7], W[4, 130], W[5, 0], W[5, 127] = inf, -inf, inf, -inf
    W[6, :128], W[7, :128] = inf, -inf                  # nothing else in the group
    W[8, 3], W[8, 4] = inf, nan
    W[9, :128] = nan
    W[9, 64] = inf
    W[10, 1], W[10, 2] = 65504, -65504                  # finite after all
    W[11, :128] = 0.25                                  # constant
    W[12, :128:2], W[12, 1:128:2] = inf, nan
    At = (rng.standard_normal((max(r, 1), K)) * 0.01).astype(np.float16)
    Bt = (rng.standard_normal((17, max(r, 1))) * 0.01).astype(np.float16)
    if r:
        Bt[13, 3], Bt[14, 2] = inf, nan                 # a branch that is no number
    dev = fbq.quantize_feedback(fbq.Desc(17, K, r, bits), t16(W), t16(At) if r else None, t16(Bt) if r else None)
    codes = fbq.unpack_codes(dev)
    torch.cuda.synchronize()
    codes, s, z = codes.cpu().numpy(), dev.scales.cpu().numpy().view(np.uint16), dev.zeros.cpu().numpy().view(np.float16)
    with np.errstate(all="ignore"):
        R = W.astype(np.float64) - (Bt.astype(np.float64) @ At.astype(np.float64) if r else 0.0)
    for n in range(17):
        for g in range(2):
            want_s, want_z, want_q = quantize_group_by_the_book(R[n, g * 128:(g + 1) * 128], 2 ** bits - 1)
            where = f"row {n} group {g}"
            assert s[n, g] == want_s, where
            # a zero that is no number is stored as an infinity, of either sign
            assert np.isinf(z[n, g]) if np.isnan(want_z) else z[n, g] == want_z, where
            assert np.array_equal(codes[n, g * 128:(g + 1) * 128], want_q), where


# ------------------------------------------------------------------ prefill GEMM: tiles of 64, 96, 128, 192 and 256 rows x 256 columns, K split over blocks

PREFILL_CASES = [
    # N, K, r, M (prefill_cases.py has a layer for every kind of cut)
    # (the per-token bar is relative to the norm of a token's outputs: a few dozen columns, so that it is no single cancelled sum)
    (25, 128, 8, 65),           # one quantization group
    (40, 256, 40, 77),          # a rank that is no multiple of 16 or 64
    (25, 2304, 24, 65),         # K split over three blocks, M N odd: the summing launch's scalar form
    (255, 4224, 200, 77),       # K split over six blocks, an odd number of groups
    (513, 1408, 256, 66),       # four tiles of taps
    (4100, 640, 0, 300),
    (33001, 128, 0, 65),
    (33001, 640, 72, 96),
    (33001, 128, 72, 97),
    (33000, 640, 8, 128),       # whole rows stored
    (33001, 128, 16, 129),
    (33000, 640, 40, 191),
    (33001, 128, 40, 193),
    (33000, 640, 64, 193),
    # several row blocks of many column blocks (several groups per row: with a single one, millions of
    # outputs include small ones of rows with a scale far above the average, which the bound on single outputs is relative to)
    (32957, 640, 24, 583),
    (26297, 640, 8, 546),
]


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M", PREFILL_CASES)
def test_prefill_tile_edges(bits, N, K, r, M):
    """Weights enter the matrix cores with two fp16 roundings (2^-11 of the weight, 2^-12 of a step) and y is rounded once:
    3.5e-4 relative; the bars are those of the other parity tests.  Output and workspace start as NaN patterns."""
    import torch
    import paper_2501_16385_amd as fbq
    spec = fbq_synth.LayerSpec("edge", N, K, r, bits)
    rng = np.random.Generator(np.random.Philox(43))
    codes, s, z = fbq_synth.make_random_quantized(spec, 42, 3)
    A, B = fbq_synth.make_branch(spec, 42, 3) if r else (None, None)
    x = rng.standard_normal((M, K)).astype(np.float16)
    want = orc.linear(x, orc.pack(codes, bits), s, z, A, B, bits, 128)
    p = fbq.pack(fbq.Desc(N, K, r, bits), codes, s, z, A, B)
    dev = fbq.upload_layer(p)
    dev = fbq.DeviceLayer(dev.desc, *[framed_in_nan(t) for t in (dev.qweight, dev.scales, dev.zeros, dev.At, dev.Bt)])
    xd = framed_in_nan(torch.from_numpy(x).cuda())
    y = framed_in_nan(torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda"))
    ws = framed_in_nan(torch.full((fbq.workspace_bytes(dev.desc, M),), 0x7D, dtype=torch.uint8, device="cuda"))
    fbq.linear(dev, xd, y, ws)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert_matches_oracle(got, want, f"{N}x{K} r={r} M={M}", tol=1e-3)
    y.fill_(float("nan"))
    fbq.linear(dev, xd, y, ws)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), got)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M,cut", CUT_CASES + ORDER_CASES)
def test_prefill_every_kind_of_cut(bits, N, K, r, M, cut):
    """The bars of the test above (assert_matches_oracle's), against W_F in 64 bits from the layer's own codes on the device: these
    layers are too large for the oracle on the host."""
    import torch
    import paper_2501_16385_amd as fbq
    from helpers import ELEMENT_SLACK, framed_layer
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(48)
    layer = framed_layer(random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0))
    x = framed_in_nan(torch.randn(M, K, device="cuda", generator=g).half())
    y = framed_in_nan(torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda"))
    ws = framed_in_nan(torch.full((fbq.workspace_bytes(layer.desc, M),), 0x7D, dtype=torch.uint8, device="cuda"))
    fbq.linear(layer, x, y, ws)
    f64 = lambda t: t.view(torch.float16).double()
    W = ((fbq.unpack_codes(layer).view(N, K // 128, 128).double() - f64(layer.zeros)[:, :, None]) * f64(layer.scales)[:, :, None]).view(N, K)
    want = x.double() @ W.T.contiguous()
    if r:
        want += (x.double() @ f64(layer.At).T.contiguous()) @ f64(layer.Bt).T.contiguous()
    miss = (y.double() - want).abs_()
    assert bool(torch.isfinite(miss).all())
    per_token = miss.norm(dim=1) / want.norm(dim=1)
    assert float(miss.norm() / want.norm()) <= 1e-3 and float(per_token.max()) <= 1e-3
    assert float((miss - want.abs() * 2.0 ** -10 - ELEMENT_SLACK["prefill"] * want.square().mean(1, keepdim=True).sqrt()).max()) <= 0.0


# ------------------------------------------------------------------ symmetric products: tiles of 192, the contraction split over blocks

@pytest.mark.parametrize("K,T", [(128, 1), (256, 4100), (384, 65), (640, 193), (1152, 300), (2176, 837),
                                 (128, 20000), (384, 5000), (1152, 1500)])     # few features: the contraction split over up to 22 blocks
def test_gram_tile_edges(K, T):
    """fp16 of a 32-bit sum: 2^-11 / sqrt(3) relative; both triangles come from the same sums, so H is symmetric to the bit."""
    import torch
    import paper_2501_16385_amd as fbq
    rng = np.random.Generator(np.random.Philox(44))
    X = rng.standard_normal((T, K)).astype(np.float16)
    d = fbq.Desc(128, K, 8, 4)
    ws = framed_in_nan(torch.full((fbq.train_workspace_bytes(d, T),), 0x7D, dtype=torch.uint8, device="cuda"))
    H = fbq.gram(d, framed_in_nan(torch.from_numpy(X).cuda()), 1.0 / T, ws)
    torch.cuda.synchronize()
    H = H.cpu().numpy()
    X64 = X.astype(np.float64)
    want = X64.T @ X64 / T
    assert np.linalg.norm(H.astype(np.float64) - want) <= 5e-4 * np.linalg.norm(want)
    assert np.array_equal(H, H.T)


def test_gram_of_few_features_takes_no_longer_than_of_many():
    """128 features have a sixty-fourth of the products of 1024.  Where the contraction is split over blocks, the sum of the
    partial tiles must not take that back (read one after the other they took 73 us and 57; 18 and 28 now)."""
    import torch
    import paper_2501_16385_amd as fbq

    def us(K, T=4096):
        d = fbq.Desc(128, K, 8, 4)
        X, ws = torch.randn(T, K, device="cuda").half(), torch.empty(fbq.train_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(7):
            torch.cuda.synchronize()
            e[0].record()
            for _ in range(10):
                fbq.gram(d, X, 1.0 / T, ws)
            e[1].record()
            torch.cuda.synchronize()
            times.append(e[0].elapsed_time(e[1]) * 100)
        return sorted(times)[3]

    assert us(128) <= us(1024)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r", [(1, 128, 8), (65, 384, 64), (200, 256, 72), (129, 640, 136), (700, 1152, 256)])
def test_train_step_tile_edges(bits, N, K, r):
    """Gradients, loss and update of one step from the step's own codes and the H it was given, in fp64.  Three fp16 roundings
    of 2^-11 and 32-bit sums (a few 1e-4); bars as in the parity tests of the step."""
    import torch
    import paper_2501_16385_amd as fbq
    L = make_oracle_layer(fbq_synth.LayerSpec("edge", N, K, r, bits), config=45)
    rng = np.random.Generator(np.random.Philox(46))
    X = rng.standard_normal((96, K))
    H = ((X.T @ X) / 96).astype(np.float16)
    H = np.triu(H) + np.triu(H, 1).T
    d = fbq.Desc(N, K, r, bits)
    At, Bt = (torch.from_numpy(np.ascontiguousarray(m.T).astype(np.float32)).cuda() for m in (L.A, L.B))
    st = fbq.train_state(d, At.clone(), Bt.clone())
    st.workspace = framed_in_nan(torch.full_like(st.workspace, 0x7D))
    lr = 1e-6
    fbq.train_step(st, t16(L.W), t16(H), 1.0 / 96, lr)
    torch.cuda.synchronize()
    A64, B64, H64 = L.A.astype(np.float64).T, L.B.astype(np.float64).T, H.astype(np.float64) * 96
    s, z = (np.repeat(v.astype(np.float64), 128, axis=1) for v in (L.scales, L.zeros))
    D = (L.W.astype(np.float64) - B64 @ A64) - s * (L.codes - z)
    P = D @ H64
    gA, gB = -2.0 * B64.T @ P, -2.0 * P @ A64.T
    rel = lambda got, want: np.linalg.norm(got.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want)
    assert rel(st.grad_At, gA) < 2e-3 and rel(st.grad_Bt, gB) < 2e-3
    assert rel(st.loss, np.array([np.sum(D * P)])) < 1e-3
    # the update is one fp32 multiply-subtract of the gradient that was written
    for got, start, grad in ((st.At32, At, st.grad_At), (st.Bt32, Bt, st.grad_Bt)):
        step = start.double() - lr * grad.double()
        assert float((got.double() - step).abs().max()) <= 2.0 ** -23 * float(start.abs().max()) + 1e-12


# ------------------------------------------------------------------ averages written with the result, silu(gate) * up

@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [1, 2, 5, 16, 40, 70])
@pytest.mark.parametrize("N,K,r", [(1, 128, 0), (33, 384, 8), (130, 256, 16), (4098, 128, 0), (2050, 8320, 24),
                                   (130, 640, 136), (2050, 8192, 200), (514, 16384, 256)])   # two taps per lane; INT4: no instance that averages
def test_group_mix_equals_result_then_average(bits, M, N, K, r):
    """Every way the averages are written (GEMV trips even and odd, matrix-core tiles, a launch of its own): y bit for bit that of
    the plain call, the average bit for bit the element-wise one."""
    import torch
    import paper_2501_16385_amd as fbq
    g = torch.Generator(device="cuda")
    g.manual_seed(47 + M + N)
    from paper_2501_16385_amd.random_layers import random_layer
    layers = [random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0) for _ in range(2)]
    x = torch.randn(M, K, device="cuda", generator=g).half()
    with_ = framed_in_nan(torch.randn(M, N, device="cuda", generator=g).half())
    want = fbq.linear_group(layers, [x, x])
    ys, out = [torch.empty_like(w) for w in want], framed_in_nan(torch.empty(M, N, dtype=torch.float16, device="cuda"))
    need = fbq.workspace_bytes(layers[0].desc, M)
    wss = [torch.zeros(need, dtype=torch.uint8, device="cuda") if need else None for _ in layers]
    arr = fbq.make_group(layers, [x, x], ys, wss)
    stream = torch.cuda.current_stream().cuda_stream
    assert fbq.load().fbq_linear_group_mix(arr, fbq.make_mix([None, with_], [None, out]), 2, M, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(ys[0], want[0]) and torch.equal(ys[1], want[1])
    assert torch.equal(out, torch.lerp(with_, want[1], 0.5))


@pytest.mark.parametrize("count", [1, 7, 8, 2047, 2049, 5 * 11008])
def test_silu_mul_equals_two_element_wise_kernels(count):
    """silu rounded to fp16, then the product.  Where the exponential differs in its last place, silu may round to the neighbouring
    number (2^-10 relative at most) and the product to one more (2^-11 each side of it): 2^-9 in all, and one subnormal step."""
    import torch
    import paper_2501_16385_amd as fbq
    g = torch.Generator(device="cuda")
    g.manual_seed(count)
    gate, up = (framed_in_nan((torch.randn(count, device="cuda", generator=g) * 3).half()) for _ in range(2))
    out = fbq.silu_mul(gate, up, framed_in_nan(torch.empty(count, dtype=torch.float16, device="cuda")))
    want = torch.nn.functional.silu(gate) * up
    torch.cuda.synchronize()
    assert float(((out.double() - want.double()).abs() - 2.0 ** -9 * want.double().abs()).max()) <= 2.0 ** -24


# ------------------------------------------------------------------ streaming kernel for 3 to 16 tokens: 10240 rows and 40 million codes on

def framed_random_layer(N, K, r, bits, seed):
    """A layer of random codes inside NaN frames, and W_F = s (q - z) + B A of it in 64 bits."""
    import torch
    import paper_2501_16385_amd as fbq
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dev = framed_layer(random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0))
    q = fbq.unpack_codes(dev).view(N, K // 128, 128).double()
    s, z = (t.view(torch.float16).double()[:, :, None] for t in (dev.scales, dev.zeros))
    W = ((q - z) * s).view(N, K)
    if r:
        W.addmm_(dev.Bt.view(torch.float16).double(), dev.At.view(torch.float16).double())
    return dev, W, g


STREAM_CASES = [
    # N, K, r, M: group counts below, at and above one pass (32), two units (64) and several passes; odd numbers of scales; tiles of
    # one row; one to more than eight tiles a block; token counts on both sides of 8; ranks on both sides of 32 and 128
    (10241, 3968, 8, 3),
    (40001, 1024, 16, 16),
    (10243, 4224, 40, 9),
    (10240, 8192, 200, 8),
    (10245, 8320, 72, 5),
    (10305, 32768, 256, 16),
    (140001, 512, 0, 4),
    (140001, 384, 24, 7),
    (70003, 1408, 136, 16),
    (16384, 4096, 64, 8),
    # sets of 16 tokens side by side, one set not full, one or two tokens left over
    (4096, 4096, 64, 64),
    (4099, 4224, 0, 51),
    (5120, 4096, 128, 49),
    (3585, 11008, 96, 34),
]


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M", STREAM_CASES)
def test_stream_edges(bits, N, K, r, M):
    import torch
    dev, W, g = framed_random_layer(N, K, r, bits, 51 + N + M)
    x = torch.randn(M, K, device="cuda", generator=g).half()
    want = (x.double() @ W.T).cpu().numpy()
    del W
    x_np = x.cpu().view(torch.int16).numpy().view(np.float16)
    y = gpu_y(dev, x_np)
    assert_matches_oracle(y, want, f"INT{bits} {N}x{K} r={r} M={M}")
    assert np.array_equal(y, gpu_y(dev, x_np))


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M,way", SETS_OR_GEMM_CASES)
def test_sets_or_gemm_edges(bits, N, K, r, M, way):
    """Each within the bound of the path that takes it (sets and split multiply the codes exactly, the GEMM rounds every weight to fp16: the
    two bounds beside ELEMENT_SLACK), also with a workspace that calls of other token counts have used."""
    import torch
    import paper_2501_16385_amd as fbq
    dev, W, g = framed_random_layer(N, K, r, bits, 71 + N + M)
    x = torch.randn(M, K, device="cuda", generator=g).half()
    want = (x.double() @ W.T).cpu().numpy()
    del W
    x_np = x.cpu().view(torch.int16).numpy().view(np.float16)
    y = gpu_y(dev, x_np)
    assert_matches_oracle(y, want, f"INT{bits} {N}x{K} r={r} M={M}", "prefill" if way == "gemm" else "few")
    x65 = torch.randn(65, K, device="cuda", generator=g).half()
    ws = torch.zeros(max(fbq.workspace_bytes(dev.desc, m) for m in (65, M, 16, 2)), dtype=torch.uint8, device="cuda")
    for other in (x65, x65[:16], x65[:2], x):
        shared = fbq.linear(dev, other, workspace=ws)
    assert np.array_equal(shared.cpu().view(torch.int16).numpy(), y.view(np.int16))


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M", [(33001, 1280, 72, 6), (10241, 4096, 8, 16)])
def test_stream_group_average_and_late_hand_over(bits, N, K, r, M):
    """Grouped, averaged and single calls agree bit for bit; and with consumers that never wait for the down-projection (they compute t
    themselves, in another order) the result is still the oracle's."""
    import torch
    import paper_2501_16385_amd as fbq
    (a, Wa, g), (b, _, _) = (framed_random_layer(N, K, r, bits, 61 + i) for i in range(2))
    x = torch.randn(M, K, device="cuda", generator=g).half()
    single = [fbq.linear(l, x) for l in (a, b)]
    with_ = framed_in_nan(torch.randn(M, N, device="cuda", generator=g).half())
    ys, out = [torch.empty_like(y) for y in single], framed_in_nan(torch.empty(M, N, dtype=torch.float16, device="cuda"))
    wss = [torch.zeros(fbq.workspace_bytes(l.desc, M), dtype=torch.uint8, device="cuda") for l in (a, b)]
    arr = fbq.make_group([a, b], [x, x], ys, wss)
    assert fbq.load().fbq_linear_group_mix(arr, fbq.make_mix([None, with_], [None, out]), 2, M, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(ys[0], single[0]) and torch.equal(ys[1], single[1])
    assert torch.equal(out, torch.lerp(with_, single[1], 0.5))
    before = fbq.load().fbq_test_set_spin_limit(-1)
    try:
        alone = fbq.linear(a, x)
        torch.cuda.synchronize()
    finally:
        assert fbq.load().fbq_test_set_spin_limit(before) == -1
    assert_matches_oracle(alone.cpu().numpy(), (x.double() @ Wa.T).cpu().numpy(), f"INT{bits} {N}x{K} r={r} M={M}, t computed by its consumers")


UNEQUAL_GROUPS = [
    # K, {N, r} of each layer: two to four layers in line, one to more than eight tiles a block, ranks on both sides of 32 and 128, none
    (4096, [(10240, 8), (14337, 256), (20001, 40)]),
    (1280, [(50001, 0), (33251, 0)]),
    (4224, [(10241, 64), (10240, 64), (12289, 8), (16385, 200)]),
    (8320, [(10240, 24), (13001, 136)]),
    (4096, [(10240, 64), (10240, 72), (10240, 64)]),
    # layers too small for the streaming kernel along with it: below one block's rows, odd numbers of scales, more blocks than CUs, alone after it
    (4096, [(10240, 64), (1024, 64), (1000, 16)]),
    (4096, [(8200, 128), (11008, 8)]),
    (1280, [(33001, 0), (700, 0), (8001, 0)]),
    (4224, [(999, 40), (10241, 200), (7, 8)]),
    (8320, [(13001, 136), (4099, 8)]),
    (12288, [(10240, 64), (1024, 64), (1024, 64)]),
]


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [5, 16])
@pytest.mark.parametrize("K,layers", UNEQUAL_GROUPS)
def test_stream_group_of_unequal_layers(K, layers, M, bits):
    """Every layer of a grouped call gets exactly what a call of its own gives it, whatever it shares the launch with."""
    import torch
    import paper_2501_16385_amd as fbq
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(81 + K + M)
    devs = [framed_layer(random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0)) for N, r in layers]
    x = framed_in_nan(torch.randn(M, K, device="cuda", generator=g).half())
    single = [fbq.linear(l, x) for l in devs]
    with_ = [framed_in_nan(torch.randn(M, N, device="cuda", generator=g).half()) for N, _ in layers]
    for order in (slice(None), slice(None, None, -1)):
        ys, outs = ([framed_in_nan(torch.empty_like(y)) for y in single[order]] for _ in range(2))
        wss = [torch.zeros(fbq.workspace_bytes(l.desc, M), dtype=torch.uint8, device="cuda") if l.desc.r else None for l in devs[order]]
        fbq.linear_group(devs[order], [x] * len(devs), ys=ys, workspaces=wss)
        torch.cuda.synchronize()
        for (N, r), y, want in zip(layers[order], ys, single[order]):
            assert torch.equal(y, want), (N, r)
            y.fill_(0)
        arr, mix = fbq.make_group(devs[order], [x] * len(devs), ys, wss), fbq.make_mix(with_[order], outs)
        assert fbq.load().fbq_linear_group_mix(arr, mix, len(devs), M, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        for (N, r), y, want, w, out in zip(layers[order], ys, single[order], with_[order], outs):
            assert torch.equal(y, want) and torch.equal(out, torch.lerp(w, want, 0.5)), (N, r)


LATE_GROUPS = [
    # K, M, {N, r}: two units a tile, several passes, in line with a small layer; one tile a block and more than the eight of two rounds
    (4224, 6, [(33001, 40)]),
    (4224, 16, [(10243, 200)]),
    (8320, 16, [(33001, 72)]),
    (16384, 3, [(10241, 8)]),
    (4096, 16, [(10240, 64), (1000, 16)]),
    (8192, 7, [(1001, 136), (10241, 24), (12289, 72)]),
    (12288, 5, [(10240, 64), (1024, 40)]),
]


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("K,M,layers", LATE_GROUPS)
def test_stream_consumers_that_never_wait(K, M, layers, bits):
    """Blocks that find no down-projection compute t themselves, in another order: the result, and its average, are the oracle's all the same."""
    import torch
    import paper_2501_16385_amd as fbq
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(91 + K + M)
    devs = [framed_layer(random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0)) for N, r in layers]
    x = framed_in_nan(torch.randn(M, K, device="cuda", generator=g).half())
    ys, outs = ([framed_in_nan(torch.empty(M, N, dtype=torch.float16, device="cuda")) for N, _ in layers] for _ in range(2))
    with_ = [framed_in_nan(torch.randn(M, N, device="cuda", generator=g).half()) for N, _ in layers]
    wss = [torch.zeros(fbq.workspace_bytes(l.desc, M), dtype=torch.uint8, device="cuda") for l in devs]
    before = fbq.load().fbq_test_set_spin_limit(-1)
    try:
        arr, mix = fbq.make_group(devs, [x] * len(devs), ys, wss), fbq.make_mix(with_, outs)
        assert fbq.load().fbq_linear_group_mix(arr, mix, len(devs), M, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
    finally:
        assert fbq.load().fbq_test_set_spin_limit(before) == -1
    f64 = lambda t: t.view(torch.float16).double()
    for dev, y, w, out in zip(devs, ys, with_, outs):
        N = dev.desc.N
        want = x.double() @ ((fbq.unpack_codes(dev).view(N, K // 128, 128).double() - f64(dev.zeros)[:, :, None]) * f64(dev.scales)[:, :, None]).view(N, K).T
        want += (x.double() @ f64(dev.At).T) @ f64(dev.Bt).T
        assert_matches_oracle(y.cpu().numpy(), want.cpu().numpy(), f"INT{bits} {N}x{K} M={M}, t computed by its consumers")
        assert torch.equal(out, torch.lerp(w, y, 0.5))


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("K,M,layers", [(4096, 9, [(10240, 64)]), (8192, 16, [(10245, 200)]), (8320, 5, [(10240, 72)]),
                                        (4096, 16, [(10240, 64), (1000, 16)]), (4096, 40, [(5121, 24)])])
def test_stream_replayed_graph_follows_new_activations(K, M, layers, bits):
    """Replays of a captured launch hand over the t of their own activations, with eager calls on the same workspace in between."""
    import torch
    import paper_2501_16385_amd as fbq
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(101 + K + M)
    devs = [random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0) for N, r in layers]
    x = torch.randn(M, K, device="cuda", generator=g).half()
    ys = [torch.empty(M, N, dtype=torch.float16, device="cuda") for N, _ in layers]
    wss = [torch.zeros(fbq.workspace_bytes(l.desc, M), dtype=torch.uint8, device="cuda") for l in devs]
    fbq.linear_group(devs, [x] * len(devs), ys=ys, workspaces=wss)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fbq.linear_group(devs, [x] * len(devs), ys=ys, workspaces=wss)
    for rep in range(4):
        x.copy_(torch.randn(M, K, device="cuda", generator=g).half())
        graph.replay()
        torch.cuda.synchronize()
        got = [y.clone() for y in ys]
        fresh = fbq.linear_group(devs, [x] * len(devs))
        fbq.linear_group(devs, [x.flip(0)] * len(devs), ys=ys, workspaces=wss)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, fresh)), rep
        assert not torch.equal(got[0], ys[0])


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M", [(10241, 4224, 40, 9), (10240, 8320, 72, 3), (33001, 1280, 8, 16)])
def test_stream_behind_the_other_entry_points(N, K, r, M, bits):
    """The library's own scratch gives the bits of fbq_linear; the unfused comparator differs by the fp16 rounding of t."""
    import torch
    import paper_2501_16385_amd as fbq
    dev, W, g = framed_random_layer(N, K, r, bits, 111 + N + M)
    x = framed_in_nan(torch.randn(M, K, device="cuda", generator=g).half())
    y = fbq.linear(dev, x)
    assert torch.equal(fbq.linear_static(dev, x), y)
    want = x.double() @ W.T
    miss = (fbq.linear_unfused(dev, x).double() - want).norm() / want.norm()
    assert float(miss) <= 1.5e-3, float(miss)


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,M,otherwise", SPLIT_CASES)
def test_split_edges(bits, N, K, r, M, otherwise):
    """Against 64 bits, with the bound of exactly multiplied codes, on a workspace whose every byte was part of a NaN; the same bits again; and,
    without the room that the split needs, within the bound of the path that serves such a workspace: hand-over words are enough where the few-token kernels do, and
    nothing less than the GEMM's own workspace where that does."""
    import ctypes
    import torch
    import paper_2501_16385_amd as fbq
    dev, W, g = framed_random_layer(N, K, r, bits, 111 + N + M)
    x = framed_in_nan(torch.randn(M, K, device="cuda", generator=g).half())
    want = (x.double() @ W.T).cpu().numpy()
    del W
    need = fbq.workspace_bytes(dev.desc, M)
    ws = framed_in_nan(torch.full((need,), 0x7D, dtype=torch.uint8, device="cuda"))
    ys = [framed_in_nan(torch.empty(M, N, dtype=torch.float16, device="cuda")) for _ in range(2)]
    for y in ys:
        fbq.linear(dev, x, y, ws)
    assert_matches_oracle(ys[0].cpu().numpy(), want, f"INT{bits} {N}x{K} r={r} M={M}", "few")
    assert torch.equal(ys[0], ys[1])
    ptr = lambda t: None if t is None else t.data_ptr()

    def given(size):
        small = framed_in_nan(torch.zeros(size, dtype=torch.uint8, device="cuda")) if size else None
        ys[1].fill_(float("nan"))
        return fbq.load().fbq_linear(ctypes.byref(dev.desc.c()), M, x.data_ptr(), ptr(dev.qweight), ptr(dev.scales), ptr(dev.zeros), ptr(dev.At), ptr(dev.Bt),
                                     ys[1].data_ptr(), ptr(small), size, torch.cuda.current_stream().cuda_stream)

    words = -(-M // 16) * 17 * 16 * r * 8                # hand-over words of 16 tokens each
    if otherwise == "gemm":
        # activations in tiles, scales and zeros by group are the least that the GEMM keeps; its plan's partial sums may come on top
        assert given(words) == (5 if words else 1) and given(4 * 17 * 16 * r * 8 + 2 * M * K) == 5
        low, high = 4 * 17 * 16 * r * 8 + 2 * M * K, need    # refused, accepted
        while high - low > 1:
            low, high = (low, (low + high) // 2) if given((low + high) // 2) == 0 else ((low + high) // 2, high)
        words = high
    elif words:
        assert given(words - 1) == 5
    assert given(words) == 0
    torch.cuda.synchronize()
    assert_matches_oracle(ys[1].cpu().numpy(), want, f"INT{bits} {N}x{K} r={r} M={M}, smaller workspace", "prefill" if otherwise == "gemm" else "few")


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r", [(2050, 16640, 64), (19001, 4096, 40)])
def test_one_workspace_for_split_and_other_calls(bits, N, K, r):
    """One workspace, zero-filled once, for calls of every kind: what a split call keeps lies behind the hand-over words of the others, and each gives what it gives by itself."""
    import torch
    import paper_2501_16385_amd as fbq
    dev, W, g = framed_random_layer(N, K, r, bits, 131 + N)
    counts = [40, 5, 1, 64, 70, 16, 2, 17, 48, 33, 9]
    ws = torch.zeros(max(fbq.workspace_bytes(dev.desc, M) for M in counts), dtype=torch.uint8, device="cuda")
    front = 4 * 17 * 16 * r * 8
    splits = 0
    for M in counts:
        x = torch.randn(M, K, device="cuda", generator=g).half()
        alone = fbq.linear(dev, x)
        before = ws[:front].clone()
        y = fbq.linear(dev, x, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(y, alone), M
        assert_matches_oracle(y.cpu().numpy(), (x.double() @ W.T).cpu().numpy(), f"INT{bits} {N}x{K} r={r} M={M}", "prefill" if M > 64 else "few" if M > 2 else "gemv")
        if fbq.workspace_bytes(dev.desc, M) > front:     # split, or the GEMM
            splits += M <= 64
            assert torch.equal(ws[:front], before), M
    assert splits >= 4


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("M", [5, 16])
def test_split_group_average_and_replayed_graph(bits, M):
    """Layers of a grouped call get the bits of their own calls, averages included, also in replays on new activations with eager calls in between."""
    import torch
    import paper_2501_16385_amd as fbq
    from paper_2501_16385_amd.random_layers import random_layer
    g = torch.Generator(device="cuda")
    g.manual_seed(121 + M)
    K, shapes = 17408, [(2049, 8), (4100, 72), (1000, 16), (2304, 0)]
    devs = [framed_layer(random_layer(fbq.Desc(N, K, r, bits), g, gain=1.0)) for N, r in shapes]
    x = torch.randn(M, K, device="cuda", generator=g).half()
    with_ = [torch.randn(M, N, device="cuda", generator=g).half() for N, _ in shapes]
    ys, outs = ([framed_in_nan(torch.empty(M, N, dtype=torch.float16, device="cuda")) for N, _ in shapes] for _ in range(2))
    need = [fbq.workspace_bytes(d.desc, M) for d in devs]
    wss = [torch.zeros(n, dtype=torch.uint8, device="cuda") if n else None for n in need]
    arr, mix = fbq.make_group(devs, [x] * 4, ys, wss), fbq.make_mix(with_, outs)
    call = lambda: fbq.load().fbq_linear_group_mix(arr, mix, 4, M, torch.cuda.current_stream().cuda_stream)
    assert call() == 0
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert call() == 0
    for _ in range(3):
        x.copy_(torch.randn(M, K, device="cuda", generator=g).half())
        single = [fbq.linear(d, x) for d in devs]
        graph.replay()
        torch.cuda.synchronize()
        for y, want, w, out in zip(ys, single, with_, outs):
            assert torch.equal(y, want) and torch.equal(out, torch.lerp(w, want, 0.5))
