"""GPU parity of the layer-wise reconstruction step (Alg. 1, Sec. 4.2) against the fp64 oracle,
through the C ABI.

Tolerances.  The quantizer runs the oracle's fp64 arithmetic, so codes, scales and zeros are compared
exactly (a code may differ on an exact tie of the rounding; none is expected on these inputs and at
most 1e-4 of the elements is accepted).  Delta_F, H and Delta_F.H enter the matrix cores rounded to
fp16 (2^-11 relative each, independent) and are accumulated in fp32: every gradient entry is a sum of
thousands of such products, so the relative L2 error of a gradient is a few 1e-4; the bar is 2e-3 for
the gradients and the updated masters' movement, 1e-3 for the loss.
"""
import ctypes

import numpy as np
import pytest
import torch

import fbq_synth
import paper_2501_16385_amd as fbq
from helpers import rel_l2
from oracle import fbq_oracle as orc

pytestmark = pytest.mark.gpu


def _dev16(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()


def _problem(N, K, r, bits, T, seed, b_zero):
    spec = fbq_synth.LayerSpec("train", N, K, r, bits)
    W = fbq_synth.make_weight(spec, 33, seed)
    A16, B16 = fbq_synth.make_branch(spec, 33, seed)
    X = fbq_synth.make_x(spec, T, 33, seed)
    A = np.ascontiguousarray(A16.astype(np.float64))
    B = np.zeros((r, N)) if b_zero else np.ascontiguousarray(B16.astype(np.float64))
    return spec, W, X, A, B


@pytest.mark.parametrize("K,T", [(256, 100), (1408, 321), (256, 4100)])     # the last one: few tiles, long contraction, K split over blocks
def test_gram_matches_definition(K, T):
    spec = fbq_synth.LayerSpec("gram", 128, K, 8, 4)
    X = fbq_synth.make_x(spec, T, 33, 1)
    d = fbq.Desc(128, K, 8, 4)
    h_scale = 1.0 / T
    H16 = fbq.gram(d, _dev16(X).view(torch.float16), h_scale)
    torch.cuda.synchronize()
    want = orc.gram(X) * h_scale
    assert rel_l2(H16.cpu().numpy().astype(np.float64), want) < 5e-4


CASES = [
    # N, K, r, T, B zero at the start (Alg. 1's initialisation)
    (256, 512, 16, 200, False),
    (300, 1408, 24, 130, False),      # ragged N: partial tiles, zero padding of the transposed operands
    (384, 1024, 64, 256, True),
    (130, 256, 8, 70, False),
    (256, 512, 128, 96, False),       # rank 128: the stacked operand [Q; At] spans two tile rows
    (1100, 384, 40, 64, False),       # more rows than input features; a rank that is no multiple of 16
]


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("N,K,r,T,b_zero", CASES)
def test_train_step_matches_oracle(bits, N, K, r, T, b_zero):
    spec, W, X, A, B = _problem(N, K, r, bits, T, 2, b_zero)
    d = fbq.Desc(N, K, r, bits)
    Hfull = orc.gram(X)
    h_scale = 1.0 / T
    lr = 0.02 / float(np.linalg.eigvalsh(Hfull)[-1] * np.linalg.norm(A, 2) ** 2)

    At32 = torch.from_numpy(np.ascontiguousarray(A.T).astype(np.float32)).cuda()
    Bt32 = torch.from_numpy(np.ascontiguousarray(B.T).astype(np.float32)).cuda()
    # both sides start from the same masters: the fp32 values
    A = np.ascontiguousarray(At32.cpu().numpy().T.astype(np.float64))
    B = np.ascontiguousarray(Bt32.cpu().numpy().T.astype(np.float64))
    st = fbq.train_state(d, At32, Bt32)
    Wd = _dev16(W).view(torch.float16)
    H16 = fbq.gram(d, _dev16(X).view(torch.float16), h_scale)

    for step in range(3):
        print(f"step {step}: N={N} K={K} r={r} T={T} bits={bits}", flush=True)
        A_before, B_before = A.copy(), B.copy()
        want = orc.train_step(W, X, A, B, lr, bits, spec.group)
        fbq.train_step(st, Wd, H16, h_scale, lr)
        torch.cuda.synchronize()

        # the layer written by the step: fp16 branch exactly, quantizer output exactly
        assert np.array_equal(st.layer.At.cpu().numpy().view(np.float16), want["A16"].T)
        assert np.array_equal(st.layer.Bt.cpu().numpy().view(np.float16), want["B16"].T)
        codes = fbq.unpack_codes(st.layer).cpu().numpy()
        cdiff = codes.astype(np.int16) - want["codes"].astype(np.int16)
        assert np.mean(cdiff != 0) <= 1e-4 and np.all(np.abs(cdiff) <= 1)     # a near-tie of the rounding, one step at most
        assert np.mean(st.layer.scales.cpu().numpy().view(np.float16) != want["scales"]) <= 1e-4
        assert np.mean(st.layer.zeros.cpu().numpy().view(np.float16) != want["zeros"]) <= 1e-4

        assert float(st.loss.cpu()[0]) == pytest.approx(want["loss"], rel=1e-3)
        gA = st.grad_At.cpu().numpy().astype(np.float64).T
        gB = st.grad_Bt.cpu().numpy().astype(np.float64).T
        if b_zero and step == 0:
            assert np.all(gA == 0.0)
        else:
            assert rel_l2(gA, want["gradA"]) < 2e-3
        assert rel_l2(gB, want["gradB"]) < 2e-3

        # the update, measured as movement of the masters
        dA = st.At32.cpu().numpy().astype(np.float64).T - A_before
        dB = st.Bt32.cpu().numpy().astype(np.float64).T - B_before
        if np.abs(A - A_before).max() > 0:
            assert rel_l2(dA, A - A_before) < 2e-3
        assert rel_l2(dB, B - B_before) < 2e-3
        # keep both sides on the same trajectory: hand the oracle the GPU's fp32 masters
        A = np.ascontiguousarray(st.At32.cpu().numpy().T.astype(np.float64))
        B = np.ascontiguousarray(st.Bt32.cpu().numpy().T.astype(np.float64))


def test_zero_learning_rate_leaves_the_masters_and_writes_a_usable_layer():
    spec, W, X, A, B = _problem(256, 512, 16, 4, 64, 3, False)
    d = fbq.Desc(256, 512, 16, 4)
    At32 = torch.from_numpy(np.ascontiguousarray(A.T).astype(np.float32)).cuda()
    Bt32 = torch.from_numpy(np.ascontiguousarray(B.T).astype(np.float32)).cuda()
    a0, b0 = At32.clone(), Bt32.clone()
    st = fbq.train_state(d, At32, Bt32)
    H16 = fbq.gram(d, _dev16(X).view(torch.float16), 1.0 / 64)
    fbq.train_step(st, _dev16(W).view(torch.float16), H16, 1.0 / 64, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(At32, a0) and torch.equal(Bt32, b0)
    # the layer it wrote runs through the inference path and reproduces x.W_F^T
    x = fbq_synth.make_x(spec, 5, 33, 9)
    y = fbq.linear(st.layer, _dev16(x).view(torch.float16))
    torch.cuda.synchronize()
    codes, s, z = orc.quantize(W, A.astype(np.float16), B.astype(np.float16), 4, 128)
    want = orc.linear(x, orc.pack(codes, 4), s, z, A.astype(np.float16), B.astype(np.float16), 4, 128)
    assert rel_l2(y.cpu().numpy().astype(np.float64), want) < 1e-3


def test_step_without_loss_gives_the_same_gradients():
    spec, W, X, A, B = _problem(256, 512, 16, 4, 64, 4, False)
    d = fbq.Desc(256, 512, 16, 4)
    mk = lambda: (torch.from_numpy(np.ascontiguousarray(A.T).astype(np.float32)).cuda(),
                  torch.from_numpy(np.ascontiguousarray(B.T).astype(np.float32)).cuda())
    st1, st2 = fbq.train_state(d, *mk()), fbq.train_state(d, *mk())
    Wd = _dev16(W).view(torch.float16)
    H16 = fbq.gram(d, _dev16(X).view(torch.float16), 1.0 / 64)
    fbq.train_step(st1, Wd, H16, 1.0 / 64, 1e-3)
    fbq.train_step(st2, Wd, H16, 1.0 / 64, 1e-3, want_loss=False)
    torch.cuda.synchronize()
    assert torch.equal(st1.grad_At, st2.grad_At) and torch.equal(st1.grad_Bt, st2.grad_Bt)
    assert torch.equal(st1.At32, st2.At32) and torch.equal(st1.Bt32, st2.Bt32)


def test_reconstruction_loop_lowers_the_loss_and_keeps_the_bound():
    """Alg. 1 end to end on a small layer: B starts at zero, the loss of every iterate is evaluated, the
    last layer is checked against the oracle's loss for the same parameters and against the s/2 bound."""
    from paper_2501_16385_amd.reconstruction import reconstruct_layer
    N, K, r, T, bits = 256, 512, 16, 256, 4
    spec = fbq_synth.LayerSpec("loop", N, K, r, bits)
    W = fbq_synth.make_weight(spec, 34, 0)
    X = fbq_synth.make_x(spec, T, 34, 0)
    d = fbq.Desc(N, K, r, bits)
    lam = float(np.linalg.eigvalsh(orc.gram(X))[-1])
    a_std = 0.01
    # plain gradient descent on a product of two factors: the step that is stable at the start stops being so once B has
    # grown, so stay well below 1 / (lambda_max |A|^2)
    lr = 0.05 / (lam * (a_std * (np.sqrt(K) + np.sqrt(r))) ** 2)
    layer, losses = reconstruct_layer(d, _dev16(W).view(torch.float16), _dev16(X).view(torch.float16), 40, lr, a_std=a_std)
    torch.cuda.synchronize()
    vals = [l for _, l in losses]
    assert vals[-1] < 0.85 * vals[0], f"loss {vals[0]:.4g} -> {vals[-1]:.4g}"
    assert all(np.isfinite(vals))
    # the oracle's loss for the final parameters (lr = 0 leaves them alone)
    A16 = layer.At.cpu().numpy().view(np.float16).T
    B16 = layer.Bt.cpu().numpy().view(np.float16).T
    want = orc.train_step(W, X, np.ascontiguousarray(A16.astype(np.float64)), np.ascontiguousarray(B16.astype(np.float64)), 0.0,
                          bits, spec.group)
    assert vals[-1] == pytest.approx(want["loss"], rel=1e-3)
    # Sec. 4.1: the reconstructed weight of the trained layer stays within s/2 of W
    WF = fbq.reconstruct(layer).cpu().numpy().astype(np.float64)
    s = np.repeat(layer.scales.cpu().numpy().view(np.float16).astype(np.float64), 128, axis=1)
    assert np.all(np.abs(W.astype(np.float64) - WF) <= 0.5 * s * (1 + 1e-4) + 1e-7)


@pytest.mark.parametrize("bits,N,K,r", [(3, 4100, 4096, 8), (4, 2100, 2048, 72), (4, 1030, 4096, 136), (3, 4100, 4096, 72), (4, 70, 256, 200), (3, 129, 128, 128)])
def test_gradients_at_the_quantizers_block_shapes(bits, N, K, r):
    """Blocks of four and eight waves, of one and two row tiles, rows past the last: the gradients, one of which contracts Delta_F over its rows and the other over its columns,
    against 64 bits from the step's own layer.  Three roundings to fp16 of 2^-11 each, as above: 2e-3."""
    g = torch.Generator(device="cuda")
    g.manual_seed(N + r)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    W, X, At, Bt = (rand(N, K) * 0.02).half(), rand(256, K).half(), rand(r, K) * 0.01, rand(N, r) * 0.01
    d = fbq.Desc(N, K, r, bits)
    H16 = fbq.gram(d, X, 1.0 / 256)
    st = fbq.train_state(d, At.clone(), Bt.clone())
    fbq.train_step(st, W, H16, 1.0 / 256, 0.0, want_loss=False)
    plain = fbq.quantize_feedback(d, W, At.half().view(torch.int16), Bt.half().view(torch.int16))
    for a, b in ((st.layer.qweight, plain.qweight), (st.layer.scales, plain.scales), (st.layer.zeros, plain.zeros)):
        assert torch.equal(a, b)
    A, B, H = At.half().double(), Bt.half().double(), H16.double() * 256
    s, z = (t.view(torch.float16).double()[:, :, None] for t in (plain.scales, plain.zeros))
    delta = W.double() - B @ A - (s * (fbq.unpack_codes(plain).view(N, K // 128, 128) - z)).view(N, K)
    P = delta @ H
    want_A, want_B = -2 * (B.T.contiguous() @ P), -2 * (P @ A.T.contiguous())
    for got, want in ((st.grad_At, want_A), (st.grad_Bt, want_B)):
        assert float((got.double() - want).norm() / want.norm()) < 2e-3


@pytest.mark.parametrize("bits,N,r,near", [(4, 4, 256, False), (3, 4, 72, True), (4, 3, 8, True), (3, 5, 136, False), (4, 4, 64, True)])
def test_delta_is_the_fp16_number_of_64_bits(bits, N, r, near):
    """With an H of one diagonal entry the loss is the sum over the rows of one feature's Delta_F squared, and so shows fp16(256 Delta_F).  The next
    fp16 number in one of the rows moves the sum by 2^-10 of that row's square; the sum of N fp32 products is within N 2^-23 of itself, and
    H's 2^-10 is exact.  Also with weights near the branch's product, where Delta_F is small beside what the 32-bit sums add up."""
    K, gain, scale = 128, 256.0, 2.0**-10
    g = torch.Generator(device="cuda")
    g.manual_seed(10 * r + N)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    At, Bt = rand(r, K) * 0.1, rand(N, r) * 0.1
    A, B = At.half().double(), Bt.half().double()
    W = ((B @ A).float() + 0.02 * rand(N, K)).half() if near else (rand(N, K) * 0.1).half()
    d = fbq.Desc(N, K, r, bits)
    st = fbq.train_state(d, At.clone(), Bt.clone())
    losses = []
    for k in range(K):
        H16 = torch.zeros(K, K, dtype=torch.float16, device="cuda")
        H16[k, k] = 1.0
        fbq.train_step(st, W, H16, scale, 0.0, want_loss=True)
        losses.append(st.loss.clone())
    losses = torch.cat(losses).double() * scale
    s, z = (t.view(torch.float16).double() for t in (st.layer.scales, st.layer.zeros))
    delta = (W.double() - B @ A) - s * (fbq.unpack_codes(st.layer).double() - z)
    want = ((delta * gain).float().half().double() / gain).square().sum(0)
    miss = (losses - want).abs() / want
    assert float(miss.max()) <= N * 2.0**-23, (float(miss.max()), int((miss > N * 2.0**-23).sum()))


@pytest.mark.parametrize("K,T", [(128, 1), (256, 63), (1408, 65), (384, 1000), (4224, 129)])
def test_gram_of_turned_reads_is_exact_on_whole_numbers(K, T):
    """Small whole numbers: every sum is exact, so H is, whatever the order.  Tiles past the last feature, steps past the last token, contractions split
    over blocks; and H written over the activations themselves."""
    g = torch.Generator(device="cuda")
    g.manual_seed(K + T)
    X = torch.randint(-3, 4, (T, K), device="cuda", generator=g).half()
    want = (X.double().T.contiguous() @ X.double() / 16).half()
    d = fbq.Desc(128, K, 8, 4)
    assert torch.equal(fbq.gram(d, X, 1.0 / 16), want)
    both = torch.full((max(T, K) * K,), float("nan"), dtype=torch.float16, device="cuda")
    both[: T * K] = X.flatten()
    ws = torch.empty(fbq.train_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    rc = fbq.load().fbq_gram(ctypes.byref(d.c()), T, both.data_ptr(), 1.0 / 16, both.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(both[: K * K].view(K, K), want)


@pytest.mark.parametrize("bits,r", [(4, 64), (3, 24), (4, 128), (3, 200)])
@pytest.mark.parametrize("where", ["taps", "rows of B", "both"])
def test_step_with_a_branch_near_the_end_of_fp16(bits, r, where):
    """Numbers that the split of the 32-bit sums has no room for (from 59360 on, and infinities) go to 64 bits as they are: codes, scales and zeros are those of
    the quantizer by itself, and Delta_F is finite where the branch is (fp16 roundings of the gradient of B as above: 2e-3)."""
    N, K, scale = 48, 384, 2.0**-10
    g = torch.Generator(device="cuda")
    g.manual_seed(r)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    W, At, Bt = (rand(N, K) * 0.02).half(), rand(r, K) * 3e-4, rand(N, r) * 0.01    # (256 Delta_F stays an fp16 number)
    if where != "rows of B":
        At[2, 7], At[1, 140] = 60000.0, -65504.0
        At[3, 260], At[4, 261], At[5, 262] = float("inf"), float("nan"), 2048.0    # (the third group's taps)
    if where != "taps":
        Bt[3, 5], Bt[4, 0], Bt[7, 2], Bt[40] = 60000.0, -65504.0, 3000.0, 59500.0
        Bt[9, 1], Bt[10, 4] = float("inf"), float("nan")
    d = fbq.Desc(N, K, r, bits)
    H16 = torch.eye(K, device="cuda").half() * scale
    st = fbq.train_state(d, At.clone(), Bt.clone())
    fbq.train_step(st, W, H16, scale, 0.0, want_loss=False)
    plain = fbq.quantize_feedback(d, W, At.half().view(torch.int16), Bt.half().view(torch.int16))
    for a, b in ((st.layer.qweight, plain.qweight), (st.layer.scales, plain.scales), (st.layer.zeros, plain.zeros)):
        assert torch.equal(a, b)
    if where == "rows of B":
        A, B = At.half().double(), Bt.half().double()
        s, z = (t.view(torch.float16).double()[:, :, None] for t in (plain.scales, plain.zeros))
        delta = W.double() - B @ A - (s * (fbq.unpack_codes(plain).view(N, K // 128, 128) - z)).view(N, K)
        rows = [n for n in range(N) if n not in (9, 10)]
        want = -2 * (delta @ A.T.contiguous())[rows]
        assert float((st.grad_Bt.double()[rows] - want).norm() / want.norm()) < 2e-3


def stored_delta(st):
    """fp16(256 Delta_F) of a state's last step, as the quantizer left it in the workspace: behind B^T with rows padded to 64."""
    N, K, r = st.desc.N, st.desc.K, st.desc.r
    at = (r * (-(-N // 64) * 64) * 2 + 255) // 256 * 256
    return st.workspace[at:at + N * K * 2].view(torch.float16).view(N, K)


@pytest.mark.parametrize("bits,N,K,r,kind", [
    # blocks that all start at once, which go to 64 bits as they are: whole tiles and not, ranks of each class
    (4, 100, 512, 64, "near"), (3, 63, 128, 200, "plain"), (4, 33, 256, 72, "offset"), (3, 4096, 512, 8, "plain"),
    # one block more: one tile a block; two tiles a block; blocks of eight waves and two tiles
    (4, 4097, 512, 64, "plain"), (3, 4097, 512, 40, "offset"), (4, 4100, 512, 128, "one size"), (3, 4100, 512, 72, "near"), (4, 4097, 512, 200, "ties"),
    (3, 4100, 4096, 64, "ties"), (4, 4100, 4096, 24, "near"), (4, 4100, 4096, 200, "plain"), (3, 4100, 4096, 136, "near"), (3, 4100, 4096, 136, "offset")])
def test_every_element_of_delta_is_that_of_64_bits(bits, N, K, r, kind):
    """Rows that 32 bits decide, that they leave open one by one, and that are open nearly all: far from zero, on half steps, with taps all of one size (r = 128: their
    whole parts have no room), and weights near the branch's product (more than 128 pairs of elements open in a wave's tile).  Every word of the layer is that of the quantizer by itself,
    and every stored element the fp16 number of 64 bits, by way of fp32 as the kernel rounds it."""
    g = torch.Generator(device="cuda")
    g.manual_seed(17 * r + N)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    At, Bt, W = rand(r, K) * 0.01, rand(N, r) * 0.01, rand(N, K) * 0.02
    if kind == "offset":
        W = 4 + torch.randint(0, 4, (N, K), device="cuda", generator=g) * 2.0**-8
    elif kind == "one size":
        At = torch.sign(At) * 0.0149
    elif kind == "ties":
        W = torch.randint(0, 2 * (2**bits - 1) + 1, (N, K), device="cuda", generator=g) / 2.0
        W[:, ::128], W[:, 1::128] = 0.0, 2.0**bits - 1
        Bt = Bt * 0
    elif kind == "near":
        At, Bt = At * 30, Bt * 30
        W = Bt.half().float() @ At.half().float() + 0.02 * W
    W = W.half()
    d = fbq.Desc(N, K, r, bits)
    st = fbq.train_state(d, At.clone(), Bt.clone())
    H16 = torch.zeros(K, K, dtype=torch.float16, device="cuda")
    fbq.train_step(st, W, H16, 1.0, 0.0, want_loss=False)
    plain = fbq.quantize_feedback(d, W, At.half().view(torch.int16), Bt.half().view(torch.int16))
    for a, b in ((st.layer.qweight, plain.qweight), (st.layer.scales, plain.scales), (st.layer.zeros, plain.zeros)):
        assert torch.equal(a, b)
    s, z = (t.view(torch.float16).double()[:, :, None] for t in (plain.scales, plain.zeros))
    R = W.double() - Bt.half().double() @ At.half().double()
    want = (256.0 * (R.view(N, K // 128, 128) - s * (fbq.unpack_codes(plain).view(N, K // 128, 128) - z))).view(N, K).float().half()
    off = stored_delta(st) != want
    assert not bool(off.any()), (int(off.sum()), off.nonzero()[:5].tolist())


@pytest.mark.parametrize("bits,N,K,r", [(4, 1000, 1024, 64), (3, 65, 384, 200), (4, 4100, 512, 8), (3, 300, 4096, 128)])
def test_step_stays_inside_the_workspace_asked_for(bits, N, K, r):
    """A workspace of exactly that size, between guard bytes, holds all that a step writes; a larger one gives the same bits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(23 + N)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g)
    d, W, At, Bt = fbq.Desc(N, K, r, bits), (rand(N, K) * 0.02).half(), rand(r, K) * 0.01, rand(N, r) * 0.01
    H16 = fbq.gram(d, rand(300, K).half(), 1.0 / 256)
    need, guard = fbq.train_workspace_bytes(d, 1), 4096
    results = []
    for room in (need, 2 * need):
        st = fbq.train_state(d, At.clone(), Bt.clone())
        whole = torch.full((room + 2 * guard,), 0xA5, dtype=torch.uint8, device="cuda")
        st.workspace = whole[guard:guard + room]
        fbq.train_step(st, W, H16, 1.0 / 256, 1e-4)
        assert bool((whole[:guard] == 0xA5).all()) and bool((whole[guard + need:] == 0xA5).all())
        results.append([st.layer.qweight, st.layer.scales, st.layer.zeros, st.grad_At, st.grad_Bt, st.At32, st.Bt32, st.loss])
    assert all(torch.equal(a, b) for a, b in zip(*results))
    st.workspace = whole[guard:guard + need - 1]
    with pytest.raises(fbq.FbqError, match="workspace"):
        fbq.train_step(st, W, H16, 1.0 / 256, 1e-4)


def test_gram_over_its_activations_in_a_replayed_graph():
    """H written over X goes by way of a copy of X, also in a captured graph: every replay on new activations gives what an eager call gives, with eager work in between."""
    K, T = 384, 1000
    g = torch.Generator(device="cuda")
    g.manual_seed(29)
    d = fbq.Desc(128, K, 8, 4)
    both = torch.zeros(T * K, dtype=torch.float16, device="cuda")
    ws = torch.empty(fbq.train_workspace_bytes(d, T), dtype=torch.uint8, device="cuda")
    call = lambda: fbq.load().fbq_gram(ctypes.byref(d.c()), T, both.data_ptr(), 1.0 / 16, both.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert call() == 0
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert call() == 0
    for _ in range(4):
        X = torch.randint(-3, 4, (T, K), device="cuda", generator=g).half()
        want = fbq.gram(d, X, 1.0 / 16)
        both.copy_(X.flatten())
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(both[: K * K].view(K, K), want)
