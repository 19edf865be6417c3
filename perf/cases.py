"""Performance cases of the library: what a program that serves or prepares FBQuant layers has it do.

listed() names the cases, draw() gives further ones of the same ranges, prepare() makes inputs and whatever a program
keeps between calls (quantized layers, workspaces, output buffers, a captured decode step), run() is one pass through
the public entry points, exact() the same quantities in 64 bits from plain torch, work() the bytes and operations one
pass cannot do without, tolerance() what rounding at the data types' precision accounts for.

Kinds of case
  linear    one sub-branched quantized linear layer on M tokens (fbq.linear; y and workspace are kept by the caller)
  stack     one step of a decoder stack of quantized linears (decode_loop.DecoderStack, a captured HIP graph):
            grouped q/k/v and gate/up launches, `batch` sequences decoded together
  quantize  the feedback quantizer Q(W - B A) of one weight matrix (fbq.quantize_feedback)
  train     one iteration of the layer-wise reconstruction (fbq.train_step), with or without the loss
  gram      H = X^T X of a calibration set (fbq.gram)
"""
from __future__ import annotations

import math

import torch

import paper_2501_16385_amd as fbq
from paper_2501_16385_amd import decode_loop

GROUP = 128


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # one token through one attention projection, called eagerly: the smallest call, where launch and call overhead count
        {"name": "linear_m1_4096x4096_i4", "kind": "linear", "N": 4096, "K": 4096, "r": 32, "bits": 4, "M": 1},
        # token-by-token generation, one sequence: Llama2-7B-shaped decoder layers, four grouped launches per layer
        {"name": "stack_b1_7b_i4", "kind": "stack", "hidden": 4096, "inter": 11008, "layers": 4, "r": 64, "bits": 4, "batch": 1},
        # the same with eight sequences decoded together, INT3
        {"name": "stack_b8_7b_i3", "kind": "stack", "hidden": 4096, "inter": 11008, "layers": 4, "r": 64, "bits": 3, "batch": 8},
        # sixteen sequences through the largest layer of the large-layer sweep (up-projection of a 70B-shaped MLP)
        {"name": "linear_m16_28672x8192_i4", "kind": "linear", "N": 28672, "K": 8192, "r": 128, "bits": 4, "M": 16},
        # a few dozen sequences, or a short prompt, through a 13B-shaped MLP layer with a long K, INT3
        {"name": "linear_m48_5120x13824_i3", "kind": "linear", "N": 5120, "K": 13824, "r": 128, "bits": 3, "M": 48},
        # prompt pass, medium: 256 tokens down a 70B-shaped MLP, INT3
        {"name": "linear_m256_8192x28672_i3", "kind": "linear", "N": 8192, "K": 28672, "r": 128, "bits": 3, "M": 256},
        # prompt pass of a ragged batch: odd token count, a row count that is no multiple of a tile, an odd number of groups
        {"name": "linear_m777_5001x4224_i4", "kind": "linear", "N": 5001, "K": 4224, "r": 40, "bits": 4, "M": 777},
        # prompt pass of the 7B-shaped MLP at 1024 tokens
        {"name": "linear_m1024_11008x4096_i4", "kind": "linear", "N": 11008, "K": 4096, "r": 64, "bits": 4, "M": 1024},
        # the largest call: a long prompt through a 70B-shaped MLP layer
        {"name": "linear_m2048_28672x8192_i4", "kind": "linear", "N": 28672, "K": 8192, "r": 128, "bits": 4, "M": 2048},
        # preparing a checkpoint: the feedback quantizer on an MLP weight, INT3
        {"name": "quantize_11008x4096_i3", "kind": "quantize", "N": 11008, "K": 4096, "r": 64, "bits": 3},
        # one iteration of the reconstruction on an attention projection, loss reported (the loop's default)
        {"name": "train_4096x4096_i4_loss", "kind": "train", "N": 4096, "K": 4096, "r": 64, "bits": 4, "T": 2048, "loss": True},
        # second moments of the calibration activations of an attention projection
        {"name": "gram_4096_t2048", "kind": "gram", "N": 4096, "K": 4096, "r": 64, "bits": 4, "T": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rank(rng):
    return rng.choice([8, 16, 32, 40, 64, 64, 96, 128, 128, 200])


def draw(rng):
    kind = rng.choices(["linear", "stack", "quantize", "train", "gram"], [10, 3, 2, 3, 1])[0]
    bits = rng.choice([3, 4])
    if kind == "stack":
        hidden = GROUP * _log_int(rng, 8, 64)
        return {"kind": kind, "hidden": hidden, "inter": GROUP * max(8, int(hidden / GROUP * rng.uniform(2.0, 3.5))),
                "layers": rng.randint(1, 3), "r": _rank(rng), "bits": bits, "batch": _log_int(rng, 1, 16)}
    if kind == "linear":
        while True:
            M, N, K = _log_int(rng, 1, 2048), _log_int(rng, 500, 28672), GROUP * _log_int(rng, 8, 224)
            if rng.random() < 0.5:
                N = GROUP * max(1, N // GROUP)
            if N * K <= 28672 * 8192:
                return {"kind": kind, "N": N, "K": K, "r": rng.choice([0, _rank(rng), _rank(rng), _rank(rng)]), "bits": bits, "M": M}
    while True:                                         # 64-bit checks multiply N x K x K or K x K x T: keep that to the 7B shapes
        N, K, T = _log_int(rng, 1000, 14000), GROUP * _log_int(rng, 8, 86), _log_int(rng, 128, 4096)
        if N * K <= 11008 * 4096:
            break
    if rng.random() < 0.5:
        N = GROUP * (N // GROUP)
    if kind == "quantize":
        return {"kind": kind, "N": N, "K": K, "r": rng.choice([0, _rank(rng), _rank(rng)]), "bits": bits}
    if kind == "train":
        return {"kind": kind, "N": N, "K": K, "r": _rank(rng), "bits": bits, "T": T, "loss": rng.random() < 0.5}
    return {"kind": kind, "N": N, "K": K, "r": _rank(rng), "bits": bits, "T": T}


# ------------------------------------------------------------------ inputs, from the seed alone

def _gen(seed, which):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + which) % (1 << 62))
    return g


def _weight(N, K, std, g):
    """Gaussian weights with one per cent of outliers ten times as large, fp16."""
    w = torch.randn(N, K, device="cuda", generator=g) * std
    w *= torch.where(torch.rand(N, K, device="cuda", generator=g) < 0.01, 10.0, 1.0)
    return w.half()


def _codes(w, bits):
    """Group-wise asymmetric round-to-nearest codes of w (a layer as a checkpoint would hold it): q uint8, s and z fp16."""
    N, K = w.shape
    qmax = 2**bits - 1
    g = w.view(N, K // GROUP, GROUP).float()
    mn, mx = g.amin(2), g.amax(2)
    s = ((mx - mn) / qmax).clamp_min(6.2e-5).half()
    z = (-mn / s.float()).half()
    q = torch.round(g / s.float()[:, :, None] + z.float()[:, :, None]).clamp_(0, qmax).to(torch.uint8)
    return q.view(N, K), s, z


def _packed(q, bits):
    """Codes [N, K] in the layout that include/fbq.h states, as int32 words."""
    N, K = q.shape
    if bits == 4:
        f = q.view(N, K // 8, 8).to(torch.int32)
        w = torch.zeros(N, K // 8, dtype=torch.int32, device=q.device)
        for i in range(8):
            w |= f[:, :, i] << (4 * i)
        return w
    u = q.view(N, K // 32, 32).to(torch.int32)
    w = torch.zeros(N, K // 32, 3, dtype=torch.int32, device=q.device)
    for word in range(3):
        for f in range(10):
            w[:, :, word] |= u[:, :, 10 * word + f] << (3 * f if f < 5 else 16 + 3 * (f - 5))
        w[:, :, word] |= ((u[:, :, 30] >> word) & 1) << 15
        w[:, :, word] |= ((u[:, :, 31] >> word) & 1) << 31
    return w.view(N, 3 * K // 32)


def _branch(N, K, r, g):
    """The sub-branch: A^T [r, K] and B^T [N, r] ~ N(0, 0.01^2), fp16."""
    if r == 0:
        return None, None
    return ((torch.randn(r, K, device="cuda", generator=g) * 0.01).half(),
            (torch.randn(N, r, device="cuda", generator=g) * 0.01).half())


def _quantized(N, K, r, bits, std, g):
    """Canonical tensors of one quantized layer: codes, s, z, A^T, B^T."""
    q, s, z = _codes(_weight(N, K, std, g), bits)
    return (q, s, z) + _branch(N, K, r, g)


def _device_layer(N, K, r, bits, tensors):
    q, s, z, At, Bt = tensors
    raw = lambda t: None if t is None else t.view(torch.int16)
    return fbq.DeviceLayer(fbq.Desc(N, K, r, bits), _packed(q, bits), raw(s), raw(z), raw(At), raw(Bt))


def _effective(tensors):
    """W_F = s (q - z) + B A in 64 bits."""
    q, s, z, At, Bt = tensors
    N, K = q.shape
    w = (q.view(N, K // GROUP, GROUP).double() - z.double()[:, :, None]) * s.double()[:, :, None]
    w = w.view(N, K)
    return w if At is None else w.addmm_(Bt.double(), At.double())


def _linear_inputs(c, seed):
    return (_quantized(c["N"], c["K"], c["r"], c["bits"], 0.02, _gen(seed, 0)),
            torch.randn(c["M"], c["K"], device="cuda", generator=_gen(seed, 1)).half())


def _stack_inputs(c, seed):
    """Per decoder layer the seven linears, scaled so that activations keep their size through the stack; and the input rows."""
    shapes = decode_loop.layer_shapes(c["hidden"], c["inter"])
    layers = []
    for i in range(c["layers"]):
        g = _gen(seed, 10 + i)
        layers.append({n: _quantized(N, K, c["r"], c["bits"], 0.35 / math.sqrt(K), g) for n, (N, K) in shapes.items()})
    return layers, torch.randn(c["batch"], c["hidden"], device="cuda", generator=_gen(seed, 1)).half()


def _calibration(K, T, g):
    """Calibration activations with channels of different size, fp16."""
    scale = torch.exp(0.5 * torch.randn(K, device="cuda", generator=g)).clamp_(0.1, 4.0)
    return (torch.randn(T, K, device="cuda", generator=g) * scale).half()


def _train_inputs(c, seed):
    """A reconstruction in progress: W, H = X^T X / T as the loop keeps it, and the fp32 masters."""
    N, K, r = c["N"], c["K"], c["r"]
    g = _gen(seed, 0)
    W, X = _weight(N, K, 0.02, g), _calibration(K, c["T"], g).float()
    H16 = ((X.T.contiguous() @ X) / c["T"]).half()
    At, Bt = torch.randn(r, K, device="cuda", generator=g) * 0.01, torch.randn(N, r, device="cuda", generator=g) * 0.01
    return W, H16, At, Bt


def _h_scale(c):
    return 1.0 / c["T"]


def _learning_rate(c):
    """A step well inside the stable range: lambda_max(X^T X) <= 16 T (1 + sqrt(K / T))^2 for the channels above, the
    branch's squared norms about 1e-4 (sqrt(max(N, K)) + sqrt(r))^2."""
    lam = 16.0 * c["T"] * (1.0 + math.sqrt(c["K"] / c["T"])) ** 2
    return 0.02 / (lam * 1e-4 * (math.sqrt(max(c["N"], c["K"])) + math.sqrt(c["r"])) ** 2)


# ------------------------------------------------------------------ the path

def prepare(case, seed):
    c = case
    if c["kind"] == "linear":
        tensors, x = _linear_inputs(c, seed)
        layer = _device_layer(c["N"], c["K"], c["r"], c["bits"], tensors)
        need = fbq.workspace_bytes(layer.desc, c["M"])
        return {"c": c, "layer": layer, "x": x, "y": torch.empty(c["M"], c["N"], dtype=torch.float16, device="cuda"),
                "ws": torch.zeros(need, dtype=torch.uint8, device="cuda") if need else None}
    if c["kind"] == "stack":
        layers, x = _stack_inputs(c, seed)
        shapes = decode_loop.layer_shapes(c["hidden"], c["inter"])
        dev = [{n: _device_layer(shapes[n][0], shapes[n][1], c["r"], c["bits"], l[n]) for n in l} for l in layers]
        del layers
        stack = decode_loop.DecoderStack(dev, c["hidden"], c["inter"], batch=c["batch"])
        return {"c": c, "stack": stack, "graph": stack.capture(), "x": x}
    d = fbq.Desc(c["N"], c["K"], c["r"], c["bits"])
    if c["kind"] == "quantize":
        g = _gen(seed, 0)
        return {"c": c, "d": d, "W": _weight(c["N"], c["K"], 0.02, g), "branch": _branch(c["N"], c["K"], c["r"], g)}
    if c["kind"] == "train":
        W, H16, At, Bt = _train_inputs(c, seed)
        return {"c": c, "W": W, "H16": H16, "st": fbq.train_state(d, At, Bt)}
    X = _calibration(c["K"], c["T"], _gen(seed, 0))
    return {"c": c, "d": d, "X": X, "ws": torch.empty(max(256, fbq.train_workspace_bytes(d, c["T"])), dtype=torch.uint8, device="cuda")}


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "linear":
        return fbq.linear(s["layer"], s["x"], s["y"], s["ws"])
    if c["kind"] == "stack":
        s["stack"].x.copy_(s["x"])                      # the step's input rows (embeddings of the tokens just chosen)
        s["graph"].replay()
        return s["stack"].x
    if c["kind"] == "quantize":
        layer = fbq.quantize_feedback(s["d"], s["W"], *s["branch"])
        return {"qweight": layer.qweight, "scales": layer.scales.view(torch.float16), "zeros": layer.zeros.view(torch.float16)}
    if c["kind"] == "train":
        st = s["st"]
        fbq.train_step(st, s["W"], s["H16"], _h_scale(c), _learning_rate(c), want_loss=c["loss"])
        l = st.layer
        out = {"qweight": l.qweight, "scales": l.scales.view(torch.float16), "zeros": l.zeros.view(torch.float16),
               "At16": l.At.view(torch.float16), "Bt16": l.Bt.view(torch.float16), "grad_At": st.grad_At, "grad_Bt": st.grad_Bt,
               "At32": st.At32, "Bt32": st.Bt32}
        if c["loss"]:
            out["loss"] = st.loss
        return out
    return fbq.gram(s["d"], s["X"], _h_scale(c), s["ws"])


# ------------------------------------------------------------------ 64 bits

def _half64(d):
    """fp64 -> fp16, rounded once (by way of an fp32 value rounded to odd: a plain conversion may round twice)."""
    f = d.float()
    bits = f.view(torch.int32)
    bits = torch.where(f.double().abs() > d.abs(), bits - 1, bits)
    bits = torch.where(f.double() != d, bits | 1, bits)
    return bits.view(torch.float32).half()


def _quantizer64(W, sigma, bits):
    """Q(W - sigma) as the paper defines it: fp64 extremes, s and z rounded to fp16 (s stepped up until both ends of the
    range lie within half a step of the code range), codes rounded half to even.  Returns codes (fp64), s, z (fp16)."""
    N, K = W.shape
    qmax = 2**bits - 1
    R = (W.double() - sigma).view(N, K // GROUP, GROUP)
    mn, mx = R.amin(2), R.amax(2)
    s = (mx - mn) / qmax
    s16 = _half64(torch.where(s > 0, s, torch.ones_like(s))).clamp_min(2.0**-14)
    while True:
        sd = s16.double()
        z16 = _half64(-mn / sd)
        zd = z16.double()
        off = ~((mn / sd + zd >= -0.5) & (mx / sd + zd <= qmax + 0.5)) & (s16.view(torch.int16) < 0x7BFF)
        if not bool(off.any()):
            break
        s16 = torch.where(off, (s16.view(torch.int16) + 1).view(torch.float16), s16)
    q = torch.round(R / sd[:, :, None] + zd[:, :, None]).clamp_(0, qmax)
    return q.view(N, K), s16, z16


def exact(case, seed):
    c = case
    if c["kind"] == "linear":
        tensors, x = _linear_inputs(c, seed)
        return x.double() @ _effective(tensors).T
    if c["kind"] == "stack":
        layers, x = _stack_inputs(c, seed)
        x = x.double()
        for l in layers:
            lin = lambda n, v: v @ _effective(l[n]).T
            h = (x + lin("o", lin("v", x))) / 2
            x = (h + lin("down", torch.nn.functional.silu(lin("gate", h)) * lin("up", h))) / 2
        return x
    if c["kind"] == "gram":
        X = _calibration(c["K"], c["T"], _gen(seed, 0)).double()
        return X.T.contiguous() @ X * _h_scale(c)
    if c["kind"] == "quantize":
        g = _gen(seed, 0)
        W = _weight(c["N"], c["K"], 0.02, g)
        At, Bt = _branch(c["N"], c["K"], c["r"], g)
        _, s16, z16 = _quantizer64(W, 0.0 if At is None else Bt.double() @ At.double(), c["bits"])
        return {"qweight": None, "scales": s16.double(), "zeros": z16.double()}
    W, H16, At32, Bt32 = _train_inputs(c, seed)
    A, B = At32.half().double(), Bt32.half().double()
    sigma = B @ A
    q, s16, z16 = _quantizer64(W, sigma, c["bits"])
    N, K = W.shape
    D = (W.double() - sigma).view(N, K // GROUP, GROUP) - s16.double()[:, :, None] * (q.view(N, K // GROUP, GROUP) - z16.double()[:, :, None])
    D = D.view(N, K)
    H = H16.double() / _h_scale(c)
    P = D @ H
    gA, gB = -2.0 * (B.T.contiguous() @ P), -2.0 * (P @ A.T.contiguous())
    out = {"qweight": None, "scales": s16.double(), "zeros": z16.double(), "At16": A, "Bt16": B, "grad_At": gA, "grad_Bt": gB,
           "At32": At32.double() - _learning_rate(c) * gA, "Bt32": Bt32.double() - _learning_rate(c) * gB}
    if c["loss"]:
        out["loss"] = (D * P).sum().view(1)
    return out


# ------------------------------------------------------------------ work and tolerance

def _linear_work(N, K, r, bits, M, x_reads=1):
    return (N * K * bits / 8 + 4 * N * (K // GROUP) + 2 * r * (K + N) + 2 * M * (K * x_reads + N), 2 * M * N * K + 2 * M * r * (K + N))


def work(case):
    c = case
    if c["kind"] == "linear":
        b, f = _linear_work(c["N"], c["K"], c["r"], c["bits"], c["M"])
        return {"bytes": b, "flops": f}
    if c["kind"] == "stack":
        b = f = 0.0
        for N, K in decode_loop.layer_shapes(c["hidden"], c["inter"]).values():
            lb, lf = _linear_work(N, K, c["r"], c["bits"], c["batch"])
            b, f = b + lb, f + lf
        return {"bytes": c["layers"] * b, "flops": c["layers"] * f}
    N, K, r = c["N"], c["K"], c["r"]
    if c["kind"] == "gram":                             # H is symmetric: one triangle determines it
        return {"bytes": 2 * c["T"] * K + 2 * K * K, "flops": c["T"] * K * (K + 1)}
    layer_bytes = N * K * c["bits"] / 8 + 4 * N * (K // GROUP)
    if c["kind"] == "quantize":
        return {"bytes": 2 * N * K + 2 * r * (N + K) + layer_bytes, "flops": 2 * N * K * r}
    # train: W and H in, masters in and out, the layer, its fp16 branch and the gradients out; B A, B^T D, (B^T D) H, A H, D (A H)^T,
    # and for the loss tr(D H D^T) one triangle of the symmetric H
    return {"bytes": 2 * N * K + 2 * K * K + r * (N + K) * (4 + 4 + 2 + 4) + layer_bytes,
            "flops": 6 * N * K * r + 4 * r * K * K + (N * K * (K + 1) if c["loss"] else 0)}


def tolerance(case):
    c = case
    if c["kind"] == "quantize":                         # codes, scales and zeros are defined in 64 bits
        return "exact"
    if c["kind"] == "linear":
        # y is fp16 (2.1e-4 against 64 bits); with more tokens the weights meet the matrix cores rounded to fp16 as well (2.9e-4)
        return {"rel": 1.2e-3 if c["M"] > 16 else 8.5e-4, "max": 2e-2}
    if c["kind"] == "stack":
        return {"rel": 2.4e-3, "max": 5e-2}      # (6e-4 against 64 bits, every layer rounded to fp16)
    if c["kind"] == "gram":                             # fp16 of a 32-bit sum
        return {"rel": 8.5e-4, "max": 5e-3}
    # Delta, H and their products with the branch enter the matrix cores as fp16: gradients are a few 1e-4 off; a second
    # iteration starts from masters that moved by them, so an fp16 rounding of a master, and with it a code, may differ
    return {"rel": 1.2e-3, "max": 5e-2, "differ": 1e-3}
