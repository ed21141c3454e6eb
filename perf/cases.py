"""The calls a private training loop makes to this library, as measurable cases.

A user has, per layer, the inputs A[B, T, d_in] and the back-propagated gradients G[B, T, d_out] on the GPU and wants
the per-example squared norms, the clip factors and the clipped gradient sums (noise, biases and LayerNorm parameters
where the model has them).  Three ways to ask for that:

  "step"   dp.layers_step: the whole model in one call;
  "block"  dp.layers_sqnorm with bias rows, dp.layernorm_sqnorm, dp.clip_factors, dp.layers_clipped_grad and
           dp.clipped_bias_grad: a model with biases and LayerNorm parameters;
  "image"  dp.conv_sqnorm, dp.bias_sqnorm, dp.clip_factors, dp.conv_clipped_grad, dp.clipped_bias_grad and
           dp.add_noise: a convolution layer given by its input image.

A case is a dict of plain values.  "layers" is a text, one "T:d_inxd_out" per layer ("*n" repeats it).
"""
from __future__ import annotations

import math

import torch

from paper_2009_03106_amd import dpclip as dp

# storage types of (A, G)
TYPES = {
    "f32": (torch.float32, torch.float32),
    "bf16": (torch.bfloat16, torch.bfloat16),
    "f16": (torch.float16, torch.float16),
    "f8": (torch.float8_e4m3fn, torch.float8_e5m2),      # 8-bit training: e4m3 activations, e5m2 gradients
}

STACK_32 = ("1024:27x64 1024:576x64*4 256:576x128 256:1152x128*3 64:1152x256 64:2304x256*3 "
            "16:2304x512 16:4608x512*3 1:512x10")


def listed():
    return [
        # the smallest call: one dense layer and a small batch, where launches and the host's call rate count
        {"name": "dense_f32", "way": "step", "B": 32, "dtype": "f32", "layers": "1:64x32",
         "dist": "normal", "g_std": 0.1, "C": 1.0, "noise": 0.0},
        # a three-layer perceptron on 28 x 28 images at an ordinary batch, float32 as the paper ran it
        {"name": "mlp_f32", "way": "step", "B": 256, "dtype": "f32", "layers": "1:784x512 1:512x256 1:256x10",
         "dist": "relu", "g_std": 0.01, "C": 1.0, "noise": 0.0},
        # the same model at the large batches private training prefers
        {"name": "mlp_f32_large_batch", "way": "step", "B": 65536, "dtype": "f32",
         "layers": "1:784x512 1:512x256 1:256x10", "dist": "relu", "g_std": 0.01, "C": 1.0, "noise": 0.0},
        # a recurrent layer: one linear map shared by 64 time steps
        {"name": "rnn_bf16", "way": "step", "B": 128, "dtype": "bf16", "layers": "64:256x256",
         "dist": "tanh", "g_std": 0.01, "C": 0.5, "noise": 0.0},
        # a 3 x 3 convolution, 64 -> 128 channels on 32 x 32 inputs, whose patches the caller has unfolded
        {"name": "conv_unfolded_bf16", "way": "step", "B": 128, "dtype": "bf16", "layers": "1024:576x128",
         "dist": "relu", "g_std": 0.001, "C": 1.0, "noise": 0.0},
        # the same convolution given by its image, with its bias and noise of the paper's default sigma
        {"name": "conv_image_bf16", "way": "image", "B": 128, "dtype": "bf16", "H": 32, "W": 32, "channels": 64,
         "K": 3, "pad": 1, "d_out": 128, "dist": "relu", "g_std": 0.001, "C": 1.0, "noise": 0.05},
        # the linears of a transformer block (QKV, attention output, both feed-forward maps) with noise of sigma = C
        {"name": "transformer_bf16", "way": "step", "B": 64, "dtype": "bf16",
         "layers": "512:768x2304 512:768x768 512:768x3072 512:3072x768", "dist": "normal", "g_std": 0.001, "C": 1.0,
         "noise": 1.0},
        # the same with 8-bit activations and gradients, under a loss scale of 1000
        {"name": "transformer_f8", "way": "step", "B": 64, "dtype": "f8",
         "layers": "512:768x2304 512:768x768 512:768x3072 512:3072x768", "dist": "normal", "g_std": 1.0, "C": 1000.0,
         "noise": 0.0},
        # the same in float32, the precision of the paper's experiments: the largest case
        {"name": "transformer_f32", "way": "step", "B": 64, "dtype": "f32",
         "layers": "512:768x2304 512:768x768 512:768x3072 512:3072x768", "dist": "normal", "g_std": 0.001, "C": 1.0,
         "noise": 0.0},
        # an image model of 18 unfolded convolutions on 32 x 32 inputs at the paper's batch of 32: many layers of very
        # different shapes, each too small for the chip, the first with 27 (unaligned) patch columns
        {"name": "image_stack_bf16", "way": "step", "B": 32, "dtype": "bf16", "layers": STACK_32,
         "dist": "relu", "g_std": 0.001, "C": 1.0, "noise": 0.05},
        # the same in float32
        {"name": "image_stack_f32", "way": "step", "B": 32, "dtype": "f32", "layers": STACK_32,
         "dist": "relu", "g_std": 0.001, "C": 1.0, "noise": 0.05},
        # one encoder block over 200-wide word vectors with a two-way head, ragged sequence length, float16 gradients
        # under a loss scale, biases and two LayerNorms: every call of a model with all parameter kinds
        {"name": "encoder_f16_biases", "way": "block", "B": 32, "dtype": "f16",
         "layers": "250:200x600 250:200x200 250:200x512 250:512x200 1:200x2", "norms": "250:200*2",
         "dist": "normal", "g_std": 0.5, "C": 512.0, "noise": 25.6},
    ]


def layer_sizes(text):
    """[(T, d_in, d_out), ...] of a case's "layers"; [(T, d), ...] of its "norms"."""
    out = []
    for item in text.split():
        body, _, times = item.partition("*")
        T, _, sizes = body.partition(":")
        out += [(int(T), *(int(v) for v in sizes.split("x")))] * (int(times) if times else 1)
    return out


def _out_positions(case):
    return (case["H"] + 2 * case["pad"] - case["K"] + 1) * (case["W"] + 2 * case["pad"] - case["K"] + 1)


def work(case):
    """Bytes (every input read once, every output written once) and operations of one pass: the cheaper of the two
    norms' forms and the clipped sum."""
    ea, eg = (torch.empty(0, dtype=t).element_size() for t in TYPES[case["dtype"]])
    B = case["B"]
    if case["way"] == "image":
        T, d_in, d_out = _out_positions(case), case["K"] ** 2 * case["channels"], case["d_out"]
        byts = B * (case["H"] * case["W"] * case["channels"] * ea + T * d_out * eg) + 4 * (d_in * d_out + d_out) + 8 * B
        return {"bytes": byts + 4 * B * d_out, "flops": 4 * B * T * d_in * d_out + 3 * B * T * d_out}
    byts, flops = 8 * B, 0
    biases = case["way"] == "block"
    for T, d_in, d_out in layer_sizes(case["layers"]):
        byts += B * T * (d_in * ea + d_out * eg) + 4 * d_in * d_out + (4 * d_out + 4 * B * d_out if biases else 0)
        direct, gram = 2 * T * d_in * d_out, T * (T + 1) * (d_in + d_out)
        norm = 2 * (d_in + d_out) if T == 1 else min(direct, gram)
        flops += B * (norm + direct + (T * d_out + 4 * d_out if biases else 0))
    for T, d in layer_sizes(case.get("norms", "")):
        byts += B * T * d * (ea + eg) + 8 * d + 8 * B * d
        flops += B * (3 * T * d + 8 * d)
    return {"bytes": byts, "flops": flops}


# Rough rates of the device (operations and bytes per second) that a drawn case's cost is held against.
_OPS = {"f32": 1e14, "bf16": 5e14, "f16": 5e14, "f8": 7e14}
_BYTES = 3e12


def _cost(case):
    w = work(case)
    return w["flops"] / _OPS[case["dtype"]] + w["bytes"] / _BYTES


def _log_int(rng, lo, hi):
    """Whole number between lo and hi, evenly spread over the logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _width(rng, lo, hi, aligned):
    """A layer width: usually a multiple of 8 or 64, as models have them, sometimes any number."""
    n = _log_int(rng, lo, hi)
    step = rng.choice((8, 64) if aligned else (1, 4, 8, 64))
    return max(step, n // step * step)


def draw(rng):
    kind = rng.choice(("dense", "dense", "sequence", "sequence", "sequence", "convolutions", "image", "block"))
    if kind == "dense":                      # perceptrons of 1 to 6 layers, batches from 16 to 65536
        dtype = rng.choice(("f32", "f32", "f32", "bf16"))
        sizes = [_width(rng, 32, 1024, False) for _ in range(rng.randint(1, 6))] + [rng.choice((2, 10, 32, 100, 256))]
        layers = " ".join(f"1:{a}x{b}" for a, b in zip(sizes, sizes[1:]))
        case = {"way": "step", "B": _log_int(rng, 16, 65536), "dtype": dtype, "layers": layers, "dist": "relu",
                "g_std": 0.01, "C": 1.0, "noise": rng.choice((0.0, 0.05))}
    elif kind == "sequence":                 # recurrent and attention linears
        dtype = rng.choice(("f32", "bf16", "bf16", "f16", "f8"))
        T = rng.choice((_log_int(rng, 16, 1024), 64 * rng.randint(1, 10)))
        layers = " ".join(f"{T}:{_width(rng, 64, 3072, dtype == 'f8')}x{_width(rng, 64, 3072, dtype == 'f8')}"
                          for _ in range(rng.randint(1, 4)))
        case = {"way": "step", "B": _log_int(rng, 4, 128), "dtype": dtype, "layers": layers,
                "dist": rng.choice(("normal", "tanh")), "g_std": 0.001, "C": 1.0, "noise": 0.0}
    elif kind == "convolutions":             # stacks of unfolded convolutions: the image halves as the channels double
        dtype = rng.choice(("f32", "bf16", "bf16"))
        side, ch, taps = rng.choice((14, 16, 28, 32, 56, 64)), rng.choice((16, 32, 48, 64)), 9
        items, d = [], 3 * rng.choice((9, 25))
        for _ in range(rng.randint(1, 4)):
            items.append(f"{side * side}:{d}x{ch}")
            items += [f"{side * side}:{taps * ch}x{ch}"] * rng.randint(0, 2)
            side, d, ch = max(4, side // 2), taps * ch, min(512, 2 * ch)
        case = {"way": "step", "B": _log_int(rng, 8, 128), "dtype": dtype, "layers": " ".join(items), "dist": "relu",
                "g_std": 0.001, "C": 1.0, "noise": 0.05}
    elif kind == "image":                    # 3 x 3 convolutions from the image
        side = rng.choice((8, 14, 16, 28, 32, 56))
        case = {"way": "image", "B": _log_int(rng, 8, 256), "dtype": rng.choice(("bf16", "bf16", "f16", "f8")),
                "H": side, "W": side, "channels": 64 * rng.randint(1, 4), "K": 3, "pad": 1,
                "d_out": 64 * rng.randint(1, 4), "dist": "relu", "g_std": 0.001, "C": 1.0, "noise": 0.05}
    else:                                    # encoder blocks with biases and LayerNorms
        dtype = rng.choice(("f32", "bf16", "f16"))
        T, d = _log_int(rng, 16, 640), _width(rng, 100, 1024, False)
        f = _width(rng, 128, 3072, False)
        case = {"way": "block", "B": _log_int(rng, 4, 128), "dtype": dtype,
                "layers": f"{T}:{d}x{3 * d} {T}:{d}x{d} {T}:{d}x{f} {T}:{f}x{d} 1:{d}x{rng.choice((2, 10))}",
                "norms": f"{T}:{d}*2", "dist": "normal", "g_std": 0.001, "C": 1.0, "noise": 0.0}
    if case["dtype"] in ("f16", "f8"):       # the narrow formats come with a loss scale
        case.update({k: case[k] * 512.0 for k in ("g_std", "C", "noise")})
    while case["B"] > 1 and _cost(case) > 0.25 * max(_cost(c) for c in listed()):
        case["B"] = max(1, case["B"] * 2 // 3)
    return case


def _values(gen, shape, dist, std, dtype):
    x = torch.randn(shape, device="cuda", dtype=torch.float32, generator=gen)
    if dist == "relu":
        x.clamp_(min=0.0)
    elif dist == "tanh":
        x.tanh_()
    if std != 1.0:
        x.mul_(std)
    return x.to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ta, tg = TYPES[case["dtype"]]
    B = case["B"]
    # the examples' gradients differ in size: most exceed the threshold and some do not
    spread = torch.exp(torch.empty(B, device="cuda").uniform_(math.log(0.01), math.log(2.0), generator=gen))

    def gradient(*shape):
        g = _values(gen, shape, "normal", case["g_std"], torch.float32)
        return g.mul_(spread.view(B, *([1] * (len(shape) - 1)))).to(tg)

    def zeros(*shape):
        return torch.zeros(shape, device="cuda", dtype=torch.float32)

    st = {"way": case["way"], "C": case["C"], "noise": case["noise"], "seed": seed & 0xFFFF,
          "sqnorm": zeros(B), "clip": zeros(B)}
    if case["way"] == "image":
        H, W, ch, K, pad, d_out = (case[k] for k in ("H", "W", "channels", "K", "pad", "d_out"))
        st.update(X=_values(gen, (B, H, W, ch), case["dist"], 1.0, ta), G=gradient(B, _out_positions(case), d_out), K=K, pad=pad,
                  rows=zeros(B, d_out), grad=zeros(K * K * ch, d_out), grad_b=zeros(d_out))
        code = {"bf16": dp.DP_BF16, "f16": dp.DP_F16, "f8": dp.DP_F8_E4M3_E5M2}[case["dtype"]]
        need = max(dp.conv_workspace_bytes(op, B, H, W, ch, K, K, pad, d_out, code)
                   for op in (dp.DP_OP_SQNORM, dp.DP_OP_CLIPPED_GRAD))
        st["workspace"] = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
        return st
    sizes = layer_sizes(case["layers"])
    pairs = []
    for T, d_in, d_out in sizes:
        lead = (B,) if T == 1 else (B, T)
        pairs.append((_values(gen, (*lead, d_in), case["dist"], 1.0, ta), gradient(*lead, d_out)))
    # the gradients lie one after the other in the model's flat gradient, each on a 16-byte boundary as the calls ask
    flat = zeros(sum((a * b + 3) // 4 * 4 for _, a, b in sizes))
    grads, at = [], 0
    for _, d_in, d_out in sizes:
        grads.append(flat[at:at + d_in * d_out].view(d_in, d_out))
        at += (d_in * d_out + 3) // 4 * 4
    st.update(pairs=pairs, flat=flat, grads=grads)
    if case["way"] == "block":
        st["rows"] = [zeros(B, d_out) for _, _, d_out in sizes]
        st["grad_bs"] = [zeros(d_out) for _, _, d_out in sizes]
        st["descs"] = dp.layer_descs(pairs, grads, bias_rows=st["rows"], grad_bs=st["grad_bs"])
        st["norms"] = [(gradient(B, T, d), _values(gen, (B, T, d), "normal", 1.0, ta), zeros(d), zeros(d))
                       for T, d in layer_sizes(case["norms"])]
    else:
        st["descs"] = dp.layer_descs(pairs, grads)
    arr, _, code = st["descs"]
    need = max(dp.layers_workspace_bytes(arr, B, code), dp.layers_clipped_workspace_bytes(arr, B, code))
    st["workspace"] = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
    return st


def run(state):
    st = state
    sq, clip, ws = st["sqnorm"], st["clip"], st["workspace"]
    if st["way"] == "step":
        dp.layers_step(st["descs"], st["C"], sq, clip, ws, noise_std=st["noise"], seed=st["seed"])
        return {"sqnorm": sq, "clip": clip, "grads": st["grads"]}
    if st["way"] == "image":
        X, G, K, pad = st["X"], st["G"], st["K"], st["pad"]
        dp.conv_sqnorm(X, G, K, K, pad, sq, workspace=ws)
        dp.bias_sqnorm(G, sq, st["rows"], accumulate=True)
        dp.clip_factors(sq, st["C"], clip)
        dp.conv_clipped_grad(X, G, clip, K, K, pad, st["grad"], workspace=ws)
        dp.clipped_bias_grad(st["rows"], clip, st["grad_b"])
        dp.add_noise(st["grad"], st["noise"], st["seed"])
        dp.add_noise(st["grad_b"], st["noise"], st["seed"], st["grad"].numel())
        return {"sqnorm": sq, "clip": clip, "grad": st["grad"], "grad_b": st["grad_b"]}
    dp.layers_sqnorm(st["pairs"], sq, workspace=ws, descs=st["descs"])
    rows = []
    for G, Hbar, _, _ in st["norms"]:
        _, gamma, beta = dp.layernorm_sqnorm(G, Hbar, sq, accumulate=True)
        rows.append((gamma, beta))
    dp.clip_factors(sq, st["C"], clip)
    dp.layers_clipped_grad(st["pairs"], clip, st["grads"], workspace=ws, descs=st["descs"], noise_std=st["noise"],
                           seed=st["seed"])
    for (gamma, beta), (_, _, grad_gamma, grad_beta) in zip(rows, st["norms"]):
        dp.clipped_bias_grad(gamma, clip, grad_gamma)
        dp.clipped_bias_grad(beta, clip, grad_beta)
    return {"sqnorm": sq, "clip": clip, "grads": st["grads"], "grad_bs": st["grad_bs"],
            "norm_grads": [(gg, gb) for _, _, gg, gb in st["norms"]]}


def tolerance(case):
    """Four times the largest error against 64-bit arithmetic on the same inputs, over the listed and some drawn cases.

    float32 sums of exact products: 1.2e-6 (largest entry 9.5e-6) over 32768 float32 rows, 4e-7 (2e-6) for 16-bit
    inputs, whose terms are fewer bits long, and 1.5e-5 (7e-5) for the 8-bit matrix instruction.  Layers that are small
    or not whole blocks of 32 rows and 64 columns may have the clip factor multiplied into the 16-bit rows, which rounds
    them once more: 1.7e-3 (7.7e-3) for bfloat16, an eighth of that for float16 (which 8-bit inputs of such shapes are
    widened to)."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 4e-5}
    whole = case["way"] == "image" or all(T % 32 == 0 and a % 64 == 0 and b % 64 == 0 and a * b >= 1 << 16
                                          for T, a, b in layer_sizes(case["layers"]))
    if whole:
        return {"rel": 6e-5, "max": 3e-4} if case["dtype"] == "f8" else {"rel": 2e-6, "max": 1e-5}
    return {"rel": 7e-3, "max": 3e-2} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 4e-3}
