"""The float32 kernels that run on the bf16 matrix instruction with every operand split into three bf16 numbers
(long clipped sums, direct norms, Gram norms): tile edges, remainders, and the values the three parts cannot carry."""
import numpy as np
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu

# A float32 sum of K terms in any order is within about K 2^-24 of the sum of absolute values; for terms of random sign
# the 2-norm error is a few sqrt(K) 2^-24 / sqrt(K) = a few 2^-24 of the result's.  1e-6 is 17 units of 2^-24.
REL = 1e-6


def _data(B, T, d_in, d_out, seed, scale=1.0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn((B, T, d_in), device="cuda", generator=gen)
    G = torch.randn((B, T, d_out), device="cuda", generator=gen) * scale
    clip = torch.rand(B, device="cuda", generator=gen) + 0.25
    return A, G, clip


def _sum64(A, G, clip):
    a = (A * clip.view(-1, 1, 1)).double().reshape(-1, A.shape[-1])
    return a.T @ G.double().reshape(-1, G.shape[-1])


def _norm64(A, G):
    return torch.stack([(a.double().T @ g.double()).pow(2).sum() for a, g in zip(A, G)])


def _rel(x, ref):
    return float((x.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("B,T,d_in,d_out", [
    (600, 1, 128, 128), (1031, 1, 252, 508), (3, 347, 256, 256), (5, 260, 100, 124), (260, 5, 512, 260),
    (600, 1, 784, 512), (2, 512, 260, 512), (64, 9, 128, 1028), (521, 1, 200, 1024),
    (300, 1, 1500, 1030), (4097, 1, 64, 120), (2053, 1, 577, 64), (3, 700, 101, 61), (33000, 1, 512, 251), (2, 333, 63, 127)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_clipped_sum(B, T, d_in, d_out, accumulate):
    A, G, clip = _data(B, T, d_in, d_out, 1)
    start = torch.ones((d_in, d_out), device="cuda") if accumulate else None
    g = dp.clipped_grad(A, G, clip, grad=start, accumulate=accumulate)
    ref = _sum64(A, G, clip) + (1.0 if accumulate else 0.0)
    assert _rel(g, ref) < REL


@pytest.mark.parametrize("path,T,d_in,d_out", [
    ("gram", 33, 36, 68), ("gram", 64, 17, 40), ("gram", 65, 64, 128), ("gram", 127, 30, 33), ("gram", 128, 48, 260),
    ("gram", 129, 1, 16), ("gram", 256, 48, 33), ("gram", 512, 18, 61), ("gram", 300, 132, 20), ("direct", 128, 128, 64), ("direct", 260, 577, 61), ("direct", 131, 60, 125), ("direct", 256, 128, 128), ("direct", 300, 252, 100), ("direct", 1024, 384, 128)])
def test_norms(path, T, d_in, d_out):
    A, G, _ = _data(9, T, d_in, d_out, 2)
    s = dp.layer_sqnorm(A, G, path=path)
    ref = _norm64(A, G)
    assert float(((s.double() - ref) / ref).abs().max()) < REL


@pytest.mark.parametrize("B,shapes", [
    (1, [(12544, 64, 128)]), (17, [(3136, 63, 127)]), (300, [(1030, 64, 128)]), (40, [(1100, 577, 61)]), (130, [(196, 128, 128)]),
    (3, [(12544, 64, 128), (3136, 128, 256), (784, 256, 512)]), (3, [(784, 64, 128), (128, 128, 64)]), (65, [(784, 576, 64), (196, 576, 64)]),
    (2, [(1600, 96, 64)] * 2 + [(700, 250, 60)] * 3), (20, [(1024, 64, 128)] * 18)])
def test_direct_norms_on_either_side_of_the_choice(B, shapes):
    """Layers on the split kernel and on the fp32 one, alone and in a shared launch that leaves the long ones out."""
    layers = [_data(B, T, a, b, 11 + i)[:2] for i, (T, a, b) in enumerate(shapes)]
    s = dp.layers_sqnorm(layers, path="direct")
    ref = sum(_norm64(A, G) for A, G in layers)
    assert float(((s.double() - ref) / ref).abs().max()) < REL


@pytest.mark.parametrize("B,shapes", [
    (384, [(1, 844, 1664)]), (512, [(1, 844, 1664)] * 2), (500, [(1, 4608, 512)]), (256, [(1, 2304, 512)] * 2 + [(1, 64, 30)]), (256, [(1, 2304, 512)] * 4),
    (12500, [(1, 63, 127)]), (25000, [(1, 63, 127)]), (6000, [(1, 576, 64)]), (20000, [(1, 576, 64)]), (14100, [(1, 64, 128)] * 2),
    (9000, [(1, 64, 128)] * 2), (9000, [(1, 64, 128), (1, 96, 64), (1, 128, 128)]), (400, [(2, 126, 62), (1, 600, 1030)]), (1031, [(1, 600, 1030)])])
@pytest.mark.parametrize("noise", [0.0, 1.0])
def test_clipped_sums_on_either_side_of_the_choice(B, shapes, noise):
    """Layers on the split kernel and on the fp32 ones, alone and beside each other."""
    layers = [_data(B, T, a, b, 31 + i)[:2] for i, (T, a, b) in enumerate(shapes)]
    grads = [torch.ones((a, b), device="cuda") for _, a, b in shapes]
    clip = torch.rand(B, device="cuda") + 0.25
    descs = dp.layer_descs(layers, grads)
    dp.layers_clipped_grad(layers, clip, grads, accumulate=True, descs=descs, noise_std=noise, seed=3)
    off = 0
    for (A, G), g in zip(layers, grads):
        ref = _sum64(A, G, clip) + 1.0
        if noise:
            z = torch.zeros_like(g)
            dp.add_noise(z, noise, 3, off)
            ref = ref + z
        off += g.numel()
        assert _rel(g, ref) < REL


@pytest.mark.parametrize("B", [1, 7, 8, 19])
@pytest.mark.parametrize("kind", ["gram", "direct"])
def test_layers_of_one_launch(B, kind):
    """Layers of different widths and lengths share a launch; examples that are no multiple of the eight XCDs."""
    shapes = ([(200, 256, 512), (130, 768, 260), (64, 260, 320), (50, 512, 400), (70, 301, 402)] if kind == "gram"
              else [(1024, 128, 128), (1024, 576, 64), (512, 256, 124), (300, 128, 256), (400, 64, 128)])
    layers = [_data(B, T, a, b, 3 + i)[:2] for i, (T, a, b) in enumerate(shapes)]
    s = dp.layers_sqnorm(layers)
    ref = sum(_norm64(A, G) for A, G in layers)
    assert float(((s.double() - ref) / ref).abs().max()) < REL
    clip = torch.rand(B, device="cuda") + 0.25
    for (A, G), g in zip(layers, dp.layers_clipped_grad(layers, clip)):
        assert _rel(g, _sum64(A, G, clip)) < REL


@pytest.mark.parametrize("scale", [1e-20, 1e-25, 1e-28, 1e-30, 1e-33, 1e-36])
def test_small_gradients_keep_their_bits(scale):
    """(The squared norms of such gradients are below the smallest float32; theirs are tested from 1e-17 on.)"""
    A, G, clip = _data(4, 256, 128, 128, 4, scale)
    assert _rel(dp.clipped_grad(A, G, clip), _sum64(A, G, clip)) < REL


@pytest.mark.parametrize("a_scale,g_scale", [(1e10, 1e-36), (1e10, 1e-37), (1e12, 1e-38), (1e20, 1e-40), (1e30, 1e-41), (1e30, 1e-43)])
@pytest.mark.parametrize("small_a", [False, True])
@pytest.mark.parametrize("B,T,d", [(4, 256, 128), (65536, 1, 256)])
def test_small_operands_with_large_partners(B, T, d, small_a, a_scale, g_scale):
    """Operands whose low parts fall below the smallest bf16, subnormal ones among them, in sums that are not small."""
    A, G, clip = _data(B, T, d, d, 6)
    A, G = (A * g_scale, G * a_scale) if small_a else (A * a_scale, G * g_scale)
    # factors of 1 and 2: the reference's product a * c is exact also where it is subnormal
    clip.copy_(torch.exp2(torch.randint(0, 2, (B,), device="cuda").float()))
    assert _rel(dp.clipped_grad(A, G, clip), _sum64(A, G, clip)) < REL
    if T > 1 and a_scale >= 1e20:                             # (squares of the sums that float32 holds)
        s, ref = dp.layer_sqnorm(A, G, path="direct"), _norm64(A, G)
        assert float(((s.double() - ref) / ref).abs().max()) < REL


@pytest.mark.parametrize("a_scale,g_scale,path", [(1e13, 1e-10, "gram"), (1e-10, 1e13, "gram"), (1e20, 1e8, "sum")])
def test_sums_that_are_formed_again(a_scale, g_scale, path):
    """Finite sums of 2^80 and more are formed again in float32 (odd lengths and widths: its remainders)."""
    A, G, clip = _data(3, 333, 132, 128, 13)
    A, G = A * a_scale, G * g_scale
    if path == "sum":
        # sums of 999 float32 products in the order of k: sqrt(999) 2^-24 of the result, four times that
        assert _rel(dp.clipped_grad(A, G, clip), _sum64(A, G, clip)) < 8e-6
    else:
        s, ref = dp.layer_sqnorm(A, G, path=path), _norm64(A, G)
        assert float(((s.double() - ref) / ref).abs().max()) < REL


@pytest.mark.parametrize("g_scale", [1e-10, 1e-14, 1e-17])
@pytest.mark.parametrize("path", ["gram", "direct"])
def test_norms_of_small_gradients(path, g_scale):
    A, G, _ = _data(4, 256, 128, 128, 7, g_scale)            # 1e-17 gives norms of 1e-28
    s, ref = dp.layer_sqnorm(A, G, path=path), _norm64(A, G)
    assert float(((s.double() - ref) / ref).abs().max()) < REL


@pytest.mark.parametrize("path,T,d_in,d_out", [("gram", 512, 768, 768), ("direct", 1024, 576, 128)])
def test_small_rows_take_no_longer(path, T, d_in, d_out):
    """A position whose gradient is almost zero (a prediction that is almost perfect), a column of gradients of almost
    zero (a class that never occurs): ordinary data, in the ordinary time."""
    A, G, _ = _data(32, T, d_in, d_out, 8, 1e-3)
    small = G.clone()
    small[:, 5::64] *= 1e-16
    small[:, :, 7] *= 1e-33

    def ms(g):
        best = 1e9
        for _ in range(5):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            s = dp.layer_sqnorm(A, g, path=path)
            e[1].record()
            e[1].synchronize()
            best = min(best, e[0].elapsed_time(e[1]))
        return best, s
    (usual, _), (time, s) = ms(G), ms(small)
    ref = _norm64(A, small)
    assert float(((s.double() - ref) / ref).abs().max()) < REL
    assert time < 1.5 * usual, (time, usual)


@pytest.mark.parametrize("value", [float("inf"), float("-inf")])
@pytest.mark.parametrize("in_g", [False, True])
@pytest.mark.parametrize("B,T,d_in,d_out", [(3, 257, 128, 128), (65, 131, 577, 61), (3, 101, 70, 33)])
def test_infinity_in_the_last_of_an_odd_number_of_rows(B, T, d_in, d_out, in_g, value):
    """The sums of its column are infinite, not NaN: the clip factor of an infinite norm is 0."""
    A, G, clip = _data(B, T, d_in, d_out, 9)
    clip.fill_(0.5)
    A[A == 0] = 1.0
    G[G == 0] = 1.0
    (G if in_g else A)[-1, T - 1, 5] = value
    s = dp.layer_sqnorm(A, G, path="direct")
    assert torch.isfinite(s[:-1]).all() and torch.isposinf(s[-1])
    got = dp.clipped_grad(A, G, clip)
    line = got[:, 5] if in_g else got[5]
    other = (A if in_g else G)[-1, T - 1]
    assert torch.equal(line, torch.sign(other) * value)
    rest = got.clone()
    (rest[:, 5] if in_g else rest[5]).zero_()
    assert torch.isfinite(rest).all()


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.4e38])
@pytest.mark.parametrize("d", [128, 256])
def test_values_without_three_parts(value, d):
    """Infinities, NaN and numbers that round to an infinite bf16 come out as float32 sums give them."""
    A, G, clip = _data(4, 256, d, d, 5, 1e-3)
    clip.fill_(0.5)
    A[1, 17, 5] = value
    got = dp.clipped_grad(A, G, clip).cpu().numpy()
    a = (A * 0.5).cpu().numpy().astype(np.float64).reshape(-1, d)
    with np.errstate(all="ignore"):
        ref = a.T @ G.cpu().numpy().astype(np.float64).reshape(-1, d)
    assert (np.isnan(got) == np.isnan(ref)).all()
    assert (np.isinf(got) == np.isinf(ref)).all()
    inf = np.isinf(ref)
    assert (np.sign(got[inf]) == np.sign(ref[inf])).all()
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= 1e-5 * np.abs(ref[ok]).max()
    for path in ("gram", "direct"):
        s = dp.layer_sqnorm(A, G, path=path).cpu().numpy()
        assert not np.isfinite(s[1]) and np.isfinite(s[[0, 2, 3]]).all()
