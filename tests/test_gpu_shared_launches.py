"""Layers that share launches: 16-bit Gram norms of ragged shapes, bias rows and bias gradients, and the layers that must
not share one (gradients of one array)."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu


def _layers(B, shapes, dtype, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return [(torch.randn((B, T, a), device="cuda", generator=gen).to(dtype), (torch.randn((B, T, b), device="cuda", generator=gen)).to(dtype))
            for T, a, b in shapes]


def _norm64(A, G):
    return torch.stack([(a.double().T @ g.double()).pow(2).sum() for a, g in zip(A, G)])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B", [1, 9, 32])
def test_ragged_gram_norms_of_one_launch(dtype, B):
    layers = _layers(B, [(250, 200, 600), (65, 199, 201), (128, 100, 444), (129, 300, 333)], dtype)
    s = dp.layers_sqnorm(layers, path="gram")
    ref = sum(_norm64(A, G) for A, G in layers)
    # float32 sums of exact products, all of them squares' sums of up to 2^15 terms: K 2^-24 at the worst, 1e-5 covers it
    assert float(((s.double() - ref) / ref).abs().max()) < 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,n", [(1, 2), (5, 3), (32, 17), (2050, 2)])
@pytest.mark.parametrize("noise", [0.0, 0.7])
def test_biases_of_one_launch_equal_one_by_one(dtype, B, n, noise):
    """Widths of 16-byte rows and ragged ones; the shared launches add in the order of the single ones: same bits."""
    shapes = [(1 + 3 * (l % 5), 8, (40, 33, 520, 2, 128)[l % 5]) for l in range(n)]
    layers = _layers(B, shapes, dtype, 1)
    grads = [torch.zeros((a, b), device="cuda") for _, a, b in shapes]
    rows = [torch.zeros((B, b), device="cuda") for _, _, b in shapes]
    gbs = [torch.ones(b, device="cuda") for _, _, b in shapes]
    offs = [4 * 10 ** 6 + 1001 * l for l in range(n)]
    descs = dp.layer_descs(layers, grads, bias_rows=rows, grad_bs=gbs, bias_noise_offsets=offs)
    s = dp.layers_sqnorm(layers, descs=descs)
    clip = torch.rand(B, device="cuda") + 0.25
    dp.layers_clipped_grad(layers, clip, grads, descs=descs, noise_std=noise, seed=11)
    ref_s = dp.layers_sqnorm(layers)
    for (A, G), r, g, off in zip(layers, rows, gbs, offs):
        one = torch.empty_like(r)
        dp.bias_sqnorm(G, ref_s, one, accumulate=True)
        assert torch.equal(one, r)
        gb = torch.empty_like(g)
        dp.clipped_bias_grad(one, clip, gb)
        if noise:
            dp.add_noise(gb, noise, 11, off)
        assert torch.equal(gb, g)
    # the weights' norms are added before the biases' in both
    assert torch.allclose(s, ref_s, rtol=1e-6, atol=0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_tied_weights_accumulate_into_one_array(dtype):
    shapes = [(64, 128, 128), (64, 128, 128), (64, 256, 128)]
    layers = _layers(8, shapes, dtype, 2)
    tied = torch.zeros((128, 128), device="cuda")
    grads = [tied, tied, torch.zeros((256, 128), device="cuda")]
    bias = torch.zeros(128, device="cuda")
    rows = [torch.zeros((8, 128), device="cuda") for _ in shapes]
    clip = torch.rand(8, device="cuda") + 0.25
    descs = dp.layer_descs(layers, grads, bias_rows=rows, grad_bs=[bias] * 3)
    dp.layers_sqnorm(layers, descs=descs)
    dp.layers_clipped_grad(layers, clip, grads, accumulate=True, descs=descs)
    w = clip.double().view(-1, 1, 1)
    sums = [(A.double() * w).reshape(-1, A.shape[-1]).T @ G.double().reshape(-1, G.shape[-1]) for A, G in layers]
    ref, ref_b = sums[0] + sums[1], sum((G.double() * w).sum((0, 1)) for _, G in layers)
    # bfloat16 rows may be rounded once more by the factor: 2^-9 each
    tol = 1e-6 if dtype == torch.float32 else 4e-3
    assert float((tied.double() - ref).norm() / ref.norm()) < tol
    assert float((grads[2].double() - sums[2]).norm() / sums[2].norm()) < tol
    assert float((bias.double() - ref_b).norm() / ref_b.norm()) < 1e-5


@pytest.mark.parametrize("dtype,shapes,B", [
    (torch.float32, [(128, 256, 128)] * 2 + [(128, 512, 768), (128, 768, 512)], 64),
    (torch.bfloat16, [(128, 256, 256)] * 2 + [(128, 256, 512), (128, 512, 256)], 64),
    (torch.bfloat16, [(64, 576, 64)] * 2 + [(64, 576, 128)] * 3, 32)])
@pytest.mark.parametrize("left_out", ["tied", "offset"])
def test_layers_beside_some_that_cannot_share(dtype, shapes, B, left_out):
    """The remaining layers of a group do with the scratch that the query gave for the whole one."""
    layers = _layers(B, shapes, dtype, 3)
    grads = [torch.zeros((a, b), device="cuda") for _, a, b in shapes]
    offs, at = [], 0
    for l, (_, a, b) in enumerate(shapes):
        offs.append(at + (1 if left_out == "offset" and l < 2 else 0))
        at += a * b + 4
    std = 1.0 if left_out == "offset" else 0.0
    if left_out == "tied":
        grads[1] = grads[0]
    clip = torch.rand(B, device="cuda") + 0.25
    descs = dp.layer_descs(layers, grads, noise_offsets=offs)
    dp.layers_clipped_grad(layers, clip, grads, accumulate=True, descs=descs, noise_std=std, seed=5)
    w = clip.double().view(-1, 1, 1)
    sums = [(A.double() * w).reshape(-1, A.shape[-1]).T @ G.double().reshape(-1, G.shape[-1]) for A, G in layers]
    if left_out == "tied":
        sums[0] = sums[1] = sums[0] + sums[1]
    # bfloat16 rows may be rounded once more by the factor: 2^-9 each
    tol = 1e-6 if dtype == torch.float32 else 4e-3
    for g, r, off in zip(grads, sums, offs):
        if std:
            z = torch.zeros_like(g)
            dp.add_noise(z, std, 5, off)
            r = r + z
        assert float((g.double() - r).norm() / r.norm()) < tol


@pytest.mark.parametrize("dtype,B,n", [(torch.bfloat16, 4100, 2), (torch.float32, 2031, 4)])
def test_more_items_than_a_launch_holds(dtype, B, n):
    """2080 tile pairs per example: the layers together have more workgroups than one launch can."""
    gen = torch.Generator(device="cuda").manual_seed(4)
    A = torch.randn((B, 8192, 3), device="cuda", generator=gen).to(dtype)
    G = torch.randn((B, 8192, 2), device="cuda", generator=gen).to(dtype)
    s = dp.layers_sqnorm([(A, G)] * n, path="gram")
    one = dp.layer_sqnorm(A, G, path="direct")
    # float32 sums of 2^26 terms of random sign, in two ways
    assert torch.allclose(s, n * one, rtol=1e-4, atol=0)
