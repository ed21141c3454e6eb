"""Clipped sums and direct norms on 256 x 256 tiles, whose two halves of waves work in opposite phases: few stages, slices that
end inside an example, examples that are left out, and launches whose slices have two lengths."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu
F8 = (torch.float8_e4m3fn, torch.float8_e5m2)


def _pair(gen, B, T, a, b, types):
    A = torch.randn((B, T, a), device="cuda", generator=gen).to(types[0])
    G = torch.randn((B, T, b), device="cuda", generator=gen).to(types[1])
    return A, G


def _sum64(A, G, clip):
    w = clip.double().view(-1, 1, 1)
    return (A.double() * w).reshape(-1, A.shape[-1]).T.contiguous() @ G.double().reshape(-1, G.shape[-1])


# float32 sums of up to 2^15 products: 1e-6 of the largest; the 8-bit instruction aligns its 64 products and drops 2^-16 of the
# largest of them
@pytest.mark.parametrize("types,tol", [((torch.bfloat16,) * 2, 2e-6), ((torch.float16,) * 2, 2e-6), (F8, 6e-5), ((F8[0],) * 2, 6e-5)])
@pytest.mark.parametrize("B,T,a,b", [(1, 64, 256, 256), (1, 128, 512, 256), (3, 64, 256, 512), (2, 192, 496, 512), (5, 320, 256, 768),
                                     (40, 64, 512, 512), (7, 96, 512, 512), (9, 1000, 256, 256)])
def test_few_stages(types, tol, B, T, a, b):
    gen = torch.Generator(device="cuda").manual_seed(B * T)
    A, G = _pair(gen, B, T, a, b, types)
    clip = torch.rand(B, device="cuda", generator=gen) + 0.25
    if B > 2:
        clip[1] = 0.0                                        # left out
        clip[-1] = clip[-2]                                  # nothing to rescale
    got = dp.clipped_grad(A, G, clip).double()
    ref = _sum64(A, G, clip)
    # layers that are not whole blocks may have the factor multiplied into the 16-bit rows (2^-9 and 2^-12 of a term)
    loose = dp.load_library().dp_clipped_grad_rounds_inputs(B, T, a, b, dp.layer_descs([(A, G)])[2]) != 0
    assert float((got - ref).norm() / ref.norm()) < (4e-3 if loose else tol)
    s = dp.layer_sqnorm(A, G, path="direct").double()
    want = torch.stack([(x.double().T.contiguous() @ g.double()).pow(2).sum() for x, g in zip(A, G)])
    assert float(((s - want) / want).abs().max()) < 4 * tol


@pytest.mark.parametrize("types,tol", [((torch.bfloat16,) * 2, 2e-6), (F8, 6e-5)])
@pytest.mark.parametrize("B,T,shapes", [
    (16, 512, [(768, 2304), (768, 768), (768, 3072), (3072, 768)]),
    (24, 256, [(1024, 1024), (1024, 2048)]),
    (70, 64, [(2048, 1024), (1024, 2048), (1024, 1024)]),       # a slice may touch 64 examples
    (33, 192, [(3072, 1008), (1008, 1024)]),
])
@pytest.mark.parametrize("noise,accumulate", [(0.0, False), (0.5, False), (0.0, True)])
def test_several_layers(types, tol, B, T, shapes, noise, accumulate):
    gen = torch.Generator(device="cuda").manual_seed(B + T)
    layers = [_pair(gen, B, T, a, b, types) for a, b in shapes]
    clip = torch.rand(B, device="cuda", generator=gen) + 0.25
    clip[0] = clip[5] = 0.0
    grads = [torch.ones((a, b), device="cuda") for a, b in shapes]
    descs = dp.layer_descs(layers, grads)
    need = dp.layers_clipped_workspace_bytes(descs[0], B, descs[2])
    ws = torch.full((need + 4096,), 7, dtype=torch.uint8, device="cuda")
    dp.layers_clipped_grad(layers, clip, grads, workspace=ws[:need], descs=descs, noise_std=noise, seed=3, accumulate=accumulate)
    assert bool((ws[need:] == 7).all())                     # nothing behind the scratch that was asked for
    at = 0
    for (A, G), g, (a, b) in zip(layers, grads, shapes):
        ref = _sum64(A, G, clip) + (1.0 if accumulate else 0.0)
        if noise:
            z = torch.zeros_like(g)
            dp.add_noise(z, noise, 3, at)
            ref += z
        at += a * b
        assert float((g.double() - ref).norm() / ref.norm()) < tol


@pytest.mark.parametrize("types", [F8, (F8[0],) * 2])
@pytest.mark.parametrize("B,layers_of", [
    (8, [(384, 1792, 2304), (64, 1024, 2048), (64, 1536, 1792), (384, 2304, 1280)]),     # packs of two over 63 and 45 tiles, two layers without
    (14, [(256, 1280, 2304), (64, 2048, 2048), (256, 2048, 2048)]),                      # a layer without rests between two with them
    (64, [(512, 768, 2304), (512, 768, 768), (512, 768, 3072), (512, 3072, 768)]),       # packs of three
    (14, [(256, 1264, 2304), (256, 2048, 2032), (64, 2048, 2048)]),                      # edge tiles
])
@pytest.mark.parametrize("noise,accumulate", [(0.0, False), (0.5, False), (0.0, True)])
def test_slices_of_two_lengths(types, B, layers_of, noise, accumulate):
    gen = torch.Generator(device="cuda").manual_seed(B)
    layers = [_pair(gen, B, T, a, b, types) for T, a, b in layers_of]
    clip = torch.rand(B, device="cuda", generator=gen) + 0.25
    clip[0] = clip[B // 2] = clip[-1] = 0.0                 # the last examples lie in the rests
    clip[-2] = 2e-14                                        # left out: below 2^-40 of the largest before it
    counted = torch.where(clip < 1e-12, torch.zeros_like(clip), clip)
    grads = [torch.ones((a, b), device="cuda") for _, a, b in layers_of]
    descs = dp.layer_descs(layers, grads)
    assert dp.load_library().dp_plan_sums_in_two_lengths(descs[0], len(layers), B, descs[2]) > 0
    need = dp.layers_clipped_workspace_bytes(descs[0], B, descs[2])
    ws = torch.full((need + 4096,), 7, dtype=torch.uint8, device="cuda")
    dp.layers_clipped_grad(layers, clip, grads, workspace=ws[:need], descs=descs, noise_std=noise, seed=3, accumulate=accumulate)
    assert bool((ws[need:] == 7).all())                     # nothing behind the scratch that was asked for
    at = 0
    for (A, G), g, (_, a, b) in zip(layers, grads, layers_of):
        ref = _sum64(A, G, counted) + (1.0 if accumulate else 0.0)
        if noise:
            z = torch.zeros_like(g)
            dp.add_noise(z, noise, 3, at)
            ref += z
        at += a * b
        assert float((g.double() - ref).norm() / ref.norm()) < 6e-5
