"""Gram norms of layers of few positions and wide rows in a small batch: the columns of an example are split over
workgroups, whose shares are added by a second launch."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu


def _tensor(gen, B, T, d, dtype):
    """B x T x d numbers in the middle of NaNs: nothing outside the matrix may count."""
    pad = 1024
    buf = torch.full((B * T * d + 2 * pad,), float("nan"), device="cuda", dtype=dtype)
    x = buf[pad:pad + B * T * d].view(B, T, d)
    x.copy_(torch.randn((B, T, d), device="cuda", generator=gen))
    return x


def _norm64(A, G):
    return (A.double() @ A.double().transpose(1, 2).contiguous() * (G.double() @ G.double().transpose(1, 2).contiguous())).sum((1, 2))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B", [1, 20, 200])
@pytest.mark.parametrize("shapes", [
    [(16, 4608, 512)],                                                          # alone: the norms in the second launch
    [(33, 1032, 264)],
    [(2, 1024, 512), (7, 1048, 520), (31, 2304, 256), (32, 1152, 1032)],        # one 32-row block
    [(64, 2304, 256), (33, 1160, 512), (8, 1024, 1024), (57, 3080, 72)],        # one and two in a launch
    [(5 + 3 * l, 1024 + 8 * l, 512) for l in range(18)],                        # more than a launch takes
])
def test_norms_against_float64(dtype, B, shapes):
    gen = torch.Generator(device="cuda").manual_seed(7)
    layers = [(_tensor(gen, B, T, a, dtype), _tensor(gen, B, T, b, dtype)) for T, a, b in shapes]
    ref = sum(_norm64(A, G) for A, G in layers)
    s = dp.layers_sqnorm(layers, path="gram")
    # float32 sums over at most 4608 columns of products of random sign: sqrt(4608) 2^-24 of an entry, 1e-5 covers it
    assert float(((s.double() - ref) / ref).abs().max()) < 1e-5
    acc = torch.full((B,), 2.0, device="cuda")
    dp.layers_sqnorm(layers, acc, path="gram", accumulate=True)
    assert torch.allclose(acc.double(), ref + 2.0, rtol=1e-5, atol=0)


@pytest.mark.parametrize("shapes", [[(17, 1023, 769)], [(64, 1025, 514), (16, 2047, 333), (3, 1021, 1022)]])
def test_float32_rows_of_any_length(shapes):
    gen = torch.Generator(device="cuda").manual_seed(8)
    layers = [(_tensor(gen, 9, T, a, torch.float32), _tensor(gen, 9, T, b, torch.float32)) for T, a, b in shapes]
    ref = sum(_norm64(A, G) for A, G in layers)
    s = dp.layers_sqnorm(layers, path="gram")
    assert float(((s.double() - ref) / ref).abs().max()) < 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_clip_factors_beside_other_layers(dtype):
    """Dense layers and layers of other norm kernels in the same step: the factors are those of the complete norms."""
    gen = torch.Generator(device="cuda").manual_seed(9)
    shapes = [(16, 1152, 512), (64, 1152, 256), (1, 512, 10), (256, 64, 64), (1024, 27, 64), (16, 2304, 512)]
    layers = [(_tensor(gen, 12, T, a, dtype), _tensor(gen, 12, T, b, dtype)) for T, a, b in shapes]
    ref = sum(_norm64(A, G) for A, G in layers)
    for keep in (slice(0, 2), slice(0, 3), slice(0, 6), slice(1, 3), slice(0, 4)):
        part = layers[keep]
        want = sum(_norm64(A, G) for A, G in part)
        C = float(want.median().sqrt())
        sq, clip = torch.zeros(12, device="cuda"), torch.zeros(12, device="cuda")
        grads = [torch.zeros((A.shape[-1], G.shape[-1]), device="cuda") for A, G in part]
        squeezed = [(A.squeeze(1), G.squeeze(1)) if A.shape[1] == 1 else (A, G) for A, G in part]
        arr, n, code = descs = dp.layer_descs(squeezed, grads)
        need = max(dp.layers_workspace_bytes(arr, n, code), dp.layers_clipped_workspace_bytes(arr, n, code))
        dp.layers_step(descs, C, sq, clip, torch.empty(need, dtype=torch.uint8, device="cuda"))
        assert torch.allclose(sq.double(), want, rtol=1e-5, atol=0)
        assert torch.allclose(clip.double(), (C / want.sqrt()).clamp(max=1.0), rtol=1e-5, atol=0)
    assert torch.allclose(dp.layers_sqnorm([(A.squeeze(1), G.squeeze(1)) if A.shape[1] == 1 else (A, G) for A, G in layers]).double(), ref, rtol=1e-5, atol=0)


def _time(call):
    """The shortest of 5 times of 20 calls, in microseconds."""
    best = float("inf")
    for _ in range(5):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(20):
            call()
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end) / 20 * 1e3)
    return best


def test_float32_rows_of_any_length_share_a_launch():
    """One launch for several such layers is no slower than a launch each (it took 2.3 times as long when every example had one
    workgroup per layer: 22 examples, 133 and 57 us)."""
    gen = torch.Generator(device="cuda").manual_seed(11)
    layers = [(_tensor(gen, 22, T, a, torch.float32), _tensor(gen, 22, T, b, torch.float32)) for T, a, b in
              [(51, 1003, 592), (40, 684, 4586), (31, 2710, 1264)]]
    s = torch.zeros(22, device="cuda")

    def shared(part):
        descs = dp.layer_descs(part)
        ws = torch.empty(dp.layers_workspace_bytes(descs[0], 22, descs[2], "gram"), dtype=torch.uint8, device="cuda")
        return lambda: dp.layers_sqnorm(part, s, path="gram", workspace=ws, descs=descs)

    assert _time(shared(layers)) < 1.4 * sum(_time(shared([x])) for x in layers)


@pytest.mark.parametrize("B", [1, 22, 100])
@pytest.mark.parametrize("shapes", [
    [(51, 1003, 592), (40, 684, 4586), (31, 2710, 1264)],                       # both numbers of 32-row blocks
    [(16, 2047, 333), (16, 2304, 512), (64, 2304, 256), (9, 1025, 1023)],       # whole pieces in the same launch, and in one of their own
    [(33 + l, 1023 + l, 515) for l in range(20)],                               # more than a launch takes
])
@pytest.mark.parametrize("others", [[], [(256, 64, 64), (1024, 27, 64)]])       # with others the sums go to the queue
def test_float32_rows_of_any_length_beside_others(B, shapes, others):
    gen = torch.Generator(device="cuda").manual_seed(12)
    layers = [(_tensor(gen, B, T, a, torch.float32), _tensor(gen, B, T, b, torch.float32)) for T, a, b in shapes + others]
    ref = sum(_norm64(A, G) for A, G in layers)
    descs = dp.layer_descs(layers)
    need = dp.layers_workspace_bytes(descs[0], B, descs[2])
    ws = torch.full((need + 4096,), 7, dtype=torch.uint8, device="cuda")
    s = torch.zeros(B, device="cuda")
    dp.layers_sqnorm(layers, s, workspace=ws[:need], descs=descs)
    # float32 sums over at most 4586 columns of products of random sign
    assert float(((s.double() - ref) / ref).abs().max()) < 1e-5
    assert bool((ws[need:] == 7).all())                     # nothing behind the scratch that was asked for


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,T,a,b", [
    (60, 8, 5312, 2048), (100, 20, 1456, 528), (300, 32, 712, 504), (500, 25, 712, 504), (511, 31, 712, 504),      # one 32-row block: two to four workgroups
    (300, 40, 1456, 528), (192, 48, 1216, 440), (174, 64, 1456, 528), (130, 49, 712, 504), (256, 64, 1456, 528)])  # two: two or three, copied or loaded
def test_layers_alone_with_many_workgroups(dtype, B, T, a, b):
    gen = torch.Generator(device="cuda").manual_seed(B)
    A, G = _tensor(gen, B, T, a, dtype), _tensor(gen, B, T, b, dtype)
    ref = _norm64(A, G)
    s = dp.layer_sqnorm(A, G, path="gram")
    # float32 sums over at most 5312 columns of products of random sign
    assert float(((s.double() - ref) / ref).abs().max()) < 1e-5


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,shapes", [(64, [(16, 4608, 512)] * 3 + [(64, 2304, 256)] * 3), (100, [(4, 4128, 304), (4, 3000, 600)]),
                                      (64, [(25, 4464, 784), (9, 1496, 496), (36, 3976, 656), (4, 3704, 640)])])
def test_norms_of_several_layers_are_not_off_to_one_side(dtype, B, shapes):
    """A chain of matrix instructions may round its running sum to one side.  Chains of 8 steps put the mean of the 256 or 400
    errors (standard error 4e-9) at 1.8e-8 at most; the longer waves of a shared launch, without an end to their chains, at
    5.6e-8 to 8e-8 in bf16."""
    errors = []
    for seed in range(4):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        layers = [(_tensor(gen, B, T, a, dtype), _tensor(gen, B, T, b, dtype)) for T, a, b in shapes]
        ref = sum(_norm64(A, G) for A, G in layers)
        errors.append((dp.layers_sqnorm(layers, path="gram").double() - ref) / ref)
    assert abs(float(torch.cat(errors).mean())) < 3e-8


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("others", [[(12, 64, 64)] * 2, [(100, 200, 72)], [(100, 200, 72)] * 2, [(12, 64, 64), (100, 200, 72), (300, 200, 72)], [(12, 64, 64)] * 2 + [(256, 64, 64)]])
@pytest.mark.parametrize("biased", [False, True])
def test_beside_layers_that_add_their_own_norms(dtype, others, biased):
    """16-bit Gram norms of one sum an example are added by their own kernels, other layers' by the queue: complete norms and
    their clip factors with both, and accumulated."""
    gen = torch.Generator(device="cuda").manual_seed(13)
    B = 10
    layers = [(_tensor(gen, B, T, a, dtype), _tensor(gen, B, T, b, dtype)) for T, a, b in [(16, 1152, 512), (64, 1152, 256)] + others]
    ref = sum(_norm64(A, G) for A, G in layers)
    rows = [torch.zeros((B, G.shape[-1]), device="cuda") if biased and l % 2 else None for l, (_, G) in enumerate(layers)]
    ref = ref + sum(G.double().sum(1).pow(2).sum(1) for (_, G), r in zip(layers, rows) if r is not None)
    C = float(ref.median().sqrt())
    descs = dp.layer_descs(layers, bias_rows=rows)
    for start in (None, 5.0):
        s, clip = torch.full((B,), start or float("nan"), device="cuda"), torch.zeros(B, device="cuda")
        dp.layers_sqnorm(layers, s, path="gram", accumulate=start is not None, descs=descs, C=C, clip=clip)
        want = ref + (start or 0.0)
        assert torch.allclose(s.double(), want, rtol=1e-5, atol=0)
        assert torch.allclose(clip.double(), (C / want.sqrt()).clamp(max=1.0), rtol=1e-5, atol=0)
