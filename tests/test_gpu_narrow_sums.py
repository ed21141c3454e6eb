"""Clipped sums of many rows with one operand of at most 32 columns."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T,a,b", [
    (4096, 1, 64, 10), (4097, 1, 128, 32), (5000, 1, 1, 1), (70000, 1, 129, 2), (20011, 1, 256, 10), (4500, 1, 1000, 32),
    (9001, 1, 2, 500), (20, 1024, 27, 64), (3, 4100, 31, 33), (30, 197, 33, 31), (1, 9999, 75, 16), (513, 8, 3, 131),
])
@pytest.mark.parametrize("accumulate,noise", [(False, 0.0), (True, 0.0), (False, 0.5)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_sums_against_float64(B, T, a, b, accumulate, noise, dtype):
    gen = torch.Generator(device="cuda").manual_seed(B + T)
    lead = (B,) if T == 1 else (B, T)

    def tensor(d):                                           # in the middle of NaNs: nothing around the matrix may count
        buf = torch.full((B * T * d + 2048,), float("nan"), device="cuda", dtype=dtype)
        x = buf[1024:1024 + B * T * d].view(*lead, d)
        x.copy_(torch.randn((*lead, d), device="cuda", generator=gen))
        return x

    A, G = tensor(a), tensor(b)
    clip = torch.rand(B, device="cuda", generator=gen)
    if B > 1:
        clip[0] = 0.0
    w = clip.double().view(-1, *([1] * (len(lead))))
    ref = (A.double() * w).reshape(-1, a).T @ G.double().reshape(-1, b)
    grad = torch.full((a, b), 2.0, device="cuda")
    descs = dp.layer_descs([(A, G)], [grad])
    dp.layers_clipped_grad([(A, G)], clip, [grad], descs=descs, accumulate=accumulate, noise_std=noise, seed=5)
    if accumulate:
        ref = ref + 2.0
    if noise:
        z = torch.zeros_like(grad)
        dp.add_noise(z, noise, 5, 0)
        ref = ref + z
    # sums of random sign in blocks of at most 512 rows: below 1e-6 of the result; the kernels of the other 16-bit shapes may
    # round the rows once more after the factor (2^-9 and 2^-12 of a term)
    rounds = dp.load_library().dp_clipped_grad_rounds_inputs(B, T, a, b, dp.layer_descs([(A, G)])[2]) != 0
    assert not (rounds and max(a, b) <= 128)
    assert float((grad.double() - ref).norm() / ref.norm()) < (4e-3 if rounds else 1e-6)


def test_infinite_rows_stay_in_their_columns():
    """A row past the end of a slice is read again and counts as zero: infinities of the last row must not become NaN elsewhere."""
    A, G = torch.ones((4099, 40), device="cuda"), torch.ones((4099, 10), device="cuda")
    A[-1, 3] = float("inf")
    g = dp.clipped_grad(A, G, torch.ones(4099, device="cuda"))
    assert bool(torch.isinf(g[3]).all()) and bool((g[torch.arange(40, device="cuda") != 3] == 4099.0).all())
