"""Norms of more examples than the workgroups of one launch."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu


def _ones(B, T, a, b, dtype):
    A, G = torch.ones((B, T, a), device="cuda", dtype=dtype), torch.ones((B, T, b), device="cuda", dtype=dtype)
    A[-1] = 2.0
    return A, G


# every product of ones is exact: T^2 a b, and four times that for the last example
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,path", [((1 << 24) + 3, "direct"), ((1 << 23) + 5, "gram"), ((1 << 24) + 3, "gram")])
def test_short_examples(dtype, B, path):
    A, G = _ones(B, 2, 8, 2, dtype)
    want = 4.0 * 16.0
    s = dp.layer_sqnorm(A, G, path=path)
    assert bool((s[:-1] == want).all()) and float(s[-1]) == 4 * want
    # two layers: their sums are added up by one launch
    s, clip = torch.full((B,), float("nan"), device="cuda"), torch.zeros(B, device="cuda")
    dp.layers_sqnorm([(A, G), (A, G)], s, path=path, C=1.0, clip=clip)
    assert bool((s[:-1] == 2 * want).all()) and float(s[-1]) == 8 * want
    assert torch.allclose(clip, s.sqrt().reciprocal(), rtol=1e-6, atol=0)


def test_several_sums_an_example():
    """Three sums of 128 x 128 positions each, widths of 8 (as a launch of 256 threads: 2^24 workgroups less 7)."""
    B = 5592403
    A = torch.ones((B, 129, 8), device="cuda", dtype=torch.bfloat16)
    A[-1] = 2.0
    s = dp.layer_sqnorm(A, A, path="gram")
    want = (129.0 * 8.0) ** 2
    assert bool((s[:-1] == want).all()) and float(s[-1]) == 16 * want


def test_groups_and_biases_in_pieces():
    """Arrays of their own, bias rows and scratch of the queried size, in pieces of the examples."""
    B = (1 << 22) + 100
    A, G = _ones(B, 2, 8, 2, torch.bfloat16)
    own, rows, s = torch.zeros(B, device="cuda"), torch.zeros((B, 2), device="cuda"), torch.zeros(B, device="cuda")
    descs = dp.layer_descs([(A, G), (A, G)], bias_rows=[rows, None], groups=[(own, None, 0.0), None])
    need = dp.layers_workspace_bytes(descs[0], B, descs[2])
    ws = torch.full((need + 4096,), 7, dtype=torch.uint8, device="cuda")
    dp.layers_sqnorm([(A, G), (A, G)], s, workspace=ws[:need], descs=descs)
    assert bool((rows == 2.0).all()) and bool((s[:-1] == 64.0).all()) and float(s[-1]) == 256.0
    assert bool((own[:-1] == 64.0 + 8.0).all()) and float(own[-1]) == 256.0 + 8.0
    assert bool((ws[need:] == 7).all())
