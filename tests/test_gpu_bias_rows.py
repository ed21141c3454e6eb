"""Bias and LayerNorm rows of widths that are no whole 16-byte pieces, and norms written by the launch that has whole rows."""
import pytest
import torch

from paper_2009_03106_amd import dpclip as dp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("B,T,D", [(1, 1, 1), (3, 7, 31), (5, 8, 33), (2, 31, 65), (4, 33, 10), (9, 447, 940), (3, 1000, 7),      # any width
                                   (3, 5, 8), (2, 64, 128), (128, 65, 128), (40, 33, 512), (2000, 3, 512), (7, 9, 200)])           # whole pieces
def test_rows_and_norms(dtype, B, T, D):
    gen = torch.Generator(device="cuda").manual_seed(T)
    G = torch.randn((B, T, D), device="cuda", generator=gen).to(dtype)
    H = torch.randn((B, T, D), device="cuda", generator=gen).to(dtype)
    g, h = G.double(), H.double()
    u, beta, gamma = g.sum(1), g.sum(1), (g * h).sum(1)
    # float32 sums of up to 1000 numbers of random sign
    tol = dict(rtol=1e-5, atol=1e-4)
    for start in (None, 2.0):
        s = torch.full((B,), start or float("nan"), device="cuda")
        rows = torch.empty((B, D), device="cuda")
        dp.bias_sqnorm(G, s, rows, accumulate=start is not None)
        assert torch.allclose(rows.double(), u, **tol)
        assert torch.allclose(s.double(), u.pow(2).sum(1) + (start or 0.0), rtol=1e-5, atol=1e-4)
        s = torch.full((B,), start or float("nan"), device="cuda")
        _, gr, br = dp.layernorm_sqnorm(G, H, s, accumulate=start is not None)
        assert torch.allclose(gr.double(), gamma, **tol) and torch.allclose(br.double(), beta, **tol)
        assert torch.allclose(s.double(), gamma.pow(2).sum(1) + beta.pow(2).sum(1) + (start or 0.0), rtol=1e-5, atol=1e-4)


def test_more_workgroups_than_a_launch_holds():
    """65535 examples of 8225 columns in pieces of 32: 2^24 workgroups are passed."""
    G = torch.ones((65535, 1, 8225), device="cuda", dtype=torch.bfloat16)
    G[-1] = 2.0
    s = torch.zeros(65535, device="cuda")
    rows = torch.empty((65535, 8225), device="cuda")
    dp.bias_sqnorm(G, s, rows)
    assert bool((rows[:-1] == 1.0).all()) and bool((rows[-1] == 2.0).all())
    assert bool((s[:-1] == 8225.0).all()) and float(s[-1]) == 4.0 * 8225.0
