"""Sums of squares of vectors and of their kept values in one launch (k_squares), at lengths around a block's tile of
vector elements, a thread's group of eight values and the number of blocks a row gets."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 255, 256, 2047, 2049, 4096, 4097, 70_001])
@pytest.mark.parametrize("n,w", [(70_001, 3), (70_004, 17), (131_072, 2)])
def test_gain_against_float64(n, w, k):
    """Each sum has at most n + k terms, each rounded to float64 once: relative error below (n + k) 2^-53 < 3e-11 of a
    sum of positive terms, and three times that in the quotient."""
    import torch
    import paper_2312_02493_amd as lib

    gen = torch.Generator(device="cuda").manual_seed(n + k)
    x = [torch.randn(n, generator=gen, device="cuda") * (r + 1) for r in range(w)]
    vals = torch.randn(w, k, generator=gen, device="cuda")  # k odd: rows that are not 16-byte aligned
    vals[w - 1] = 0.0
    x[w - 1].zero_()
    gain = torch.full((w,), -1.0, dtype=torch.float64, device="cuda")
    ctx = lib.Context(w, n, max(k, 1))
    ctx.artopk_compression_gain(x, vals, k, gain)
    ctx.status()
    v = vals.double().square().sum(1).cpu().numpy()
    r = np.array([float(a.double().square().sum()) for a in x])
    want = np.divide(v, v + r, out=np.zeros(w), where=v + r > 0.0)
    np.testing.assert_allclose(gain.cpu().numpy(), want, rtol=1e-10)


@pytest.mark.parametrize("k", [1, 2047, 2049, 4097, 39_999])
def test_norms_of_the_kept_values(k):
    """As above: at most k terms a sum."""
    import torch
    import paper_2312_02493_amd as lib

    n, w = 40_001, 5
    gen = torch.Generator(device="cuda").manual_seed(k)
    x = [torch.randn(n, generator=gen, device="cuda") for _ in range(w)]
    idx = torch.full((w * k,), -1, dtype=torch.int32, device="cuda")
    vals = torch.empty(w, k, dtype=torch.float32, device="cuda")
    sq = torch.zeros(w, dtype=torch.float64, device="cuda")
    ctx = lib.Context(w, n, k)
    ctx.artopk_topk_workers(x, k, idx, vals, sq)
    ctx.status()
    np.testing.assert_allclose(sq.cpu().numpy(), vals.double().square().sum(1).cpu().numpy(), rtol=1e-10)
