"""The selection at the sizes where its kernels' tiles, chunks and copies meet: against the oracle, bit for bit."""

import numpy as np
import pytest

from oracle import artopk_oracle as orc

pytestmark = pytest.mark.gpu


def _values(rng, n, kind):
    x = (rng.standard_normal(n) * 0.01).astype(np.float32)
    if kind == "ties":
        x[rng.integers(0, n, n // 3)] = np.float32(-0.0125)
    elif kind == "special":  # infinities, NaN, zeros and the smallest denormal
        x[rng.integers(0, n, 40)] = np.inf
        x[rng.integers(0, n, 40)] = -np.nan
        x[rng.integers(0, n, n // 4)] = 0.0
        x[rng.integers(0, n, n // 4)] = np.float32(1e-45)
    return x


# one chunk more than a single copy of the whole-range histogram serves, one less, a ragged last group, the
# largest vector whose list holds everything and one element more, one tile of the fused pass and its neighbours
@pytest.mark.parametrize("n", [32767, 32769, 128 * 8192, 128 * 8192 + 1, 129 * 8192 + 3, (1 << 22), (1 << 22) + 5])
@pytest.mark.parametrize("kind", ["normal", "ties", "special"])
def test_stand_alone_selection(n, kind):
    import torch
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n)
    x = _values(rng, n, kind)
    xd = torch.from_numpy(x).cuda()
    ctx = lib.Context(1, n, n // 2)
    for k in (1, n // 700 + 1, n // 9, n // 2):
        idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
        ctx.artopk_select_topk(xd, k, idx)
        ctx.status()
        assert np.array_equal(idx.cpu().numpy(), orc.topk_indices(x, k)), (n, k)


@pytest.mark.parametrize("start", [0, 1, 2, 3, 5, 8191])
def test_segments_that_begin_and_end_inside_a_group(start):
    import torch
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(start)
    sizes = ([start] if start else []) + [1, 2, 3, 4, 5, 6, 7, 8, 9, 8190, 8193, 2, 32766, 32771, 1, 300_001, 3]
    off = np.concatenate([[0], np.cumsum(sizes)])
    n = int(off[-1])
    x = _values(rng, n, "ties")
    ks = [max(1, s // 3) for s in sizes]
    xd = torch.from_numpy(x).cuda()
    ctx = lib.Context(1, n, sum(ks), max_segments=len(sizes))
    idx = torch.full((sum(ks),), -1, dtype=torch.int32, device="cuda")
    ctx.artopk_select_topk(xd, sum(ks), idx, seg_off=[int(o) for o in off], seg_k=ks)
    ctx.status()
    assert np.array_equal(idx.cpu().numpy(), orc.topk_indices_segmented(x, [int(o) for o in off], ks))


# kept entries around one tile of the final list pass (4096 entries, 8192 for long lists), and enough of them
# for the longer tile; a plateau of equal values at the threshold is cut by the tie quota inside a tile
@pytest.mark.parametrize("k", [1, 7, 8, 4095, 4096, 4097, 8192 * 3 + 1, (1 << 19), (1 << 19) + 1, 1_300_001])
def test_final_list_pass_tiles_and_quota(k):
    import torch
    import paper_2312_02493_amd as lib

    n = 2_000_003
    rng = np.random.default_rng(k)
    x = (rng.standard_normal(n) * 1e-3).astype(np.float32)
    x[rng.permutation(n)[:k // 2]] += np.float32(1.0)                    # above the plateau
    free = np.flatnonzero(x < 0.5)
    x[rng.permutation(free)[:k]] = np.float32(-0.25)                     # twice as many as are still needed
    xd = torch.from_numpy(x).cuda()
    ctx = lib.Context(1, n, k)
    idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
    ctx.artopk_select_topk(xd, k, idx)
    ctx.status()
    assert np.array_equal(idx.cpu().numpy(), orc.topk_indices(x, k))


@pytest.mark.parametrize("w,n", [(1, 134_217_728), (1, 134_217_732), (3, 44_739_245), (2, 1023)])
def test_gain_and_variance_on_both_sides_of_the_cache_limit(w, n):
    """float64 sums in another order: relative difference below n rounding errors of 2^-53, 1e-9 at these sizes."""
    import torch
    import paper_2312_02493_amd as lib

    gen = torch.Generator(device="cuda").manual_seed(n)
    x = [torch.randn(n, generator=gen, device="cuda") for _ in range(w)]
    vals = torch.randn(w, 500, generator=gen, device="cuda")
    ctx = lib.Context(w, n, 500)
    out, gain = (torch.zeros(w, dtype=torch.float64, device="cuda") for _ in range(2))
    ctx.artopk_variance(x, out)
    ctx.artopk_compression_gain(x, vals, 500, gain)
    ctx.status()
    for r in range(w):
        d = x[r].double()
        v = float(vals[r].double().square().sum())
        np.testing.assert_allclose(float(out[r]), float(d.var(correction=0)), rtol=1e-9)
        np.testing.assert_allclose(float(gain[r]), v / (v + float(d.square().sum())), rtol=1e-9)
