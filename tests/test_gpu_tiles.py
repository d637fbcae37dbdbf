"""GPU parity of the selection by marked tiles (k_mark_tiles and what follows it): flat steps whose leader is known up
front, and segments, bit for bit against the oracle.  The length from which it is used is lowered through
ARTOPK_OPT_GUESS_MIN_N; the sizes lie around a tile's 16384 elements, pairs and groups of tiles and a float4 group,
and the values are those for which a sampled bound, a tile's piece or the narrow bins do not do."""

import numpy as np
import pytest

import artopk_inputs as inp
from oracle import artopk_oracle as orc
from tests import gpu_util
from tests.gpu_util import GpuRunner, assert_step_matches

pytestmark = pytest.mark.gpu
TILE = 32768


@pytest.fixture(autouse=True)
def tiles_on(monkeypatch):
    monkeypatch.setitem(gpu_util.OPTIONS, "guess_min_n", 4096)
    monkeypatch.setitem(gpu_util.OPTIONS, "stage_tiles", 2)
    monkeypatch.setitem(gpu_util.OPTIONS, "short_max_n", 0)


def _values(kind, n, rng):
    x = rng.standard_normal(n).astype(np.float32)
    if kind == "normal":
        return x
    if kind == "equal":
        return np.full(n, -0.375, dtype=np.float32)
    if kind == "zeros":
        return np.where(rng.random(n) < 1e-3, x, 0.0).astype(np.float32)
    if kind == "ties":  # a few hundred values, so that the threshold is one of them
        return (np.round(x * 32.0) / 32.0).astype(np.float32)
    if kind == "run":  # tiles with more marks than a piece takes, and a sample that sees few of them
        x *= np.float32(1e-3)
        lo = n // 3
        x[lo:lo + n // 20] += np.float32(2.0)
        return x
    if kind == "sorted":
        return np.sort(np.abs(x))
    if kind == "narrow":  # all in one top digit
        return (1.0 + 0.06 * rng.random(n)).astype(np.float32)
    if kind == "steps":  # a few hundred neighbouring values, a few thousand times each: bins of a few keys
        return (1.0 + rng.integers(0, 300, n) * 2.0 ** -23).astype(np.float32)
    if kind == "odd":  # infinities, NaNs of either sign, negative zeros and denormals
        x[::977] = np.inf
        x[5::1931] = -np.inf
        x[3::2003] = np.float32(np.nan)
        x[7::2003] = -np.float32(np.nan)
        x[2::11] = -0.0
        x[4::13] = np.float32(1e-41)
        return x
    raise ValueError(kind)


def _by_tiles(ctx, bounds=None):
    """The selection went by tiles, and so many of its segments' bounds held."""
    info = ctx.select_info()
    assert gpu_util.FORCED or info["tiles"] == 1, info
    assert gpu_util.FORCED or bounds is None or info["tile_bounds"] == bounds, info


def _steps(w, n, k, mode, gen, steps=2, seg_off=None, seg_k=None, max_k=None, bounds=None):
    runner = GpuRunner(w, n, max_k or k, max_segments=len(seg_k) if seg_k else 1)
    res = [np.zeros(n, dtype=np.float32) for _ in range(w)]
    for step_no in range(1, steps + 1):
        g = [gen(step_no, r) for r in range(w)]
        with np.errstate(all="ignore"):
            want = orc.step(g, res, k, mode, step_no=step_no, seg_off=seg_off, seg_k=seg_k)
        runner.load_g(g)
        got = runner.step(k, mode, step_no, seg_off=seg_off, seg_k=seg_k)
        if bounds != "other":
            _by_tiles(runner.ctx, bounds)
        assert_step_matches(got, want, mode)
        res = want.residual
    return runner


@pytest.mark.parametrize("n", [16384, TILE - 1, TILE, TILE + 1, 16 * TILE - 2, 16 * TILE + 5, 33 * TILE + 31])
@pytest.mark.parametrize("rho", [0.001, 0.02, 0.12])
def test_flat_lengths(n, rho):
    rng = np.random.default_rng(n)
    # (one tile's sample is too small to say that one in eight fits a piece)
    bounds = "other" if (n, rho) == (16384, 0.12) else 1
    _steps(2, n, max(1, int(n * rho)), orc.MODE_STAR, lambda s, r: _values("normal", n, rng), bounds=bounds)


@pytest.mark.parametrize("one_in,tiles", [(8, 1), (7, 1), (6.5, 0)])
def test_flat_density(one_in, tiles):
    """Up to one in seven kept a piece holds a tile's share."""
    n = 33 * TILE + 31
    rng = np.random.default_rng(11)
    runner = _steps(2, n, int(n / one_in), orc.MODE_STAR, lambda s, r: _values("normal", n, rng), bounds=1 if tiles else "other")
    assert gpu_util.FORCED or runner.ctx.select_info()["tiles"] == tiles


@pytest.mark.parametrize("kind", ["equal", "zeros", "ties", "run", "sorted", "narrow", "steps", "odd"])
@pytest.mark.parametrize("rho", [0.005, 0.1])
def test_flat_values(kind, rho):
    n = 19 * TILE + 3
    rng = np.random.default_rng(3)
    # (of a few hundred values the sample's bound is one, and whether it holds is chance)
    bounds = {"equal": 0, "zeros": 0, "steps": None}.get(kind, 1)
    _steps(2, n, int(n * rho), orc.MODE_STAR, lambda s, r: _values(kind, n, rng), steps=1 if kind == "odd" else 2, bounds=bounds)


@pytest.mark.parametrize("n,one_in,tiles", [(167_700_000, 3000, 1), (167_900_000, 3000, 0), (167_900_000, 499, 1)])
def test_long_sparse_steps_leave_the_mask_instead(n, one_in, tiles):
    """Without switches set; the result is the other route's."""
    import paper_2312_02493_amd as lib
    import torch

    k = n // one_in
    g = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(10), device="cuda")
    got = []
    for stage_tiles in (1, 2 - 2 * tiles):
        ctx = lib.Context(1, n, k)
        ctx.set_option(lib.ARTOPK_OPT_STAGE_TILES, stage_tiles)
        res, idx, total = torch.zeros(n, device="cuda"), torch.full((k,), -1, dtype=torch.int32, device="cuda"), torch.zeros(k, device="cuda")
        ctx.artopk_step([g], [res], k, orc.MODE_STAR, 1, idx, total, None)
        ctx.status()
        info = ctx.select_info()
        assert (info["guessed"], info["from_mask"]) == (1, 1)
        got.append((info["tiles"], idx, total, res))
    assert (got[0][0], got[1][0]) == (tiles, 1 - tiles)
    assert all(torch.equal(a, b) for a, b in zip(got[0][1:], got[1][1:]))
    assert torch.equal(got[0][2], g[got[0][1].long()]) and int((got[0][3] == 0).sum()) >= k


def _layout(name):
    if name == "buckets":  # whole tiles, the last one ragged
        return [0, 4 * TILE, 8 * TILE, 12 * TILE, 14 * TILE + 77]
    if name == "layers":  # none at a tile's edge, a few too short to be sampled, elements of two segments in one group
        return [0, 13, 40, 700, 40_003, 40_070, 300_001, 300_002, 420_420, 800_001, 1_100_003]
    if name == "two":
        return [0, 17 * TILE + 9, 40 * TILE]
    if name == "edges":  # around lines of 32 elements and tiles
        return [0, TILE - 1, TILE + 1, 2 * TILE + 31, 2 * TILE + 32, 3 * TILE + 33, 20 * TILE]
    raise ValueError(name)


@pytest.mark.parametrize("layout", ["buckets", "layers", "two", "edges"])
@pytest.mark.parametrize("mode", ["star", "var"])
@pytest.mark.parametrize("rho", [0.01, 0.2])
def test_segments(layout, mode, rho):
    off = _layout(layout)
    ks = [max(1, int(np.ceil(rho * (b - a)))) for a, b in zip(off, off[1:])]
    n, w = off[-1], 3
    wl = inp.workload(2, n=n, w=w)
    # (too short to be sampled: 13, 27 and one element in "layers", one of two and one of one in "edges"; more than one in
    # six kept: too many marks for a tile's piece)
    bounds = {"buckets": 4, "layers": 7, "two": 2, "edges": 4}[layout] if rho < 0.2 else 0 if layout != "layers" else None
    _steps(w, n, sum(ks), orc.MODE_STAR if mode == "star" else orc.MODE_VAR, wl.gen, seg_off=off, seg_k=ks, bounds=bounds)


@pytest.mark.parametrize("kind", ["equal", "zeros", "ties", "run", "sorted", "narrow", "steps", "odd"])
@pytest.mark.parametrize("layout", ["buckets", "layers"])
def test_segment_values(kind, layout):
    off = _layout(layout)
    ks = [max(1, (b - a) // 40) for a, b in zip(off, off[1:])]
    rng = np.random.default_rng(4)
    _steps(2, off[-1], sum(ks), orc.MODE_STAR, lambda s, r: _values(kind, off[-1], rng), seg_off=off, seg_k=ks,
           steps=1 if kind == "odd" else 2)


@pytest.mark.parametrize("values", ["normal", "run"])
def test_segments_keep_everything_or_one(values):
    off = _layout("layers")
    ks = [1 if i % 2 else b - a for i, (a, b) in enumerate(zip(off, off[1:]))]
    rng = np.random.default_rng(5)
    _steps(2, off[-1], sum(ks), orc.MODE_STAR, lambda s, r: _values(values, off[-1], rng), seg_off=off, seg_k=ks)


@pytest.mark.parametrize("layout", ["buckets", "layers", "edges"])
def test_segmented_selection_alone(layout):
    """artopk_select_topk on segments, twice on one context with another layout in between."""
    import torch

    off = _layout(layout)
    n = off[-1]
    ks = [max(1, (b - a) // 50) for a, b in zip(off, off[1:])]
    x = _values("ties", n, np.random.default_rng(6))
    ctx = gpu_util.make_context(1, n, sum(ks), max(2, len(ks)))
    t = torch.from_numpy(x).cuda()
    idx = torch.full((sum(ks),), -1, dtype=torch.int32, device="cuda")
    half = [0, n // 2, n]
    for o, q in ((off, ks), (half, [3, 5]), (off, ks)):
        idx.fill_(-1)
        ctx.artopk_select_topk(t, sum(q), idx, seg_off=o, seg_k=q)
        ctx.status()
        _by_tiles(ctx)
        want = np.concatenate([orc.topk_indices(x[a:b], m) + a for a, b, m in zip(o, o[1:], q)])
        assert np.array_equal(idx[: sum(q)].cpu().numpy(), want)
        assert np.array_equal(t.cpu().numpy(), x)


def _parts(n, m):
    return [n * i // m for i in range(m + 1)]


# lengths and layouts on either side of the lines from which segments go by tiles, (offsets, one in so many kept of each): few
# and many segments, one as long as all others together, and segments too dense for pieces: short ones, a part of the
# elements, all of them, and all but one of very different sizes
M = 1_000_000
_DEFAULTS = {
    "8.4m-two": ([0, 8_399_000, 8_400_000], None, 1),
    "8.4m-three": (_parts(8_400_000, 3), None, 0),
    "8.4m-half": ([0, 4_300_000, 6_000_000, 8_400_000], None, 1),
    "8.3m-half": ([0, 8_000_000, 8_300_000], None, 0),
    "11m-twenty": (_parts(11 * M, 20), None, 1),
    "11m-fifty": (_parts(11 * M, 50), None, 0),
    "16m-hundred": (_parts(16 * M, 100), None, 1),
    "16m-many": (_parts(16 * M, 250), None, 0),
    "16m-some-dense": (_parts(16 * M, 16), lambda i: 5 if i == 3 else 100, 0),
    "16m-short-dense": ([0, 500, 1000, 16 * M], lambda i: 4 if i < 2 else 100, 1),
    "16m-tile-dense": ([0, 2000, 16 * M], lambda i: 4 if i < 1 else 100, 0),
    "26m-tile-dense": ([0, 16_000, 26 * M], lambda i: 4 if i < 1 else 100, 1),
    "26m-tiles-dense": ([0, 26 * M, 26 * M + 33_000], lambda i: 4 if i > 0 else 100, 0),
    "16m-one-in-eight": (_parts(16 * M, 8), lambda i: 8, 1),
    "26m-some-dense": (_parts(26 * M, 8), lambda i: 5 if i == 3 else 100, 0),
    "26m-all-dense": (_parts(26 * M, 8), lambda i: 5, 0),
    "26m-half-kept": (_parts(26 * M, 8), lambda i: 2, 1),
    "26m-uneven": ([0, 20 * M] + [20 * M + 200_000 * (i + 1) for i in range(30)], lambda i: 5, 1),
    "26m-many": (_parts(26 * M, 520), lambda i: 5, 1),
    "101m-some-dense": (_parts(101 * M, 8), lambda i: 5 if i == 3 else 100, 1),
    "101m-more-dense": (_parts(101 * M, 8), lambda i: 5 if i % 2 else 100, 0),
}


@pytest.mark.parametrize("name", sorted(_DEFAULTS))
def test_which_segments_go_by_tiles(name):
    """Without switches set; the results are those of the other route."""
    import paper_2312_02493_amd as lib
    import torch

    off, one_in, tiles = _DEFAULTS[name]
    ks = [-(-(b - a) // (one_in(i) if one_in else 100)) for i, (a, b) in enumerate(zip(off, off[1:]))]
    n, k = off[-1], sum(ks)
    x = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(9), device="cuda")
    got = []
    for guess_min_n in (None, 1 << 31 if tiles else 4096):
        ctx = lib.Context(1, n, k, len(ks))
        if guess_min_n:
            ctx.set_option(lib.ARTOPK_OPT_GUESS_MIN_N, guess_min_n)
        idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")
        ctx.artopk_select_topk(x, k, idx, seg_off=off, seg_k=ks)
        ctx.status()
        got.append((ctx.select_info()["tiles"], idx))
    assert (got[0][0], got[1][0]) == (tiles, 1 - tiles)
    assert torch.equal(got[0][1], got[1][1])
    a, b = off[-2], off[-1]
    assert np.array_equal(got[0][1][k - ks[-1]:].cpu().numpy(), orc.topk_indices(x[a:b].cpu().numpy(), ks[-1]) + a)


@pytest.mark.parametrize("stage_tiles", [0, 1, 2])
def test_the_switch_holds_for_segments(stage_tiles):
    import paper_2312_02493_amd as lib
    import torch

    off = _layout("layers")
    n, ks = off[-1], [max(1, (b - a) // 50) for a, b in zip(off, off[1:])]
    k = sum(ks)
    ctx = gpu_util.make_context(2, n, k, len(ks))
    ctx.set_option(lib.ARTOPK_OPT_STAGE_TILES, stage_tiles)
    x = _values("normal", n, np.random.default_rng(12))
    t = torch.from_numpy(x).cuda()
    idx, total = torch.zeros(k, dtype=torch.int32, device="cuda"), torch.zeros(k, device="cuda")
    want = np.concatenate([orc.topk_indices(x[a:b], m) + a for a, b, m in zip(off, off[1:], ks)])
    for call in ("select", "var", "star"):
        idx.fill_(-1)
        if call == "select":
            ctx.artopk_select_topk(t, k, idx, seg_off=off, seg_k=ks)
        else:
            res = [torch.zeros(n, device="cuda") for _ in range(2)]
            ctx.artopk_step([0.5 * t, t], res, k, orc.MODE_VAR if call == "var" else orc.MODE_STAR, 1, idx, total, None,
                            seg_off=off, seg_k=ks)
        ctx.status()
        assert ctx.select_info()["tiles"] == (1 if stage_tiles else 0), call
        assert np.array_equal(idx.cpu().numpy(), want)


def test_what_select_info_says_behind_a_selection_in_one_launch():
    """A segmented selection takes many launches, whatever the call before it took."""
    import torch

    off, ks = _layout("two"), [3000, 5000]
    n = off[-1]
    ctx = gpu_util.make_context(2, n, sum(ks), 2)
    x = torch.from_numpy(_values("normal", n, np.random.default_rng(7))).cuda()
    g, res = [x, 2 * x], [torch.zeros(n, device="cuda") for _ in range(2)]
    idx, total = torch.zeros(sum(ks), dtype=torch.int32, device="cuda"), torch.zeros(sum(ks), device="cuda")
    update = torch.zeros(n, device="cuda")
    for call in ("select", "var", "star"):
        ctx.artopk_select_topk(x, 4000, idx)
        assert gpu_util.FORCED or ctx.select_info()["one_launch"] == 1
        if call == "select":
            ctx.artopk_select_topk(x, sum(ks), idx, seg_off=off, seg_k=ks)
        else:
            ctx.artopk_step(g, res, sum(ks), orc.MODE_VAR if call == "var" else orc.MODE_STAR, 1, idx, total, update, seg_off=off,
                            seg_k=ks)
        assert gpu_util.FORCED or ctx.select_info()["one_launch"] == 0, call


def _kernels_of(call):
    import torch
    from torch.profiler import ProfilerActivity, profile

    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    names = [e.key for e in prof.key_averages()]
    if not names:
        pytest.skip("no kernel trace here")
    return names


def test_the_map_of_a_layouts_tiles_is_made_when_it_is_first_wanted():
    """Not for layouts that do not go by tiles, once for one that does, and for a layout that the context knows already when
    the length is lowered behind its back, also in a recorded call, whose replays leave eager calls as they were."""
    import torch

    off = _layout("layers")
    n, ks = off[-1], [max(1, (b - a) // 50) for a, b in zip(off, off[1:])]
    k, half = sum(ks), [0, n // 2, n]
    x = _values("ties", n, np.random.default_rng(6))
    want = np.concatenate([orc.topk_indices(x[a:b], m) + a for a, b, m in zip(off, off[1:], ks)])
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        t = torch.from_numpy(x).cuda()
        idx = torch.full((k,), -1, dtype=torch.int32, device="cuda")

        def select(ctx, o=off, q=ks):
            idx.fill_(-1)
            ctx.artopk_select_topk(t, sum(q), idx, seg_off=o, seg_k=q)

        def check(ctx):
            ctx.status()
            assert np.array_equal(idx.cpu().numpy(), want)

        for recorded in (False, True):
            ctx = gpu_util.make_context(1, n, k, len(ks), stream=side.cuda_stream)
            ctx.set_option(0, n + 1)
            names = _kernels_of(lambda: select(ctx))
            assert any("k_final" in s for s in names), names  # (they are seen)
            assert not any("k_tile" in s for s in names), names
            check(ctx)
            ctx.set_option(0, 4096)
            if recorded:
                side.synchronize()
                graph = torch.cuda.CUDAGraph()
                with torch.cuda.graph(graph, stream=side):
                    ctx.artopk_select_topk(t, k, idx, seg_off=off, seg_k=ks)
            for i in range(3):
                if recorded:
                    idx.fill_(-1)
                    graph.replay()
                    check(ctx)
                names = _kernels_of(lambda: select(ctx))
                assert any("k_mark_tiles" in s for s in names) and any("k_tile_map" in s for s in names) == (i == 0), names
                check(ctx)
            select(ctx, half, [3, 5])
            select(ctx)
            check(ctx)


@pytest.mark.parametrize("gtype", ["bf16", "f16"])
@pytest.mark.parametrize("layout", [None, "layers"])
def test_16_bit_gradients(gtype, layout):
    import torch

    off = _layout(layout) if layout else None
    n, w = (off[-1] if off else 20 * TILE + 3), 2
    ks = [max(1, (b - a) // 30) for a, b in zip(off, off[1:])] if off else None
    k = sum(ks) if ks else n // 30
    dtype = torch.bfloat16 if gtype == "bf16" else torch.float16
    runner = GpuRunner(w, n, k, max_segments=len(ks) if ks else 1)
    rng = np.random.default_rng(8)
    res = [np.zeros(n, dtype=np.float32) for _ in range(w)]
    for step_no in (1, 2):
        g16 = [torch.from_numpy(_values("normal", n, rng)).to(dtype).cuda() for _ in range(w)]
        g = [t.float().cpu().numpy() for t in g16]
        want = orc.step(g, res, k, orc.MODE_STAR, step_no=step_no, seg_off=off, seg_k=ks)
        more = {"seg_off": off, "seg_k": ks} if off else {}
        runner.ctx.artopk_step_g16(g16, runner.lib.ARTOPK_G_BF16 if gtype == "bf16" else runner.lib.ARTOPK_G_F16, runner.res, k,
                                   orc.MODE_STAR, step_no, runner.idx, runner.sum, runner.update, leader_out=runner.leader,
                                   **more)
        runner.ctx.status()
        _by_tiles(runner.ctx, 7 if off else 1)
        assert np.array_equal(runner.idx[:k].cpu().numpy(), want.idx)
        assert np.array_equal(gpu_util.bits(runner.sum[:k].cpu().numpy()), gpu_util.bits(want.sum))
        assert np.array_equal(gpu_util.bits(runner.update.cpu().numpy()), gpu_util.bits(want.update))
        for r in range(w):
            assert np.array_equal(gpu_util.bits(runner.res[r].cpu().numpy()), gpu_util.bits(want.residual[r]))
        res = want.residual
