"""Launches whose blocks wait for each other, when two blocks in three start 100 us late: the others take on their work,
and every result is the oracle's.  And waits that expire: an error, and the next call on the context is right again."""

import ctypes as C

import numpy as np
import pytest

from oracle import artopk_oracle as orc
from tests import gpu_util, test_gpu_tiles
from tests.gpu_util import GpuRunner, assert_step_matches, bits

pytestmark = pytest.mark.gpu

LATE = 10_000  # of 10 ns
LOOKS = 1 << 20


@pytest.fixture
def held(monkeypatch):
    """Contexts of the library built for this; held(ticks, looks) sets it up and returns the units that were taken on."""
    import torch
    from paper_2312_02493_amd import binding, build

    assert torch.cuda.is_available()  # (before the library brings in the runtime: both are to use torch's)
    monkeypatch.setattr(binding, "lib_path", lambda: build.HELD_PATH)
    monkeypatch.setattr(binding, "_lib", None)
    fn = binding.load_library().artopk_held_blocks
    fn.argtypes = [C.c_uint32, C.c_uint32, C.POINTER(C.c_uint32)]

    def call(ticks, looks):
        helped = C.c_uint32()
        assert fn(ticks, looks & 0xffffffff, C.byref(helped)) == 0
        return helped.value

    call(0, LOOKS)
    yield call
    call(0, LOOKS)


def _values(rng, n, kind, r):
    x = (rng.standard_normal(n) * 0.01 * (1.0 + 0.3 * r)).astype(np.float32)
    if kind == "ties":
        x = (np.round(x * 512) / 512).astype(np.float32)
    return x


# one chunk a block and every chunk its own workers' (a leader known up front), chunks whose workers are shared out among
# further blocks (many workers; a leader found on the device), several steps in turn on one context
@pytest.mark.parametrize("n,w,mode", [(300_002, 3, orc.MODE_STAR), (65_537, 40, orc.MODE_STAR), (65_537, 8, orc.MODE_VAR),
                                      (700_001, 2, orc.MODE_VAR), (5_000, 2, orc.MODE_STAR)])
@pytest.mark.parametrize("kind", ["normal", "ties"])
def test_short_steps(held, n, w, mode, kind):
    rng = np.random.default_rng(n)
    k = n // 50
    runner = GpuRunner(w, n, k)
    res = [np.zeros(n, np.float32) for _ in range(w)]
    runner.load_res(res)
    for step_no in range(1, 6):
        g = [_values(rng, n, kind, r) for r in range(w)]
        want = orc.step(g, res, k, mode, step_no=step_no)
        runner.load_g(g)
        held(0 if step_no == 3 else LATE, LOOKS)
        assert_step_matches(runner.step(k, mode, step_no, want_vals=step_no % 2 == 1), want, mode)
        assert runner.ctx.select_info()["short"] == 1
        assert step_no == 3 or held(0, LOOKS) > 0
        res = want.residual


# the one-launch selection behind a pass
@pytest.mark.parametrize("n", [600_001, 4_000_003])
@pytest.mark.parametrize("kind", ["normal", "ties"])
def test_selection_behind_a_pass(held, n, kind):
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n)
    w, k = 2, n // 50
    runner = GpuRunner(w, n, k)
    runner.ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, 0)
    res = [np.zeros(n, np.float32) for _ in range(w)]
    runner.load_res(res)
    for step_no in (1, 2, 3):
        g = [_values(rng, n, kind, r) for r in range(w)]
        want = orc.step(g, res, k, orc.MODE_VAR, step_no=step_no)
        runner.load_g(g)
        held(LATE, LOOKS)
        assert_step_matches(runner.step(k, orc.MODE_VAR, step_no), want, orc.MODE_VAR)
        assert runner.ctx.select_info()["one_launch"] == 1 and held(0, LOOKS) > 0
        res = want.residual


# several vectors at a time: behind nothing, behind a marking whose bound holds, and behind one whose bound does not
@pytest.mark.parametrize("kind,guess,from_mask", [("normal", None, 0), ("ties", None, 0), ("normal", 4096, 1),
                                                  ("ties", 4096, 1), ("equal", 4096, 0)])
def test_selections_of_whole_vectors(held, kind, guess, from_mask):
    import torch
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(3)
    n, w = 500_003, 3
    k = n // 100
    xs = [_values(rng, n, kind, r) if kind != "equal" else np.full(n, np.float32(0.5 + r)) for r in range(w)]
    xd = [torch.from_numpy(x).cuda() for x in xs]
    ctx = lib.Context(w, n, k)
    if guess:
        ctx.set_option(lib.ARTOPK_OPT_GUESS_MIN_N, guess)
    for _ in range(3):
        idx = torch.full((w, k), -1, dtype=torch.int32, device="cuda")
        vals = torch.zeros(w, k, device="cuda")
        torch.cuda.synchronize()
        held(LATE, LOOKS)
        ctx.artopk_topk_workers(xd, k, idx, vals)
        ctx.status()
        info = ctx.select_info()
        assert (info["one_launch"], info["guessed"], info["from_mask"]) == (1, 1 if guess else 0, from_mask), info
        assert held(0, LOOKS) > 0
        for r in range(w):
            want = orc.topk_indices(xs[r], k)
            assert np.array_equal(idx[r].cpu().numpy(), want)
            assert np.array_equal(bits(vals[r].cpu().numpy()), bits(xs[r][want]))


@pytest.fixture
def tiles_on(held, monkeypatch):
    for name, value in (("guess_min_n", 4096), ("stage_tiles", 2), ("short_max_n", 0)):
        monkeypatch.setitem(gpu_util.OPTIONS, name, value)
    return held


# the sample of a selection by tiles waits for its blocks once: late ones, none that waits at all, and one look each, so that
# most leave and the last ones still pick (nobody is the last one through, then); a vector without a bound is an ordinary one
@pytest.mark.parametrize("ticks,looks,bound", [(LATE, LOOKS, 1), (0, -1, 0), (LATE, -1, 0), (LATE, 1, 0)])
@pytest.mark.parametrize("kind", ["normal", "ties"])
def test_sample_of_marked_tiles(tiles_on, ticks, looks, bound, kind):
    rng = np.random.default_rng(looks & 7)
    n, w = 1_100_003, 2
    k = n // 60
    runner = GpuRunner(w, n, k)
    res = [np.zeros(n, np.float32) for _ in range(w)]
    runner.load_res(res)
    for step_no in (1, 2, 3):
        g = [_values(rng, n, kind, r) for r in range(w)]
        want = orc.step(g, res, k, orc.MODE_STAR, step_no=step_no)
        runner.load_g(g)
        tiles_on(ticks if step_no != 2 else 0, looks if step_no != 2 else LOOKS)
        assert_step_matches(runner.step(k, orc.MODE_STAR, step_no), want, orc.MODE_STAR)
        info = runner.ctx.select_info()
        assert (info["tiles"], info["from_mask"]) == (1, bound if step_no != 2 else 1), (step_no, info)
        res = want.residual


# the form for many tiles, a block's side by side (here from 17 on): flat and in segments, whose blocks' counts begin behind
# other segments', with tiles that have no piece, bounds that do not hold and none
# (under the variance rule flat selections do not go by tiles, and who leads has to be beyond doubt)
_BESIDE = [(layout, kind, mode) for layout in (None, "buckets", "layers", "two", "edges")
           for kind in ("normal", "equal", "zeros", "ties", "run", "sorted", "steps", "odd") for mode in ("star", "var")
           if mode == "star" or (layout is not None and kind not in ("equal", "odd"))]


@pytest.mark.parametrize("layout,kind,mode", _BESIDE)
def test_tiles_side_by_side(tiles_on, layout, kind, mode):
    tiles_on(0, LOOKS)
    off = test_gpu_tiles._layout(layout) if layout else None
    n = off[-1] if off else 21 * 32768 + 3
    ks = [max(1, (b - a) // 40) for a, b in zip(off, off[1:])] if off else None
    rng = np.random.default_rng(14)
    scale = (1.0, 1.5) if mode == "var" else (1.0, 1.0)
    test_gpu_tiles._steps(2, n, sum(ks) if ks else n // 40, orc.MODE_STAR if mode == "star" else orc.MODE_VAR,
                          lambda s, r: test_gpu_tiles._values(kind, n, rng) * np.float32(scale[r]), steps=1 if kind == "odd" else 2,
                          seg_off=off, seg_k=ks)


@pytest.mark.parametrize("dense", [20, 5, 2])
def test_tiles_side_by_side_of_dense_segments(tiles_on, dense):
    tiles_on(0, LOOKS)
    off = test_gpu_tiles._layout("layers")
    n, ks = off[-1], [-(-(b - a) // (dense if i % 2 else 50)) for i, (a, b) in enumerate(zip(off, off[1:]))]
    rng = np.random.default_rng(15)
    runner = test_gpu_tiles._steps(2, n, sum(ks), orc.MODE_STAR, lambda s, r: _values(rng, n, "normal", r), seg_off=off, seg_k=ks)
    runner.load_res([np.zeros(n, np.float32)] * 2)
    names = test_gpu_tiles._kernels_of(lambda: runner.step(sum(ks), orc.MODE_STAR, 1, seg_off=off, seg_k=ks))
    assert any("k_tiles_out<false>" in s for s in names), names


# beside a stream of copies most blocks start late: with a long wait before each unit that the others take on, a
# selection of 72 us took 345 (130 now, 157 by one kernel after the other; 3 leaves room for the clock)
def test_selection_beside_copies():
    import torch
    import paper_2312_02493_amd as lib

    n = 25_557_032
    k = n // 100
    x = torch.randn(n, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    a, b = (torch.zeros(1 << 28, device="cuda") for _ in range(2))
    want = None
    side = torch.cuda.Stream()
    best = {}
    with torch.cuda.stream(side):
        ctx = lib.Context(1, n, k, stream=side.cuda_stream)
        idx = torch.zeros(k, dtype=torch.int32, device="cuda")
    for beside in (False, True) * 4:
        torch.cuda.synchronize()
        for _ in range(20 if beside else 0):
            b.copy_(a)
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record(side)
        for _ in range(10):
            ctx.artopk_select_topk(x, k, idx)
        t1.record(side)
        ctx.status()
        best[beside] = min(best.get(beside, 1e9), t0.elapsed_time(t1))
        assert ctx.select_info()["one_launch"] == 1
        want = idx.clone() if want is None else want
        assert torch.equal(idx, want)
    assert np.array_equal(want.cpu().numpy(), orc.topk_indices(x.cpu().numpy(), k))
    assert best[True] < 3.0 * best[False], best


# waits that are given no look at all: every kernel ends, the status says what happened, and nothing of it is left
@pytest.mark.parametrize("n,w,mode,short", [(300_002, 3, orc.MODE_STAR, 1), (65_537, 40, orc.MODE_STAR, 1),
                                            (65_537, 8, orc.MODE_VAR, 1), (600_001, 2, orc.MODE_VAR, 0)])
def test_waits_that_expire(held, n, w, mode, short):
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n)
    k = n // 50
    runner = GpuRunner(w, n, k)
    if not short:
        runner.ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, 0)
    g = [_values(rng, n, "normal", r) for r in range(w)]
    res = [_values(rng, n, "normal", r) for r in range(w)]
    want = orc.step(g, res, k, mode, step_no=1)
    runner.load_g(g)
    for late in (0, LATE, 0):
        runner.load_res(res)
        runner.torch.cuda.synchronize()
        held(late, -1)
        with pytest.raises(lib.ArTopkError) as e:
            runner.step(k, mode, 1)
        assert e.value.code == -4 and "expired" in str(e.value)
        for again in (0, LATE):
            held(again, LOOKS)
            runner.load_res(res)
            assert_step_matches(runner.step(k, mode, 1), want, mode)
            assert runner.ctx.select_info()["short"] == short
