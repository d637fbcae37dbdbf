"""Launches whose blocks wait for each other, when two blocks in three start 100 us late: the others take on their work,
and every result is the oracle's.  And waits that expire: an error, and the next call on the context is right again."""

import ctypes as C

import numpy as np
import pytest

from oracle import artopk_oracle as orc
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
