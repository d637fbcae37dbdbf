"""Steps on short vectors, which run in one launch: against the oracle and against the general launch sequence."""

import numpy as np
import pytest

from oracle import artopk_oracle as orc
from tests import gpu_util
from tests.gpu_util import GpuRunner, assert_step_matches

pytestmark = pytest.mark.gpu


def _vector(rng, n, kind, r):
    x = (rng.standard_normal(n) * 0.01 * (1.0 + 0.3 * r)).astype(np.float32)
    if kind == "ties":
        x = np.round(x * 128).astype(np.float32) / 128
    elif kind == "equal":  # every magnitude the same
        x = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32) * np.float32(0.25 * (1 + r))
    elif kind == "zeros":
        x[:] = 0.0
        x[r::max(1, n // 7)] = 1.0 + r
    elif kind == "one_bin":  # one top digit, many second and third digits
        x = (1.0 + rng.random(n) * 0.01).astype(np.float32)
        x[0] += 0.001 * r
    elif kind == "special":
        x[rng.integers(0, n, 5)] = np.inf
        x[rng.integers(0, n, n // 5 + 1)] = np.float32(-1e-45)
    return x


# one element, less than a group, the edges of a wave's share and of a chunk, the longest vector of the route
# (of the variance rules with fewer than eight workers: 3 << 18)
@pytest.mark.parametrize("n", [1, 3, 1023, 1024, 1025, 8191, 8193, 65537, 300_002, 3 << 18, (3 << 18) + 1, 1 << 20])
@pytest.mark.parametrize("kind", ["normal", "ties", "equal", "zeros", "one_bin", "special"])
def test_short_steps_match_the_oracle(n, kind):
    rng = np.random.default_rng(n)
    w = 1 + n % 6
    kmax = min(n, 16384)
    runner = GpuRunner(w, n, kmax)
    for mode in (orc.MODE_STAR, orc.MODE_FIXED, orc.MODE_VAR, orc.MODE_VAR_G):
        if kind == "special" and mode in (orc.MODE_VAR, orc.MODE_VAR_G):
            continue  # variances of infinities
        if kind in ("equal", "zeros", "ties") and mode == orc.MODE_VAR_G and w > 1 and n < 64:
            continue  # equal variances up to rounding
        for step_no, k in enumerate(sorted({1, (n + 99) // 100, min(kmax, (n + 9) // 10), kmax}), 1):
            g = [_vector(rng, n, kind, r) for r in range(w)]
            res = [_vector(rng, n, "normal", r) if step_no % 2 and kind == "normal" else np.zeros(n, np.float32)
                   for r in range(w)]
            want = orc.step(g, res, k, mode, step_no=step_no, fixed_leader=w - 1)
            if mode in (orc.MODE_VAR, orc.MODE_VAR_G) and w > 1 and gpu_util.top_two_gap(want.variances) <= 1e-4:
                continue
            runner.load_g(g)
            runner.load_res(res)
            got = runner.step(k, mode, step_no, fixed_leader=w - 1, want_vals=step_no % 2 == 1)
            assert_step_matches(got, want, mode)
            on_device = mode in (orc.MODE_VAR, orc.MODE_VAR_G) and w < 8
            assert gpu_util.FORCED or runner.ctx.select_info()["short"] == (n <= (3 << 18 if on_device else 1 << 20))


# chunks of 4096 elements (up to 2^20) and 8192 (up to 2^21): one, whole ones, an element more or less, the last one
# short; one worker, more than are loaded at a time, and the most
@pytest.mark.parametrize("n", [2047, 4095, 4096, 4097, 65536, (1 << 18) - 3, 1 << 18, (1 << 18) + 1, (1 << 20) - 1, (1 << 20) + 1,
                               (1 << 20) + 8191, (1 << 20) + 8192, (1 << 20) + 8193])
@pytest.mark.parametrize("w", [1, 6, 64])
def test_short_steps_at_the_edges_of_chunks(n, w):
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n + w)
    k = max(1, min(n // 10, 16384))
    runner = GpuRunner(w, n, k)
    runner.ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, 1 << 21)
    res = [np.zeros(n, np.float32) for _ in range(w)]
    runner.load_res(res)
    for step_no, mode in enumerate((orc.MODE_STAR, orc.MODE_VAR, orc.MODE_STAR), 1):
        g = [_vector(rng, n, "ties" if step_no == 2 else "normal", r) for r in range(w)]
        want = orc.step(g, res, k, mode, step_no=step_no)
        runner.load_g(g)
        assert_step_matches(runner.step(k, mode, step_no, want_vals=step_no == 1), want, mode)
        assert gpu_util.FORCED or runner.ctx.select_info()["short"] == 1
        res = want.residual


# where the general launches are ahead of the one (many workers' values under a variance rule, until the option is set),
# and either side of the line from which on a known leader's fellow workers are shared out among further blocks
@pytest.mark.parametrize("n,w,mode,setting,short", [(524_288, 42, orc.MODE_VAR, None, 0), (524_288, 41, orc.MODE_VAR, None, 1),
                                                    (524_288, 42, orc.MODE_VAR, 1 << 20, 1), (524_287, 48, orc.MODE_VAR, None, 1),
                                                    (786_432, 28, orc.MODE_VAR_G, None, 0), (786_433, 28, orc.MODE_VAR, None, 1),
                                                    (163_840, 41, orc.MODE_STAR, None, 1), (163_841, 41, orc.MODE_STAR, None, 1),
                                                    (163_840, 40, orc.MODE_STAR, None, 1)])
def test_short_steps_of_many_workers(n, w, mode, setting, short):
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n + w)
    k = n // 100
    runner = GpuRunner(w, n, k)
    if setting is not None:
        runner.ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, setting)
    g = [_vector(rng, n, "normal", r) for r in range(w)]
    res = [np.zeros(n, np.float32) for _ in range(w)]
    want = orc.step(g, res, k, mode, step_no=1)
    runner.load_g(g)
    runner.load_res(res)
    assert_step_matches(runner.step(k, mode, 1, want_vals=False), want, mode)
    assert gpu_util.FORCED or runner.ctx.select_info()["short"] == short


# the same step on both launch sequences, in turn on one context (the short one must leave its scratch as it found it)
@pytest.mark.parametrize("n,w,k", [(70_001, 9, 700), (1 << 20, 3, 16384), ((1 << 20) - 3, 17, 1)])
@pytest.mark.parametrize("g", ["f32", "bf16", "f16"])
def test_short_steps_and_general_steps_alternate(n, w, k, g):
    import torch
    import paper_2312_02493_amd as lib

    gen = torch.Generator(device="cuda").manual_seed(n)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[g]
    gs = [(torch.randn(n, generator=gen, device="cuda") * (1.0 + 0.1 * r)).to(dt) for r in range(w)]
    r0 = [torch.randn(n, generator=gen, device="cuda") for _ in range(w)]
    ctx = lib.Context(w, n, k)

    def run(short, mode, step):
        ctx.set_step_counter(step)
        ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, (1 << 20) if short else 0)
        res = [r.clone() for r in r0]
        idx = torch.zeros(k, dtype=torch.int32, device="cuda")
        sm, up = torch.zeros(k, device="cuda"), torch.zeros(n, device="cuda")
        vals, lead = torch.zeros(w * k, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
        var = torch.zeros(w, dtype=torch.float64, device="cuda")
        more = {"vals_out": vals, "leader_out": lead, "var_out": var}
        if g == "f32":
            ctx.artopk_step(gs, res, k, mode, step, idx, sm, up, **more)
        else:
            ctx.artopk_step_g16(gs, lib.ARTOPK_G_BF16 if g == "bf16" else lib.ARTOPK_G_F16, res, k, mode, step, idx, sm,
                                up, **more)
        ctx.status()
        if mode not in (lib.ARTOPK_VAR, lib.ARTOPK_VAR_G):
            var.zero_()
        return [idx, sm.view(torch.int32), up.view(torch.int32), vals.view(torch.int32), lead] + \
            [r.view(torch.int32) for r in res], var

    for step, mode in enumerate((lib.ARTOPK_STAR, lib.ARTOPK_VAR, lib.ARTOPK_STAR_COUNTER, lib.ARTOPK_VAR_G), 1):
        a, va = run(True, mode, step)
        b, vb = run(False, mode, step)
        for x, y in zip(a, b):
            assert torch.equal(x, y)
        torch.testing.assert_close(va, vb, rtol=1e-12, atol=0.0)  # float64 sums of n terms in another order


def _few(n):
    return 10240 + 240 * ((n + 8191) // 8192)


def _narrow(rng, n, kind, r):
    """Vectors whose threshold's top digit many values share (select_info tells whether more than `few`)."""
    few = _few(n)
    x = (rng.standard_normal(n) * 0.01).astype(np.float32)
    if kind == "band":  # all of them, most second and last digits
        return (1.0 + rng.random(n) * 0.06).astype(np.float32)
    if kind == "two":  # two values: the last digit is the same for half the vector
        return np.where(rng.random(n) < 0.5, np.float32(1.0), np.float32(-1.03)).astype(np.float32)
    if kind == "near":  # neighbouring numbers: one second digit, every last digit
        return (np.uint32(0x3f800000) + rng.integers(0, 128, n).astype(np.uint32)).view(np.float32)
    if kind == "equal":
        return np.full(n, np.float32(0.75))
    m = min(n, few + {"few": 0, "few1": 1}[kind])  # exactly as many as select_info takes for few, and one more
    x[rng.permutation(n)[:m]] = (1.0 + rng.random(m) * 0.01).astype(np.float32)
    return x


# a step on narrow values before and after an ordinary one on the same context: the blocks have to leave
# the scratch as they found it; 2^21 is the option's largest value
@pytest.mark.parametrize("n", [16385, 65537, 300_002, (1 << 20) - 3, (1 << 20) + 1, 1 << 21])
@pytest.mark.parametrize("kind", ["band", "two", "near", "equal", "few", "few1"])
def test_short_steps_on_narrow_values(n, kind):
    import paper_2312_02493_amd as lib

    rng = np.random.default_rng(n)
    w, kmax = 8 if n > 1 << 20 else 2, 16384
    runner = GpuRunner(w, n, kmax)
    runner.ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, 1 << 21)
    step_no = 0
    for k, mode in ((kmax, orc.MODE_STAR), (min(kmax, n // 100), orc.MODE_VAR), (1, orc.MODE_STAR)):
        for now in (kind, "ordinary", kind):
            step_no += 1
            g = [np.zeros(n, np.float32) for _ in range(w)]
            if now == "ordinary":
                res = [_vector(rng, n, "normal", r) for r in range(w)]
            else:
                res = [_narrow(rng, n, kind, r) * np.float32(2.0 ** (r % 2)) for r in range(w)]
            want = orc.step(g, res, k, mode, step_no=step_no)
            if mode == orc.MODE_VAR and gpu_util.top_two_gap(want.variances) <= 1e-4:
                continue
            runner.load_g(g)
            runner.load_res(res)
            assert_step_matches(runner.step(k, mode, step_no, want_vals=False), want, mode)
            info = runner.ctx.select_info()
            assert gpu_util.FORCED or info["short"] == 1
            if now == "ordinary" or kind == "few":
                assert gpu_util.FORCED or info["many"] == 0, (k, now)
            elif kind != "few1" or k <= _few(n):  # (a threshold among the narrow values)
                assert gpu_util.FORCED or info["many"] == 1, (k, now)


# narrow values may not make a short step slower than the general launch sequence is on them (one block alone took
# four to thirteen times as long; half as long again leaves room for the clock)
@pytest.mark.parametrize("kind", ["band", "two", "near"])
def test_short_steps_on_narrow_values_take_no_longer(kind):
    import torch
    import paper_2312_02493_amd as lib

    n, w, k = 1 << 20, 2, 10486
    rng = np.random.default_rng(5)
    src = [torch.from_numpy(_narrow(rng, n, kind, r)).cuda() for r in range(w)]
    g = [torch.zeros(n, device="cuda") for _ in range(w)]
    idx = torch.zeros(k, dtype=torch.int32, device="cuda")
    sm, up = torch.zeros(k, device="cuda"), torch.zeros(n, device="cuda")
    best = {}
    for limit in (0, 1 << 20) * 3:
        ctx = lib.Context(w, n, k)
        ctx.set_option(lib.ARTOPK_OPT_SHORT_MAX_N, limit)
        res = [x.clone() for x in src]
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for step in range(1, 18):  # (each pass keeps one value in a hundred: the vectors stay narrow)
            if step == 3:
                t0.record()
            ctx.artopk_step(g, res, k, lib.ARTOPK_STAR, step, idx, sm, up)
        t1.record()
        ctx.status()
        best[limit] = min(best.get(limit, 1e9), t0.elapsed_time(t1))
    assert best[1 << 20] < 1.5 * best[0], best


# two contexts on streams of their own, beside long kernels of a third: blocks that look out for help or for others may
# find neither, and every result is the same
def test_narrow_steps_on_several_streams_beside_other_work():
    import torch
    import paper_2312_02493_amd as lib

    n, w, k, steps = 1 << 20, 2, 10486, 6
    rng = np.random.default_rng(11)
    src = [torch.from_numpy(_narrow(rng, n, "band", r)).cuda() for r in range(w)]
    g = [torch.full((n,), 2.0 ** -12, device="cuda") for _ in range(w)]
    busy = [torch.randn(1 << 27, device="cuda")]

    def start(stream):
        torch.cuda.synchronize()
        s = torch.cuda.Stream() if stream else torch.cuda.current_stream()
        with torch.cuda.stream(s):
            return {"s": s, "ctx": lib.Context(w, n, k, stream=s.cuda_stream), "res": [x.clone() for x in src],
                    "idx": torch.zeros(k, dtype=torch.int32, device="cuda"), "sum": torch.zeros(k, device="cuda"),
                    "up": torch.zeros(n, device="cuda"), "out": []}

    def go(c, step):
        with torch.cuda.stream(c["s"]):
            c["ctx"].artopk_step(g, c["res"], k, lib.ARTOPK_STAR, step, c["idx"], c["sum"], c["up"])
            c["out"].append((c["idx"].clone(), c["sum"].clone()))

    one, two, alone = start(True), start(True), start(False)
    other = lib.Context(1, 1 << 27, 1, stream=torch.cuda.current_stream().cuda_stream)
    var = torch.zeros(1, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    for step in range(1, steps + 1):
        for _ in range(3):
            other.artopk_variance(busy, var)
        go(one, step)
        go(two, step)
    torch.cuda.synchronize()
    for step in range(1, steps + 1):
        go(alone, step)
    torch.cuda.synchronize()
    for c in (one, two, alone):
        assert gpu_util.FORCED or c["ctx"].select_info()["many"] == 1
        c["ctx"].status()
    for c in (one, two):
        for (i, v), (iw, vw) in zip(c["out"], alone["out"]):
            assert torch.equal(i, iw) and torch.equal(v.view(torch.int32), vw.view(torch.int32))
        for r, rw in zip(c["res"], alone["res"]):
            assert torch.equal(r.view(torch.int32), rw.view(torch.int32))


# As many values share the threshold's top digit as a chunk's share of the memory for them just takes, or one more; one,
# sixteen and sixty-four chunks, and a chunk too many.
@pytest.mark.parametrize("n,room", [(4001, 2048), (65_536, 2047), (1 << 18, 511), ((1 << 18) + 1, 500)])
@pytest.mark.parametrize("kind", ["spread", "one_chunk", "equal", "last_digit"])
def test_short_steps_with_few_candidates(n, room, kind):
    rng = np.random.default_rng(n + len(kind))
    w, top = 3, 7
    runner = GpuRunner(w, n, top + room + 1)
    for step_no, m in enumerate([room - 1, room, room + 1, 65, 64, 1]):
        for mode in (orc.MODE_STAR, orc.MODE_VAR):
            def vector(r):
                x = (rng.standard_normal(n) * 0.01).astype(np.float32)
                at = rng.permutation(n if kind != "one_chunk" else min(n, 4096))[:m + top]
                v = 1.0 + rng.random(m + top) * 0.06
                if kind == "equal":
                    v[:] = 1.03
                elif kind == "last_digit":
                    v = 1.03125 + rng.integers(0, 128, m + top) * 2.0 ** -23
                v[m:] = 2.0 + rng.random(top)
                x[at] = (v * rng.choice([-1.0, 1.0], m + top)).astype(np.float32)
                if r == 1:
                    x[at[m:]] *= 3.0  # the variance rule's leader
                return x

            g, res = [vector(r) for r in range(w)], [np.zeros(n, np.float32) for _ in range(w)]
            k = top + max(1, (m * (1 + step_no % 3)) // 3)
            want = orc.step(g, res, k, mode, step_no=step_no)
            assert mode == orc.MODE_STAR or gpu_util.top_two_gap(want.variances) > 1e-4
            runner.load_g(g)
            runner.load_res(res)
            assert_step_matches(runner.step(k, mode, step_no), want, mode)
            assert gpu_util.FORCED or runner.ctx.select_info()["short"] == 1
