"""What a program does with this library, as cases that can be timed and compared.

One case is one pass of a training loop's compressor step, or of one of the calls
that a program uses instead of the whole step, through the public Python entry
points.  listed() names the cases, draw() gives more of the same ranges.  Inputs
are made on the GPU from a seed: gradients g_w and the error-feedback residual
that earlier steps left (three times the gradients' scale; a pass adds the same
gradients again, so that repeated passes drift towards the state in which the
elements below the threshold have gathered several steps' gradients).
"""

import math

import torch

import paper_2312_02493_amd as artopk

MODES = {"star": artopk.ARTOPK_STAR, "var": artopk.ARTOPK_VAR}
G_TYPES = {"bf16": (artopk.ARTOPK_G_BF16, torch.bfloat16), "f16": (artopk.ARTOPK_G_F16, torch.float16)}
CHUNK = 1 << 26  # elements made at a time, so that large inputs need little memory beside their own


def listed():
    def step(name, n, w, rho, mode, values, g="f32", layers=0, bucket=0):
        return {"name": name, "call": "step", "n": n, "w": w, "rho": rho, "mode": mode, "values": values, "g": g,
                "layers": layers, "bucket": bucket}

    return [
        # One layer of a small network compressed by itself: latency and launches are all there is.
        step("step-64k-star", 65537, 2, 0.01, "star", "normal"),
        # A small network, four workers; everything stays in the caches.
        step("step-1m-star", 1048576, 4, 0.01, "star", "normal"),
        # ResNet18-sized flat gradient, eight workers of different variances, the variance rule.
        step("step-11m-var", 11689512, 8, 0.01, "var", "normal"),
        # ResNet50-sized, compressed layer by layer: 54 tensors from a few hundred to millions of elements.
        step("step-25m-layers-var", 25557032, 8, 0.01, "var", "laplace", layers=54),
        # ResNet50-sized flat gradient held in bfloat16 (mixed-precision training).
        step("step-25m-bf16-star", 25557032, 8, 0.01, "star", "normal", g="bf16"),
        # VGG16-sized heavy-tailed gradient at both ends of the adaptive keep fraction.
        step("step-138m-star-sparse", 138357544, 4, 0.001, "star", "student"),
        step("step-138m-star-dense", 138357544, 4, 0.1, "star", "student"),
        # The same fused into 64 MB buckets, as data-parallel trainers fuse tensors; the last bucket is ragged.
        step("step-138m-buckets-star", 138357544, 4, 0.01, "star", "student", bucket=1 << 24),
        # A billion parameters, eight workers: the largest model one GPU simulates; a tenth of the values tie.
        step("step-1b-var", 1000000000, 8, 0.001, "var", "ties"),
        # Only the selection, for a program that keeps its error-fed vector itself.
        {"name": "select-138m", "call": "select", "n": 138357544, "w": 1, "rho": 0.01, "values": "student"},
        # Every worker's own Top-k with values: what the all-gather exchange sends.
        {"name": "topk-workers-25m", "call": "workers", "n": 25557032, "w": 8, "rho": 0.01, "values": "normal"},
        # A rank that has received the leader's indices: gather, (reduce,) residual rewrite, dense update, gain.
        {"name": "exchange-138m", "call": "exchange", "n": 138357544, "w": 2, "rho": 0.01, "values": "student"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    call = rng.choice(["step", "step", "step", "step", "select", "workers", "exchange"])
    c = {"call": call, "rho": round(math.exp(rng.uniform(math.log(0.001), math.log(0.1))), 5),
         "values": rng.choice(["normal", "laplace", "student", "ties"])}
    if call == "step":
        form = rng.choice(["flat", "flat", "16bit", "layers", "bucket"])
        c["n"] = _log_int(rng, 65536, 400000000 if form in ("layers", "bucket") else 1000000000)
        c["w"] = rng.choice([2, 3, 4, 5, 8] if c["n"] > 200000000 else [2, 3, 4, 6, 8, 12, 16])
        c["mode"] = rng.choice(["star", "var"])
        c["g"] = rng.choice(["bf16", "f16"]) if form == "16bit" else "f32"
        c["layers"] = rng.randint(8, 160) if form == "layers" else 0
        c["bucket"] = rng.choice([1 << 22, 1 << 24]) if form == "bucket" else 0
    else:
        c["n"] = _log_int(rng, 65536, 1000000000 if call == "select" else 400000000)
        c["w"] = 1 if call == "select" else rng.randint(1, 8) if call == "exchange" else rng.randint(2, 8)
    return c


# ---- sizes -------------------------------------------------------------------------------------
def _segments(case):
    """(first elements of the segments and the end, entries kept of each), or (None, None) for a flat vector."""
    n, rho = case["n"], case["rho"]
    if case.get("bucket"):
        off = list(range(0, n, case["bucket"])) + [n]
    elif case.get("layers"):  # sizes log-uniform over a factor of about 40,000, summing to n
        s = case["layers"]
        r = [math.exp(10.6 * ((i * 0.6180339887 + 0.31) % 1.0)) for i in range(s)]
        total, off = sum(r), [0]
        for i in range(s - 1):
            off.append(max(off[-1] + 64, min(n - 64 * (s - 1 - i), off[-1] + int(n * r[i] / total))))
        off.append(n)
    else:
        return None, None
    return off, [math.ceil(rho * (b - a)) for a, b in zip(off, off[1:])]


def _k(case):
    ks = _segments(case)[1]
    return sum(ks) if ks else math.ceil(case["rho"] * case["n"])


# ---- inputs ------------------------------------------------------------------------------------
def _fill(out, values, scale, gen):
    for a in range(0, out.numel(), CHUNK):
        o = out[a:a + CHUNK]
        x = torch.randn(o.numel(), generator=gen, device="cuda")
        if values == "student":  # three degrees of freedom
            q = torch.zeros_like(x)
            for _ in range(3):
                q += torch.randn(o.numel(), generator=gen, device="cuda").square_()
            x /= q.mul_(1.0 / 3.0).sqrt_()
        elif values == "laplace":
            q = torch.empty_like(x).exponential_(generator=gen)
            x = torch.copysign(q, x)
        x *= scale
        if values == "ties":  # a tenth of the values on a coarse grid
            q = torch.rand(o.numel(), generator=gen, device="cuda") < 0.1
            x = torch.where(q, torch.round(x * 1024.0) / 1024.0, x)
        o.copy_(x)
    return out


def _inputs(case, seed):
    """(gradients or None, error-fed vectors or residuals): W vectors each."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, w = case["n"], case["w"]
    order = torch.randperm(w, generator=torch.Generator().manual_seed(seed)).tolist()
    off, _ = _segments(case)
    layer = None
    if off is not None and case.get("layers"):
        layer = [10.0 ** (1.5 - 3.0 * ((i * 0.7548776662 + 0.5) % 1.0)) for i in range(len(off) - 1)]
    g, r = [], []
    for i in range(w):
        scale = 1e-3 * (1.0 + 0.02 * order[i])  # the workers' variances differ; who leads depends on the seed
        pair = [(r, torch.float32, 3.0 * scale)]
        if case["call"] == "step":
            pair.append((g, G_TYPES[case["g"]][1] if case["g"] in G_TYPES else torch.float32, scale))
        for into, dtype, s in pair:
            x = _fill(torch.empty(n, dtype=dtype, device="cuda"), case["values"], s, gen)
            if layer is not None:
                for a, b, m in zip(off, off[1:], layer):
                    x[a:b] *= m
            into.append(x)
    return g, r


def _topk(x, k, base=0):
    """Indices of the k largest magnitudes, the lowest index first among equal ones, ascending; plain torch."""
    key = x.view(torch.int32) & 0x7FFFFFFF
    lo, hi = 0, 0x80000000  # the largest t with at least k keys >= t
    while hi - lo > 1:
        mid = (lo + hi) // 2
        if int((key >= mid).sum()) >= k:
            lo = mid
        else:
            hi = mid
    above = torch.nonzero(key > lo).view(-1)
    at = torch.nonzero(key == lo).view(-1)[:k - above.numel()]
    return (torch.cat([above, at]).sort().values + base).to(torch.int32)


def prepare(case, seed):
    n, w, k = case["n"], case["w"], _k(case)
    off, ks = _segments(case)
    g, r = _inputs(case, seed)
    s = {"call": case["call"], "k": k, "off": off, "ks": ks, "g": g, "r": r, "step": 0,
         "ctx": artopk.Context(w, n, k, len(ks) if ks else 1)}

    def new(dtype, *shape):
        return torch.zeros(*shape, dtype=dtype, device="cuda")

    if case["call"] == "step":
        s["mode"], s["g_type"] = MODES[case["mode"]], G_TYPES.get(case["g"], (None,))[0]
        s["idx"], s["sum"], s["update"] = new(torch.int32, k), new(torch.float32, k), new(torch.float32, n)
        s["leader"], s["var"] = new(torch.int32, 1), new(torch.float64, w)
    elif case["call"] == "select":
        s["idx"] = new(torch.int32, k)
    elif case["call"] == "workers":
        s["idx"], s["vals"] = new(torch.int32, w, k), new(torch.float32, w, k)
        s["sq"], s["first"] = new(torch.float64, w), new(torch.int32, 1)
    else:
        s["idx"] = _topk(r[seed % w], k)  # comes over the network
        s["vals"], s["sum"], s["update"] = new(torch.float32, w, k), new(torch.float32, k), new(torch.float32, n)
        s["gain"] = new(torch.float64, w)
    return s


# ---- one pass ----------------------------------------------------------------------------------
def run(s):
    ctx, k = s["ctx"], s["k"]
    if s["call"] == "step":
        s["step"] += 1
        more = {"leader_out": s["leader"], "var_out": s["var"]}
        if s["off"] is not None:
            more.update(seg_off=s["off"], seg_k=s["ks"])
        if s["g_type"] is None:
            ctx.artopk_step(s["g"], s["r"], k, s["mode"], s["step"], s["idx"], s["sum"], s["update"], **more)
        else:
            ctx.artopk_step_g16(s["g"], s["g_type"], s["r"], k, s["mode"], s["step"], s["idx"], s["sum"], s["update"],
                                **more)
        return {"idx": s["idx"], "sum": s["sum"], "update": s["update"], "leader": s["leader"], "var": s["var"],
                "residual": s["r"]}
    if s["call"] == "select":
        ctx.artopk_select_topk(s["r"][0], k, s["idx"])
        return {"idx": s["idx"]}
    if s["call"] == "workers":
        ctx.artopk_topk_workers(s["r"], k, s["idx"], s["vals"], s["sq"], s["first"])
        return {"idx": s["idx"], "vals": s["vals"], "sq": s["sq"], "first": s["first"]}
    ctx.artopk_gather_sum(s["r"], s["idx"], k, s["vals"], s["sum"])
    ctx.artopk_scatter_residual(s["r"], s["idx"], k, s["sum"], s["update"])
    ctx.artopk_compression_gain(s["r"], s["vals"], k, s["gain"])
    return {"vals": s["vals"], "sum": s["sum"], "update": s["update"], "gain": s["gain"], "residual": s["r"]}


def work(case):
    n, w, k = case["n"], case["w"], _k(case)
    if case["call"] == "step":  # gradients and residuals read; residuals, update, indices and sums written
        per = 8 + (4 if case["g"] == "f32" else 2)
        return {"bytes": per * w * n + 4 * n + 8 * k, "flops": w * n}
    if case["call"] == "select":
        return {"bytes": 4 * n + 4 * k, "flops": 0}
    if case["call"] == "workers":
        return {"bytes": 4 * w * n + 8 * w * k, "flops": 2 * w * k}
    # indices, the kept values and zeros in their place, vals and sums, the update, one read of the residuals
    return {"bytes": 4 * k + 12 * w * k + 4 * k + 4 * n + 4 * w * n, "flops": 2 * w * n}


def tolerance(case):
    """Everything in 32 bits is defined bit for bit (element-wise float32 addition, selection by the magnitude's
    bits, sums in the workers' order); the variances, squared norms and gains are 64-bit sums, whose order is
    free: up to 3e-13 of difference to another order was seen on vectors with outliers, plain ones show 1e-15."""
    if case["call"] == "select" or (case["call"] == "step" and case["mode"] == "star"):
        return "exact"
    return {"rel": 1e-12, "max": 1e-12, "differ": 0.0}


def _mean64(x, of):
    total = 0.0
    for a in range(0, x.numel(), CHUNK):
        total += float(of(x[a:a + CHUNK].double()).sum())
    return total


def exact(case, seed):
    n, w, k = case["n"], case["w"], _k(case)
    if n * w > 2000000000:
        return None
    g, r = _inputs(case, seed)
    f64 = {"dtype": torch.float64, "device": "cuda"}
    if case["call"] == "select":
        return {"idx": _topk(r[0], k)}
    if case["call"] == "workers":
        idx = torch.stack([_topk(x, k) for x in r])
        vals = torch.stack([x[i.long()] for x, i in zip(r, idx)])
        sq = vals.double().square().sum(1)
        return {"idx": idx, "vals": vals, "sq": sq, "first": sq.argmax().view(1).to(torch.int32)}
    var = torch.zeros(w, **f64)
    if case["call"] == "exchange":
        idx = _topk(r[seed % w], k)
    else:  # the error-fed vector is float32 by definition: one rounding of each sum of two
        for x, y in zip(r, g):
            x += y.float()
        leader = 1 % w
        if case["mode"] == "var":
            for i, x in enumerate(r):
                mean = _mean64(x, lambda v: v) / n
                var[i] = _mean64(x, lambda v: (v - mean).square_()) / n
            leader = int(var.argmax())
        off, ks = _segments(case)
        if off is None:
            idx = _topk(r[leader], k)
        else:
            idx = torch.cat([_topk(r[leader][a:b], q, a) for a, b, q in zip(off, off[1:], ks)])
    at = idx.long()
    vals = torch.stack([x[at] for x in r])
    total = vals.double().sum(0)
    update = torch.zeros(n, **f64)
    update[at] = total
    for x in r:
        x[at] = 0.0
    if case["call"] == "exchange":
        kept = vals.double().square().sum(1)
        left = torch.tensor([_mean64(x, lambda v: v.square_()) for x in r], **f64)
        return {"vals": vals, "sum": total, "update": update, "gain": kept / (kept + left), "residual": r}
    return {"idx": idx, "sum": total, "update": update, "leader": torch.tensor([leader], dtype=torch.int32),
            "var": var, "residual": r}
