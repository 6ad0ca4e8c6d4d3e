"""The calls this library is timed on: whole scale schedules of one layer through hack_step, a compression through
the single entry points, and the offline head variance, over the range of shapes that the library's own workload
families (paper_2504_09261_amd/workload.py) and their neighbours span.

A pass of a schedule is what a generation does per layer and image: an empty managed cache, then one step per scale
(append, score, select, compact, attend).  "graph" replays the same steps from a HIP graph, as bench.py does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2504_09261_amd import workload as wl
from paper_2504_09261_amd.binding import Cache, Hack

GATE_STEP = 4        # compression allowed from this 1-based step
SINKS = 12           # sink keys per contextual head
SIDES_10 = ",".join(map(str, wl.SIDES_10))    # 256^2: 680 tokens
SIDES_13 = ",".join(map(str, wl.SIDES_13))    # 1024^2: 10521 tokens


def _schedule(name, dtype, heads, head_dim, batch, sides, keep, ctx_frac, ratio, jitter=0.0, merge=False, graph=False):
    """keep: retained fraction of the cache averaged over the heads (1: no compression); ctx_frac: share of contextual
    heads; ratio: structural : contextual budget; jitter: spread of the budgets inside a class; merge: the last step
    is hack_step_final."""
    return dict(name=name, kind="schedule", dtype=dtype, heads=heads, head_dim=head_dim, batch=batch, sides=sides, keep=keep,
                ctx_frac=ctx_frac, ratio=ratio, jitter=jitter, merge=merge, graph=graph)


def listed():
    return [
        # the first scales of a 1024^2 image, one prompt with guidance: a few queries per unit, launches and latency only
        _schedule("first-scales", "bf16", 16, 128, 2, "1,2,4,6", 1.0, 0.375, 2.0),
        # one class-conditional 256^2 image with guidance
        _schedule("256-one-image", "bf16", 30, 64, 2, SIDES_10, 0.3, 0.5, 3.0, graph=True),
        # the same model over a batch of 16 images with guidance, steps issued one by one
        _schedule("256-batch", "bf16", 30, 64, 32, SIDES_10, 0.3, 0.5, 3.0),
        # the benchmark's own line: 2B-class text-to-image model at 1024^2, one prompt with guidance
        _schedule("1024-2b", "bf16", 16, 128, 2, SIDES_13, 0.3, 0.375, 2.0, graph=True),
        # the same image without compression (the whole cache kept), the largest caches
        _schedule("1024-2b-full-cache", "bf16", 16, 128, 2, SIDES_13, 1.0, 0.375, 2.0),
        # strong compression whose last step merges what contextual heads discard
        _schedule("1024-2b-keep10-merge", "bf16", 16, 128, 2, SIDES_13, 0.1, 0.375, 2.0, merge=True),
        # 8B-class model at 1024^2
        _schedule("1024-8b", "bf16", 32, 128, 2, SIDES_13, 0.3, 0.5, 3.0),
        # four prompts with guidance, budgets of their own per head: ragged caches, the largest case
        _schedule("1024-ragged-batch", "bf16", 16, 128, 8, SIDES_13, 0.5, 0.25, 2.0, jitter=0.2),
        # a 256^2 image in float32
        _schedule("256-f32", "f32", 16, 64, 1, SIDES_10, 0.3, 0.5, 3.0),
        # odd sizes throughout: sides that fill no tile, narrow heads, an odd number of units
        _schedule("odd-sides", "bf16", 9, 64, 3, "1,2,3,5,7,11,17,26,37", 0.25, 0.4, 2.0, jitter=0.1),
        # one compression through the single entry points on a device that is shared with other work (two-pass scores)
        dict(name="compress-calls", kind="compress", dtype="bf16", heads=20, head_dim=128, batch=2, rows=2817, new=1369, keep=0.35,
             ctx_frac=0.5, n_obs=32, score="two-pass"),
        # offline classification of the heads of one layer: all queries of the last 1024^2 scale over the full cache
        dict(name="head-variance", kind="variance", heads=16, head_dim=128, batch=2, rows=10521, queries=4096),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        case = _draw_any(rng)
        if _cost(case) <= most:
            return case


def _draw_any(rng):
    kind = rng.choice(["schedule"] * 7 + ["f32", "compress", "compress", "variance"])
    head_dim = rng.choice([64, 128, 128])
    heads, batch = rng.randint(4, 32), _log_int(rng, 1, 32)
    if kind in ("schedule", "f32"):
        last, n = (_log_int(rng, 6, 64), rng.randint(4, 13)) if kind == "schedule" else (_log_int(rng, 6, 20), rng.randint(4, 10))
        sides = sorted({max(1, int(round(last ** (i / (n - 1.0))))) for i in range(n)})
        keep = rng.choice([1.0, round(rng.uniform(0.08, 0.7), 3), round(rng.uniform(0.08, 0.7), 3), round(rng.uniform(0.08, 0.7), 3)])
        f32 = kind == "f32"
        c = _schedule("", "f32" if f32 else "bf16", heads, head_dim, min(batch, 2) if f32 else batch, ",".join(map(str, sides)), keep,
                      round(rng.uniform(0.2, 0.8), 2), round(rng.uniform(1.5, 3.0), 2), rng.choice([0.0, round(rng.uniform(0.05, 0.2), 2)]),
                      not f32 and keep < 1.0 and rng.random() < 0.25, rng.random() < 0.4)
        del c["name"]
        return c
    if kind == "compress":
        score = rng.choice(["fused", "two-pass", "static"])
        if score == "static":
            batch = max(1, min(batch, 64 // heads))   # hack_score_static takes at most 64 units
        return dict(kind="compress", dtype="bf16", heads=heads, head_dim=head_dim, batch=batch, rows=_log_int(rng, 40, 8000),
                    new=_log_int(rng, 40, 4096), keep=round(rng.uniform(0.1, 0.7), 3), ctx_frac=round(rng.uniform(0.2, 0.8), 2),
                    n_obs=rng.choice([32, 32, rng.randint(4, 31)]), score=score)
    return dict(kind="variance", heads=heads, head_dim=head_dim, batch=min(batch, 4), rows=_log_int(rng, 300, 10521), queries=_log_int(rng, 100, 4096))


def _cost(case):
    """Rough seconds of a pass, to keep drawn cases within the largest listed one."""
    w = work(case)
    f32 = case.get("dtype") == "f32"
    steps = len(case["sides"].split(",")) if case["kind"] == "schedule" else 1
    units = case["heads"] * case["batch"]
    return w["bytes"] / 3e12 + w["flops"] / (2.5e11 if f32 else 6e14) + steps * (2e-5 + 2.5e-7 * units)


# ---- host-side plan of a case -------------------------------------------------------------------------------------
def _classes(case):
    """(types, budget factors): per head class and the factor of its class budget, before heads are shuffled."""
    H = case["heads"]
    n_c = int(round(case["ctx_frac"] * H))
    types = np.array([wl.CONTEXTUAL] * n_c + [wl.STRUCTURAL] * (H - n_c), np.uint8)
    j = case.get("jitter", 0.0)
    factor = np.concatenate([np.linspace(1 - j, 1 + j, m) if m > 1 else np.ones(m) for m in (n_c, H - n_c)])
    return types, factor


def _head_budgets(case, T_K, n_init):
    types, factor = _classes(case)
    a = float((types == wl.CONTEXTUAL).mean())
    r_c = case["keep"] / (a + case["ratio"] * (1 - a))
    r = np.where(types == wl.CONTEXTUAL, r_c, np.minimum(1.0, r_c * case["ratio"])) * factor
    return types, np.clip(np.ceil(r * T_K - 1e-9), min(n_init + 1, T_K), T_K).astype(np.int32)


def _steps(case):
    """(sides, n_init, types[H], cap[H], per step budgets[H]) of a schedule, heads in unshuffled order."""
    sides = [int(s) for s in case["sides"].split(",")]
    N = [s * s for s in sides]
    n_init = sum(N[:2])
    types, b = _head_budgets(case, sum(N), n_init)
    if case["keep"] >= 1.0:
        return sides, n_init, types, np.full_like(b, sum(N)), [np.full_like(b, wl.NO_COMPRESSION) for _ in N]
    # the slab of a unit holds its budget, and what it collects before the first step that may compress
    cap = np.maximum(b, sum(N[:GATE_STEP - 1]))
    return sides, n_init, types, cap, [b if k + 1 >= GATE_STEP else np.full_like(b, wl.NO_COMPRESSION) for k in range(len(N))]


def _compress_plan(case):
    """Cached rows, budgets and classes per head of a single compression: contextual caches are half as long."""
    types, _ = _classes(case)
    rows = np.where(types == wl.CONTEXTUAL, max(1, case["rows"] // 2), case["rows"]).astype(np.int32)
    t_in = rows + case["new"]
    budget = np.maximum(1, np.ceil(case["keep"] * t_in)).astype(np.int32)
    return types, rows, budget


def work(case):
    d, B = case["head_dim"], case["batch"]
    e = 4 if case.get("dtype") == "f32" else 2
    if case["kind"] == "variance":
        U, N, T = B * case["heads"], case["queries"], case["rows"]
        return {"bytes": float(U * ((N + T) * d * 2 + 8)), "flops": 2.0 * U * N * T * d}
    if case["kind"] == "compress":
        _, rows, budget = _compress_plan(case)
        t = (rows + case["new"]).astype(np.float64)
        b = budget.astype(np.float64)
        n_obs = min(case["n_obs"], case["new"])
        return {"bytes": float(B * (t * d * e + n_obs * d * e + 4 * t + 4 * b + 2 * b * d * e + b * d * e + 4 * b).sum()),
                "flops": float(B * (2.0 * n_obs * t * d).sum())}
    sides, n_init, types, cap, budgets = _steps(case)
    L = np.zeros(len(types))
    nbytes = flops = 0.0
    for k, s in enumerate(sides):
        n = s * s
        t = L + n
        out = np.minimum(budgets[k], t)
        comp = out < t
        # queries, new keys and values in, outputs out; cached rows in; the rows that change in the cache out
        nbytes += float((4 * n * d * e + 2 * L * d * e + np.where(comp, out, n) * 2 * d * e).sum())
        flops += float((4.0 * n * out * d).sum() + (2.0 * min(32, n) * t * d)[comp].sum())
        if case["merge"] and k == len(sides) - 1:
            m = comp & (types == wl.CONTEXTUAL)
            flops += float((2.0 * (t - out) * out * d)[m].sum())
        L = out
    return {"bytes": B * nbytes, "flops": B * flops}


def tolerance(case):
    """Four times what was seen: bf16 outputs of the library's other attention kernels against its own (2-norm 1.7e-3,
    largest 2.2e-2: probabilities and outputs are rounded to bf16), float32 outputs, importance and variance against
    float64 (9e-7 and 5.4e-6; 3e-7 and 7.4e-7; 5.6e-6).  Caches and kept rows are copies and integers."""
    if case["kind"] == "variance":
        return {"rel": 2.5e-5}
    if case["kind"] == "compress":
        return {"rel": 1.2e-6, "max": 3e-6}
    return {"rel": 4e-6, "max": 2.2e-5} if case["dtype"] == "f32" else {"rel": 7e-3, "max": 0.09}


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _tensors(gen, types, dirs, B, d, side, dtype):
    """q, k, v of one scale: unit normal; contextual heads share a direction u per head between all queries and a few
    sink keys, structural heads carry a positional code in queries and keys (the recipe of workload.gen_step)."""
    dev = torch.device("cuda", 0)
    n = side * side
    q, k, v = (torch.randn((B, len(types), n, d), generator=gen, device=dev) for _ in range(3))
    ctx = torch.from_numpy(np.flatnonzero(types == wl.CONTEXTUAL)).to(dev)
    st = torch.from_numpy(np.flatnonzero(types == wl.STRUCTURAL)).to(dev)
    if ctx.numel():
        u = dirs[ctx]
        q[:, ctx] += u[None, :, None, :]
        # about SINKS sink keys per head over the whole schedule: a share of every scale
        sink = torch.rand((len(ctx), n), generator=gen, device=dev) < SINKS / (2.6 * n + SINKS)
        k[:, ctx] += 3.0 * sink[None, :, :, None] * u[None, :, None, :]
    if st.numel():
        e = torch.zeros((n, d), device=dev)
        e[:, :64] = 2.0 * torch.from_numpy(wl.positional_code(side)).to(dev)
        q[:, st] += e
        k[:, st] += e
    return [x.to(torch.float32 if dtype == "f32" else torch.bfloat16).contiguous() for x in (q, k, v)]


def _shuffle(seed, H):
    return np.random.default_rng(seed).permutation(H)


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    gen = torch.Generator(dev)
    gen.manual_seed(seed)
    H, d, B = case["heads"], case["head_dim"], case["batch"]
    dirs = torch.nn.functional.normalize(torch.randn((H, d), generator=gen, device=dev), dim=-1)
    scale = float(np.float32(1.0 / math.sqrt(d)))
    perm = _shuffle(seed, H)
    if case["kind"] == "variance":
        return _prepare_variance(case, gen, scale)
    if case["kind"] == "compress":
        return _prepare_compress(case, gen, dirs, scale, perm)
    sides, n_init, types, cap, budgets = _steps(case)
    types = types[perm]
    hk = Hack(H, d, case["dtype"], B * H, sum(s * s for s in sides), sides[-1] ** 2)
    mc = hk.managed_cache(np.tile(cap[perm], B))
    for t in (mc.k, mc.v, mc.pos):
        t.zero_()
    steps = []
    for k, s in enumerate(sides):
        q, kn, vn = _tensors(gen, types, dirs, B, d, s, case["dtype"])
        steps.append((q, kn, vn, np.tile(budgets[k][perm], B).astype(np.int32), torch.zeros_like(q)))
    state = dict(kind="schedule", hk=hk, cache=mc, steps=steps, types=types, n_init=n_init, scale=scale, merge=case["merge"], graph=None)
    if case["graph"]:
        _run_schedule(state)                    # launch tables are uploaded before the capture
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            _run_schedule(state)
        state["graph"] = g
    return state


def _prepare_compress(case, gen, dirs, scale, perm):
    dev = torch.device("cuda", 0)
    H, d, B, n = case["heads"], case["head_dim"], case["batch"], case["new"]
    types, rows, budget = (x[perm] for x in _compress_plan(case))
    rows, budget = np.tile(rows, B), np.tile(budget, B)
    U = B * H
    hk = Hack(H, d, case["dtype"], U, int(rows.max()) + n, n, case["n_obs"])
    if case["score"] == "two-pass":
        hk.set_score_mode(1)
    side = math.isqrt(n - 1) + 1
    q, kn, vn = (x[:, :, :n].contiguous() for x in _tensors(gen, types, dirs, B, d, side, case["dtype"]))

    def cache(length, fill):
        off = np.concatenate([[0], np.cumsum((length + 7) // 8 * 8)]).astype(np.int64)
        k, v = (torch.randn((int(off[-1]), d), generator=gen, device=dev).to(q.dtype) if fill else torch.zeros((int(off[-1]), d), dtype=q.dtype, device=dev)
                for _ in range(2))
        pos = torch.arange(int(off[-1]), dtype=torch.int32, device=dev) if fill else torch.zeros(int(off[-1]), dtype=torch.int32, device=dev)
        return Cache(k, v, off[:-1], length, pos)
    stride = (int(rows.max()) + n + 63) // 64 * 64
    return dict(kind="compress", hk=hk, q=q, k_new=kn, v_new=vn, types=types, budget=budget, t_in=rows + n, scale=scale, n_init=5,
                n_obs=min(case["n_obs"], n), static=case["score"] == "static", src=cache(rows, True), dst=cache(np.minimum(budget, rows + n), False),
                importance=torch.zeros((U, stride), device=dev), kept=torch.full((U, stride), -1, dtype=torch.int32, device=dev))


def _prepare_variance(case, gen, scale):
    dev = torch.device("cuda", 0)
    H, d, B, N, T = case["heads"], case["head_dim"], case["batch"], case["queries"], case["rows"]
    U, stride = B * H, (T + 7) // 8 * 8
    q = torch.randn((B, H, N, d), generator=gen, device=dev)
    k = torch.randn((U, stride, d), generator=gen, device=dev)
    # every other head aligns queries with a band of keys (structural), the rest stay diffuse (contextual)
    code = torch.from_numpy(wl.positional_code(math.isqrt(max(N, T) - 1) + 1)).to(dev)
    q[:, ::2, :, :64] += 2.0 * code[torch.arange(N, device=dev) * code.shape[0] // N]
    k.view(B, H, stride, d)[:, ::2, :T, :64] += 2.0 * code[torch.arange(T, device=dev) * code.shape[0] // T]
    k = k.to(torch.bfloat16).reshape(U * stride, d)
    hk = Hack(H, d, "bf16", U, T, N)
    return dict(kind="variance", hk=hk, q=q.to(torch.bfloat16), scale=scale,
                cache=Cache(k, k, np.arange(U, dtype=np.int64) * stride, np.full(U, T, np.int32)),
                sigma=torch.zeros(U, dtype=torch.float64, device=dev))


# ---- a pass -----------------------------------------------------------------------------------------------------------
def _run_schedule(s):
    hk, mc = s["hk"], s["cache"]
    mc.reset()
    last = len(s["steps"]) - 1
    for i, (q, k, v, budget, out) in enumerate(s["steps"]):
        hk.step(mc, q, k, v, s["types"], budget, s["n_init"], s["scale"], out, final=s["merge"] and i == last)


def run(state):
    s = state
    if s["kind"] == "variance":
        s["hk"].head_variance(s["q"], s["cache"], s["scale"], s["sigma"])
        return s["sigma"]
    if s["kind"] == "compress":
        hk = s["hk"]
        B, _, n, _ = s["q"].shape
        score = hk.score_static if s["static"] else hk.score
        score(s["q"], s["src"], s["scale"], s["importance"], k_new=s["k_new"], n_obs=s["n_obs"])
        length = hk.select(B, s["importance"], s["t_in"], s["types"], s["budget"], s["n_init"], n, s["kept"])
        hk.compact(B, n, s["src"], s["kept"], s["dst"], s["k_new"], s["v_new"])
        return {"importance": s["importance"], "kept": s["kept"], "len": length, "k": s["dst"].k, "v": s["dst"].v, "pos": s["dst"].pos}
    if s["graph"] is not None:
        s["graph"].replay()
    else:
        _run_schedule(s)
    mc = s["cache"]
    off, length = mc.view()
    return {"out": [st[4] for st in s["steps"]], "k": mc.k, "v": mc.v, "pos": mc.pos, "off": off, "len": length}
