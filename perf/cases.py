"""What the framework's speed is measured on: calls that a program which schedules batches
with it makes, through the public entry points of paper_2209_00159_amd.orloj.

Kinds of case (the field "kind"):
  score     one decision: every candidate batch of every model scored and a batch selected
            per model (Scorer.score + Scorer.select)
  affine    the same under the affine batch-latency law; "noalloc": the entry point that
            allocates nothing
  iterate   one Algorithm 1 iteration for every model (Iterator.iterate)
  refresh   a profile refresh: histograms -> CDF tables, their support and the model laws
            (Iterator.build)
  feedback  a profiling window: counts cleared, finished requests' latencies accumulated,
            the tables rebuilt
  loop      the scheduling runtime over an arrival trace (Sched.simulate): admissions, drop
            phase, one scoring round per tick with an idle model

Sizes are those of the repository's five configurations and their neighbourhood.  Histograms
come from analytic execution-time laws (lognormal mixtures, normal modes of layer-skipping
models, geometric decoding steps) scaled by 1 + 0.08 (s - 1) with the batch size; queues are
backlogs of requests of random age in deadline order.  Tables are made on the GPU.
"""
import math

import numpy as np
import torch

from paper_2209_00159_amd import orloj as O
from paper_2209_00159_amd import workloads as W

DEV = "cuda"
LAWS = ("lognormal", "normal", "geometric")
BATCHES = ("all", "pow2", "thirds")


def _case(name, kind, models, classes, bins, smax, queue, span_ms, law, lo_ms, hi_ms, slo_lo,
          slo_hi, slo_scale=1.0, batches="all", ragged=False, rect=False, cost=False, trim=True,
          noalloc=False, steps=0, samples=1 << 20, arrivals=0, b=1e-4):
    c = dict(kind=kind, models=models, classes=classes, bins=bins, smax=smax, queue=queue,
             span_ms=span_ms, law=law, lo_ms=lo_ms, hi_ms=hi_ms, slo_lo=slo_lo, slo_hi=slo_hi,
             slo_scale=slo_scale, batches=batches, ragged=ragged, rect=rect, cost=cost, trim=trim,
             noalloc=noalloc, steps=steps, samples=samples, arrivals=arrivals, b=b)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one small model behind one worker: a decision is a few launches and their latency
        _case("score-tiny", "score", 1, 4, 128, 16, 64, 200.0, "lognormal", 20.0, 90.0, 0.6, 4.0),
        # a text model: geometric decoding steps, 32 applications, batches to 64
        _case("score-text", "score", 1, 32, 1024, 64, 400, 2000.0, "geometric", 1.0, 10.0, 2.0, 5.0),
        # a layer-skipping vision model: batches to 128, a long backlog with miss costs, SLOs
        # relaxed so that the large batches can finish
        _case("score-vision", "score", 1, 64, 2048, 128, 4096, 60.0, "normal", 5.0, 25.0, 1.5, 4.0,
              slo_scale=5.0, cost=True),
        # a server of 64 models with short queues
        _case("score-server", "score", 64, 16, 1024, 32, 48, 1000.0, "lognormal", 20.0, 200.0, 2.0,
              5.0, ragged=True),
        # a fleet at saturation: every prefix of 128 deep queues at 64 batch sizes
        _case("score-fleet", "score", 128, 32, 4096, 64, 256, 1000.0, "lognormal", 5.0, 40.0, 1.5, 5.0),
        # a what-if study: prefixes past the batch size, an odd bin count, sparse batch sizes,
        # histograms of an odd number of samples, no support table
        _case("score-whatif", "score", 5, 21, 1501, 48, 100, 800.0, "lognormal", 10.0, 120.0, 1.5,
              5.0, batches="thirds", ragged=True, rect=True, cost=True, trim=False, samples=99_991),
        # the fleet under the affine law: one table per class
        _case("affine-fleet", "affine", 128, 32, 4096, 64, 256, 1000.0, "lognormal", 5.0, 40.0, 1.5, 5.0),
        # Algorithm 1 for the fleet
        _case("iterate-fleet", "iterate", 128, 32, 4096, 64, 256, 1000.0, "lognormal", 5.0, 40.0, 1.5, 5.0),
        # Algorithm 1 for one model with a long queue, miss costs and two cost steps a request
        _case("iterate-long", "iterate", 1, 64, 2048, 128, 4096, 60.0, "normal", 5.0, 25.0, 1.5, 4.0,
              slo_scale=5.0, cost=True, steps=2),
        # profile refresh of a quarter of the fleet
        _case("refresh", "refresh", 32, 32, 4096, 64, 0, 1000.0, "lognormal", 5.0, 40.0, 1.5, 5.0),
        # a profiling window of a million samples over 16 models
        _case("feedback", "feedback", 16, 16, 1000, 24, 0, 1000.0, "lognormal", 20.0, 200.0, 2.0, 5.0,
              samples=1_000_000),
        # the scheduling runtime: 16 workers, an overloaded open-loop arrival trace
        _case("loop", "loop", 16, 8, 2048, 64, 0, 500.0, "lognormal", 5.0, 40.0, 1.5, 5.0, arrivals=640),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the largest listed case's candidate-bin evaluations and table entries
MOST_EVALS = 128 * 2080 * 4096
MOST_ENTRIES = 32 * 64 * 32 * 4096


def draw(rng):
    kind = rng.choice(["score", "score", "score", "affine", "affine", "iterate", "refresh",
                       "feedback", "loop"])
    law = rng.choice(["lognormal", "lognormal", "normal", "geometric"])
    bins = _log(rng, 64, 4096)
    hi = rng.uniform(20.0, 60.0)
    c = _case(None, kind, _log(rng, 1, 128), _log(rng, 2, 64), bins, _log(rng, 8, 128),
              _log(rng, 8, 512), rng.uniform(8.0, 25.0) * hi, law, 0.2 * hi if law != "geometric" else 0.02 * hi,
              hi if law != "geometric" else 0.2 * hi, 1.5, rng.uniform(3.0, 5.0),
              slo_scale=math.exp(rng.uniform(0.0, math.log(4.0))), batches=rng.choice(BATCHES),
              ragged=rng.random() < 0.5, cost=rng.random() < 0.3, trim=rng.random() < 0.8,
              samples=rng.choice([1 << 20, rng.randrange(10_000, 2_000_000)]),
              b=10.0 ** rng.uniform(-5.0, -3.0))
    if kind == "score" and rng.random() < 0.25:
        c["rect"] = True
        c["queue"] = min(c["queue"], 128)
    if kind == "affine":
        c["noalloc"] = rng.random() < 0.4
    if kind == "iterate":
        c["queue"] = _log(rng, 16, 4096)
        c["steps"] = rng.choice([0, 0, 2, 3])
        c["models"] = max(1, min(c["models"], 65536 // c["queue"]))
    if kind in ("refresh", "feedback"):
        c["queue"] = 0
    if kind == "feedback":
        c["samples"] = _log(rng, 1000, 4_000_000)
    if kind == "loop":
        c.update(queue=0, models=min(c["models"], 32), classes=min(c["classes"], 16),
                 arrivals=_log(rng, 40, 640), rect=False, trim=True)
    while c["models"] > 1 and (_entries(c) > MOST_ENTRIES or _evals(c) > 0.5 * MOST_EVALS):
        c["models"] = max(1, c["models"] * 2 // 3)
    return c


# -- sizes ------------------------------------------------------------------
def _batches(c):
    s = c["smax"]
    if c["batches"] == "all":
        return np.arange(1, s + 1, dtype=np.int32)
    step = 2.0 if c["batches"] == "pow2" else 1.5
    out, x = {s}, 1.0
    while x < s:
        out.add(int(round(x)))
        x *= step
    return np.array(sorted(out), np.int32)


def _caps(c):
    """(batch size, longest prefix) of a queue of the mean length."""
    n = max(1, c["queue"] // 2) if c["ragged"] else c["queue"]
    return [(int(s), n if c["rect"] else min(int(s), n)) for s in _batches(c)]


def _entries(c):
    return c["models"] * c["classes"] * c["bins"] * (1 if c["kind"] == "affine" else len(_batches(c)))


def _evals(c):
    return c["models"] * c["bins"] * sum(n for _, n in _caps(c))


def _distinct(c, n):
    return c["classes"] * (1.0 - (1.0 - 1.0 / c["classes"]) ** n)


def work(case):
    c, M, K = case, case["models"], case["bins"]
    bs = _batches(c)
    if c["kind"] in ("score", "affine"):
        caps = _caps(c)
        out = M * sum(4 * n * (n + 1) // 2 + 16 * n for _, n in caps)
        nmax = max(n for _, n in caps)
        if c["kind"] == "score":
            return {"bytes": int(M * sum(_distinct(c, n) for _, n in caps) * K * 4 + out), "flops": int(3 * _evals(c))}
        return {"bytes": int(M * _distinct(c, nmax) * K * 4 + out),
                "flops": int(3 * M * nmax * K + M * sum(10 * n * (n + 1) // 2 for _, n in caps))}
    if c["kind"] == "iterate":
        n = M * max(1, c["queue"] // (2 if c["ragged"] else 1))
        return {"bytes": int(M * len(bs) * c["classes"] * 4 + n * 40), "flops": int(n * (len(bs) + 40))}
    if c["kind"] == "refresh":
        return {"bytes": 16 * _entries(c), "flops": 12 * _entries(c)}
    if c["kind"] == "feedback":
        return {"bytes": 12 * _entries(c) + 24 * c["samples"], "flops": 2 * _entries(c) + 2 * c["samples"]}
    # loop: a decision reads the rows of a short queue at every batch size
    return {"bytes": int(c["arrivals"] * 0.3 * len(bs) * _distinct(c, 6) * K * 4),
            "flops": int(c["arrivals"] * 0.3 * 3 * len(bs) * 6 * K)}


# -- inputs -----------------------------------------------------------------
def _scale(bs):
    return 1.0 + 0.08 * (np.asarray(bs, np.float64) - 1.0)


def _counts(c, seed, solo):
    """Histogram counts [M, nbs, C, K] int32 (solo: [M, C, K]) and the class medians [M, C] (ms)."""
    M, C, K = c["models"], c["classes"], c["bins"]
    w = c["span_ms"] / K
    g = torch.Generator(device=DEV).manual_seed(seed)

    def u(lo, hi, *shape):
        return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)

    scales = [1.0] if solo else list(_scale(_batches(c)))
    total = c["samples"] if c["kind"] != "feedback" else 1 << 20
    x = torch.arange(K + 1, device=DEV, dtype=torch.float64) * w
    out = torch.empty(M, len(scales), C, K, dtype=torch.int32, device=DEV)
    p50 = torch.empty(M, C, dtype=torch.float64, device=DEV)
    sc = torch.tensor(scales, device=DEV, dtype=torch.float64)[:, None, None]
    for q in range(M):
        if c["law"] == "lognormal":
            med, sig, w0 = u(c["lo_ms"], c["hi_ms"], 2, C, 1), u(0.2, 0.6, 2, C, 1), u(0.2, 0.8, C, 1)
            lx = torch.log(torch.clamp(x / sc, min=1e-300))
            F = w0 * torch.special.ndtr((lx - med[0].log()) / sig[0]) + \
                (1 - w0) * torch.special.ndtr((lx - med[1].log()) / sig[1])
        elif c["law"] == "normal":
            modes = torch.linspace(c["lo_ms"], c["hi_ms"], 3, device=DEV, dtype=torch.float64)
            wt = -torch.log(u(1e-9, 1.0, 3, C, 1))
            wt = wt / wt.sum(0)
            F = sum(wt[i] * torch.special.ndtr((x / sc - modes[i]) / (0.1 * modes[i])) for i in range(3))
        else:
            base, step = u(2.0 * c["lo_ms"], 8.0 * c["lo_ms"], C, 1), u(0.1, 1.0, C, 1) * 0.2 * c["hi_ms"]
            j = torch.clamp(torch.floor((x / sc - base) / step), min=0.0)
            F = -torch.expm1(j * math.log1p(-0.02))
        cum = torch.round(F * total)
        cum[..., 0], cum[..., -1] = 0.0, float(total)
        out[q] = torch.diff(torch.cummax(cum, -1).values, dim=-1).to(torch.int32)
        p50[q] = (torch.searchsorted(cum[0].contiguous(), torch.full((C, 1), 0.5 * total, device=DEV, dtype=torch.float64))[:, 0] - 0.5) * w
    return (out[:, 0].contiguous() if solo else out), p50.cpu().numpy()


def _workload(c, seed):
    """The workload (queues and grid; its tables stay on the GPU) and the counts."""
    solo = c["kind"] == "affine"
    counts, p50 = _counts(c, seed, solo)
    M, C, K = c["models"], c["classes"], c["bins"]
    rng = np.random.Generator(np.random.PCG64([seed, 7]))
    # queue lengths belong to the case: every seed's outputs have the same shapes
    lens = np.random.Generator(np.random.PCG64([M, c["queue"], 5])).integers(0, c["queue"] + 1, M)
    off, cls, dl, now = [0], [], [], []
    for q in range(M):
        n = int(lens[q]) if c["ragged"] and M > 1 else c["queue"]
        t = 60_000.0 + rng.uniform()
        k = rng.integers(0, C, n)
        slo = c["slo_scale"] * rng.uniform(c["slo_lo"], c["slo_hi"], n) * p50[q, k]
        d = t + slo * (1.0 - rng.uniform(0.0, 0.5, n))
        o = np.argsort(d, kind="stable")
        off.append(off[-1] + n)
        cls.append(k[o])
        dl.append(d[o])
        now.append(t)
    N = off[-1]
    bs = _batches(c)
    wl = W.Workload("perf", 0, M, C, K, bs, np.full(M, c["span_ms"] / K), np.zeros(0, np.uint32),
                    np.asarray(off, np.int64), np.concatenate(cls).astype(np.int32),
                    np.concatenate(dl).astype(np.float64), np.asarray(now), b_expo=c["b"],
                    cost=rng.uniform(0.0, 3.0, N) if c["cost"] else None)
    if solo:
        wl.c0_ms, wl.c1 = 0.92 * p50.min(axis=1), np.full(M, 0.08)
    steps = None
    if c["steps"]:
        S = c["steps"]
        sd = wl.deadline_ms[:, None] + np.arange(S) * rng.uniform(1.0, 10.0, (N, 1))
        sco = np.cumsum(rng.uniform(0.1, 1.0, (N, S)), axis=1)
        steps = (np.arange(N + 1, dtype=np.int64) * S, sd.reshape(-1), sco.reshape(-1))
    return wl, counts, p50, steps


def _samples(c, seed):
    g = torch.Generator(device=DEV).manual_seed(seed + 1)
    n, nb = c["samples"], len(_batches(c))
    m, b, k = (torch.randint(0, hi, (n,), generator=g, device=DEV, dtype=torch.int32)
               for hi in (c["models"], nb, c["classes"]))
    z = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    med = c["lo_ms"] + (c["hi_ms"] - c["lo_ms"]) * (k.double() + 0.5) / c["classes"]
    return m, b, k, med * torch.exp(0.4 * z) * (1.0 + 0.05 * b.double())


def prepare(case, seed):
    c = case
    ctx = O.Context()
    if c["kind"] == "feedback":
        nb, C, K, M = _batches(c), c["classes"], c["bins"], c["models"]
        width = torch.full((M,), c["span_ms"] / K, dtype=torch.float64, device=DEV)
        # every row keeps one count in its last bin, so that no row is without samples
        base = torch.zeros(M, len(nb), C, K, dtype=torch.int32, device=DEV)
        base[..., -1] = 1
        return dict(c=c, ctx=ctx, grid=O.make_grid(M, C, K, nb, width), width=width, base=base,
                    counts=torch.empty_like(base), ccdf=torch.empty(base.shape, dtype=torch.float32, device=DEV),
                    support=torch.empty(base.shape[:-1] + (2,), dtype=torch.int32, device=DEV),
                    samples=_samples(c, seed))
    if c["kind"] == "loop":
        counts, p50 = _counts(c, seed, False)
        M, C, K = c["models"], c["classes"], c["bins"]
        ccdf = torch.empty(counts.shape, dtype=torch.float32, device=DEV)
        support = torch.empty(counts.shape[:-1] + (2,), dtype=torch.int32, device=DEV)
        ctx.build_cdfs(counts, ccdf, support)
        width = torch.full((M,), c["span_ms"] / K, dtype=torch.float64, device=DEV)
        solo = np.ascontiguousarray(counts[:, 0].cpu().numpy()).view(np.uint32)
        bs = _batches(c)
        grid = O.make_grid(M, C, K, bs, width)
        rng = np.random.Generator(np.random.PCG64([seed, 11]))
        n = c["arrivals"]
        rel = np.cumsum(rng.exponential(6.4 / M, n))
        mod, cl = rng.integers(0, M, n).astype(np.int32), rng.integers(0, C, n).astype(np.int32)
        dl = rel + c["slo_scale"] * rng.uniform(c["slo_lo"], c["slo_hi"], n) * p50[mod, cl]
        ctx.sync()
        return dict(c=c, ctx=ctx, sched=O.Sched(ctx, grid, ccdf, support, p50, c["b"]), solo=solo,
                    trace=(rel, mod, cl, dl), width=np.full(M, c["span_ms"] / K), scale=_scale(bs), seed=seed)
    wl, counts, _, steps = _workload(c, seed)
    if c["kind"] in ("iterate", "refresh"):
        it = O.Iterator(wl, ctx, counts_device=counts)
        if steps is not None:
            it.set_queues(wl.queue_off, wl.cls, wl.deadline_ms, wl.now_ms, steps=steps)
        if c["kind"] == "iterate":
            it.build()
            ctx.sync()
            it.counts = it.ccdf = None
        return dict(c=c, it=it)
    sc = O.Scorer(wl, ctx, prefix_mode=O.PREFIX_RECT if c["rect"] else O.PREFIX_TRIANGLE,
                  counts_device=counts, trim=c["trim"])
    sc.build()
    ctx.sync()
    sc.counts = None
    return dict(c=c, sc=sc)


def run(state):
    c = state["c"]
    if c["kind"] in ("score", "affine"):
        sc = state["sc"]
        sc.score(noalloc=c["noalloc"])
        sc.select()
        return dict(P=sc.finish_prob[:sc.n_probs], E=sc.expected_finish[:sc.n_cands],
                    EL=sc.expected_latency[:sc.n_cands], S=sc.score_out[:sc.n_cands],
                    sel_n=sc.sel_n, sel_bs=sc.sel_bs, sel_score=sc.sel_score)
    if c["kind"] == "iterate":
        it = state["it"]
        it.iterate()
        return dict(timed_out=it.timed_out, score=it.score, cand_bs=it.cand_bs, batch=it.batch)
    if c["kind"] == "refresh":
        it = state["it"]
        it.build()
        return dict(ccdf=it.ccdf, support=it.support, law=it.law, disc=it.disc, model_el=it.model_el)
    if c["kind"] == "feedback":
        state["counts"].copy_(state["base"])
        rejected = O.accumulate(state["ctx"], state["grid"], state["counts"], *state["samples"])
        state["ctx"].build_cdfs(state["counts"], state["ccdf"], state["support"])
        return dict(counts=state["counts"], ccdf=state["ccdf"], support=state["support"], rejected=rejected)
    n = c["arrivals"]
    stats, states = state["sched"].simulate(state["trace"], 0.5, state["solo"], state["width"],
                                            state["scale"], seed=state["seed"], max_ticks=1_000_000,
                                            record_every=1, record_limit=n)
    picks = np.zeros((n, 3), np.int64)
    for i, s in enumerate(states):
        picks[i] = s[0], s[4], s[5]
    return dict(picks=picks, counts=np.array([stats[k] for k in ("ticks", "decisions", "dispatched", "dropped",
                                                                "on_time", "late", "arrivals")]))


def tolerance(case):
    """Four times what the first version showed against exact() and between orders of the sums."""
    return {"rel": 6e-7, "max": 3e-5, "differ": 0.01}


# -- the same in 64 bits ------------------------------------------------------
def _discounted(G, d):
    """Z[..., j] = sum over i <= j of G[..., i] d^(j - i), along the last dimension."""
    Z, s = G.clone(), 1
    d = torch.as_tensor(d, dtype=torch.float64, device=G.device)
    while s < G.shape[-1]:
        Z[..., s:] = Z[..., s:] + (d ** s) * Z[..., :-s].clone()
        s *= 2
    return Z


def _cdf(counts):
    cum = torch.cumsum(counts.to(torch.int64), -1)
    return cum.double() / cum[..., -1:].double()


def _priority(G, Z, tau, w, b):
    """P and the priority x E[L] of members with time left tau [..., m] on rows G, Z
    [..., n, K] and a bin width w that broadcasts against tau: two [..., n, m]."""
    K = G.shape[-1]
    u = tau / w
    inside = (tau > 0) & (u < K)
    k = torch.clamp(torch.floor(torch.where(inside, u, torch.zeros_like(u))), 0, K - 1).long()
    th = torch.where(inside, u - k, torch.zeros_like(u))

    def at(T, idx, below):
        ix = torch.clamp(idx, min=0).unsqueeze(-2).expand(*T.shape[:-1], idx.shape[-1])
        return torch.where((idx < 0).unsqueeze(-2), torch.full_like(T[..., :1], below), torch.gather(T, -1, ix))

    gk, gk1, zk = at(G, k - 1, 0.0), at(G, k, 0.0), at(Z, k - 2, 0.0)
    bw = b * w
    omd = -torch.expm1(-bw)
    cg = (omd / bw * torch.exp(-b * th * w)).unsqueeze(-2)
    psi = (-torch.expm1(-b * th * w) / bw).unsqueeze(-2)
    omd2 = (omd + torch.zeros_like(tau)).unsqueeze(-2)
    P = gk + th.unsqueeze(-2) * (gk1 - gk)
    num = cg * (gk - omd2 * zk) + (gk1 - gk) * psi
    past = (u >= K).unsqueeze(-2)
    zl = at(Z, torch.full_like(k, K - 2), 0.0)
    cgp = (omd / bw * torch.exp(-b * torch.clamp(tau - K * w, min=0.0))).unsqueeze(-2)
    num = torch.where(past, cgp * (1.0 - omd2 * zl), num)
    P = torch.where(past, torch.ones_like(P), P)
    live = (tau > 0).unsqueeze(-2)
    return torch.where(live, P, torch.zeros_like(P)), torch.where(live, num, torch.zeros_like(num))


def _exact_score(c, seed):
    wl, counts, _, _ = _workload(c, seed)
    affine, K, b = c["kind"] == "affine", c["bins"], c["b"]
    P, E, EL, S = [], [], [], []
    for q in range(c["models"]):
        lo, hi = int(wl.queue_off[q]), int(wl.queue_off[q + 1])
        N = hi - lo
        if N == 0:
            continue
        caps = [(i, int(s), N if c["rect"] else min(int(s), N)) for i, s in enumerate(wl.batch_sizes)]
        w = float(wl.bin_width_ms[q])
        group = max(1, int(3e7 // (max(n for *_, n in caps) * K)))
        for g0 in range(0, len(caps), group):
            part = caps[g0:g0 + group]
            n = max(x[2] for x in part)
            cls = torch.from_numpy(wl.cls[lo:lo + n].astype(np.int64)).to(DEV)
            tau = torch.from_numpy(wl.deadline_ms[lo:lo + n] - wl.now_ms[q]).to(DEV)
            cost = torch.ones_like(tau) if wl.cost is None else torch.from_numpy(wl.cost[lo:lo + n]).to(DEV)
            sz = torch.tensor([float(x[1]) for x in part], device=DEV, dtype=torch.float64)[:, None]
            if affine:
                ws, c0 = float(wl.c1[q]) * sz * w, float(wl.c0_ms[q])
                G = torch.cumprod(_cdf(counts[q])[cls], 0).expand(len(part), n, K)
            else:
                ws, c0 = torch.full_like(sz, w), 0.0
                G = torch.cumprod(_cdf(counts[q, part[0][0]:part[-1][0] + 1])[:, cls], 1)
            Z = _discounted(G, torch.exp(-b * ws).unsqueeze(-1))
            el = c0 + ws * (0.5 + (1.0 - G).sum(-1))
            p, num = _priority(G, Z, (tau - c0).expand(len(part), n), ws, b)
            num = num * cost
            for i, (_, _, cap) in enumerate(part):
                r, m = torch.tril_indices(cap, cap, device=DEV)
                low = torch.tril(torch.ones(cap, cap, device=DEV, dtype=torch.float64))
                P.append(p[i, r, m])
                E.append((p[i, :cap, :cap] * low).sum(-1))
                EL.append(el[i, :cap])
                S.append((num[i, :cap, :cap] * low).sum(-1) / el[i, :cap])
    return dict(P=torch.cat(P), E=torch.cat(E), EL=torch.cat(EL), S=torch.cat(S), sel_n=None,
                sel_bs=None, sel_score=None)


def _exact_laws(counts, bs, w, b):
    """law, disc [nbs, C, K] and model_el [nbs] of one model's counts."""
    F = _cdf(counts)
    s = torch.tensor(np.asarray(bs, np.float64), device=DEV)[:, None]
    mix = F.mean(1)
    law = F * (mix ** (s - 1))[:, None]
    el = w * (0.5 + (1.0 - mix ** s).sum(-1))
    return law, _discounted(law, math.exp(-b * w)), el


def _exact_refresh(c, seed):
    wl, counts, _, _ = _workload(c, seed)
    shape = counts.shape
    out = dict(ccdf=torch.empty(shape, dtype=torch.float64, device=DEV), support=None,
               law=torch.empty(shape, dtype=torch.float64, device=DEV),
               disc=torch.empty(shape, dtype=torch.float64, device=DEV),
               model_el=torch.empty(shape[:2], dtype=torch.float64, device=DEV))
    for q in range(c["models"]):
        cum = torch.cumsum(counts[q].to(torch.int64), -1)
        out["ccdf"][q] = (cum[..., -1:] - cum).double() / cum[..., -1:].double()
        out["law"][q], out["disc"][q], out["model_el"][q] = _exact_laws(
            counts[q], wl.batch_sizes, float(wl.bin_width_ms[q]), c["b"])
    return out


def _exact_iterate(c, seed):
    wl, counts, _, steps = _workload(c, seed)
    score = torch.zeros(max(int(wl.queue_off[-1]), 1), dtype=torch.float64, device=DEV)
    for q in range(c["models"]):
        lo, hi = int(wl.queue_off[q]), int(wl.queue_off[q + 1])
        if hi == lo:
            continue
        w, now = float(wl.bin_width_ms[q]), float(wl.now_ms[q])
        D = wl.deadline_ms[lo:hi]
        if steps is None:
            sd, sco = D[:, None], np.ones((hi - lo, 1))
        else:
            sd, sco = (steps[i].reshape(-1, c["steps"])[lo:hi] for i in (1, 2))
        first = (counts[q] > 0).to(torch.int8).argmax(-1).cpu().numpy()          # [nbs, C]
        keep = (sd[:, -1] - now)[None] > first[:, wl.cls[lo:hi]] * w              # [nbs, n]
        fits = [(D[np.argmax(keep[i])], int(s), i) for i, s in enumerate(wl.batch_sizes) if keep[i].sum() >= s]
        if not fits:
            continue
        i = max(fits)[2]
        law, disc, el = _exact_laws(counts[q, i:i + 1], wl.batch_sizes[i:i + 1], w, c["b"])
        cl = torch.from_numpy(wl.cls[lo:hi].astype(np.int64)).to(DEV)
        num = torch.zeros(hi - lo, dtype=torch.float64, device=DEV)
        for j in range(sd.shape[1]):
            inc = torch.from_numpy(sco[:, j] - (sco[:, j - 1] if j else 0.0)).to(DEV)
            tau = torch.from_numpy(sd[:, j] - now).to(DEV)[:, None]
            _, x = _priority(law[0][cl][:, None], disc[0][cl][:, None], tau, torch.full_like(tau, w), c["b"])
            num += inc * x[:, 0, 0]
        if wl.cost is not None:
            num = num * torch.from_numpy(wl.cost[lo:hi]).to(DEV)
        score[lo:hi] = torch.where(torch.from_numpy(keep[i]).to(DEV), num / el[0], torch.zeros_like(num))
    return dict(timed_out=None, score=score, cand_bs=None, batch=None)


def _exact_feedback(c, seed):
    m, b, k, lat = _samples(c, seed)
    nb, C, K, M = len(_batches(c)), c["classes"], c["bins"], c["models"]
    bin_ = torch.clamp(torch.floor(lat / (c["span_ms"] / K)), max=K - 1).long()
    row = (m.long() * nb + b.long()) * C + k.long()
    counts = torch.bincount(row * K + bin_, minlength=M * nb * C * K).reshape(M, nb, C, K)
    counts[..., -1] += 1
    cum = torch.cumsum(counts, -1)
    return dict(counts=None, ccdf=(cum[..., -1:] - cum).double() / cum[..., -1:].double(), support=None, rejected=None)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("score", "affine"):
        return _exact_score(case, seed)
    if kind == "iterate":
        return _exact_iterate(case, seed)
    if kind == "refresh":
        return _exact_refresh(case, seed)
    if kind == "feedback":
        return _exact_feedback(case, seed)
    return None
