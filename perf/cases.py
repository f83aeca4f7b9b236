"""Performance cases of the allocation search and the computations around it.

Each case is one pass through a public entry point of ``paper_2604_15186_amd.alp`` as a scheduler
calls it.  The search cases follow the workloads of ``workloads/alp_workloads.py`` (2 to 5 LLMs per
workflow, 48 to 128 options per LLM, one query or thousands), the others its trace statistics,
placement, budget split, largest sustainable rate and pruned search at the sizes of ``bench.py``.
``draw`` varies what a deployment varies: LLMs per workflow, tensor-parallel degrees, GPU shares,
replica limits (so option counts that fill no wavefront), budgets, targets and batch sizes.

Results are integers and compared exactly.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2604_15186_amd import alp
from workloads import CONFIGS, make_batch, make_custom, target_from_tmax

LARGEST_SEARCH = 1 << 35        # candidates of the largest pass
TP_SETS = ((1, 2), (1, 2, 4), (1, 2, 4, 8))
SHARE_SETS = ((4,), (2, 4), (1, 2, 4), (1, 2, 3, 4))        # quarters of a GPU


def listed():
    return [
        # One query of the smallest workflow (generator + verifier on one node), answered while
        # the caller waits: latency of the call.
        {"name": "search-2llm", "kind": "search", "config": 0},
        # The same call for a 3-LLM beam-search workflow on two nodes (2^21 candidates).
        {"name": "search-3llm", "kind": "search", "config": 1},
        # One 4-LLM query (2^28 candidates) queued on the stream, as a serving loop re-plans.
        {"name": "queue-4llm", "kind": "queue", "config": 2, "count": 1},
        # The largest space: a 5-LLM workflow on eight nodes (2^35 candidates).
        {"name": "queue-5llm", "kind": "queue", "config": 3, "count": 1},
        # A fleet re-plan: 4,096 independent 3-LLM workflows in one queued call.
        {"name": "queue-3llm-x4096", "kind": "queue", "config": 4, "count": 4096},
        # Budget and rate sweep of a few workflows whose 72 options fill no whole wavefront
        # (tp up to 8, three shares, six replicas), through the host-buffer batch call.
        {"name": "batch-4llm-ragged", "kind": "batch", "llms": 4, "tp": 4, "shares": 3,
         "replicas": 6, "points": 6, "frac_tp": False, "gpus": 29, "instances": 6, "count": 24},
        # Four 4-LLM workflows sharing 32 GPUs: every budget of each searched, then the split.
        {"name": "split-4x4llm-g32", "kind": "split", "llms": 4, "tp": 4, "shares": 4,
         "replicas": 8, "points": 8, "frac_tp": False, "gpus": 32, "instances": 4, "policy": 0},
        # The paper's own pruned search at its scheduler micro-benchmark point.
        {"name": "pruned-5llm-g16-f10", "kind": "pruned", "llms": 5, "gpus": 16, "fractions": 10,
         "count": 1},
        # Statistics of a day's recorded beam-search requests, in the order they completed.
        {"name": "stats-beam-logged", "kind": "stats", "shape": "beam", "traces": 20000,
         "order": "logged"},
        # The same requests merged from several collectors: calls in no order within a trace.
        {"name": "stats-beam-shuffled", "kind": "stats", "shape": "beam", "traces": 20000,
         "order": "shuffled"},
        # Placing the fleet re-plan's allocations on their nodes.
        {"name": "place-x4096", "kind": "place", "config": 4, "count": 4096},
        # Largest sustainable rate of every workflow of the fleet (sets the targets).
        {"name": "tmax-x4096", "kind": "tmax", "config": 4, "count": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _draw_space(rng, llms, candidates):
    """A space of the given number of LLMs with at most `candidates` candidates."""
    while True:
        c = {"llms": llms, "tp": rng.randint(2, 4), "shares": rng.randint(1, 4),
             "replicas": rng.randint(2, 16), "points": rng.randint(4, 16),
             "frac_tp": rng.random() < 0.25}
        if 24 <= _options(c) <= 256 and _options(c) ** llms <= candidates:
            return c


def draw(rng):
    kind = rng.choice(["search", "queue", "queue", "batch", "split", "pruned", "stats", "place",
                       "tmax"])
    if kind in ("search", "queue", "batch", "tmax"):
        llms = rng.randint(2, 5 if kind != "batch" else 4)
        c = {"kind": kind, **_draw_space(rng, llms, LARGEST_SEARCH)}
        c["gpus"] = _log_int(rng, 4, 64)
        if kind != "search":
            most = LARGEST_SEARCH // 4 // _options(c) ** llms if kind != "tmax" else 4096
            c["count"] = _log_int(rng, 1, max(1, min(4096, most)))
            c["instances"] = min(c["count"], 256) if kind != "batch" else \
                min(c["count"], rng.randint(1, 16))
        return c
    if kind == "split":
        flows = rng.randint(2, 6)
        gpus = _log_int(rng, 2 * flows, 48)
        llms = rng.randint(2, 4)
        c = _draw_space(rng, llms, LARGEST_SEARCH // (flows * (gpus + 1)))
        return {"kind": kind, **c, "gpus": gpus, "instances": flows, "policy": rng.randint(0, 1)}
    if kind == "pruned":
        llms = rng.randint(2, 5)
        if llms <= 3:
            return {"kind": kind, "llms": llms, "gpus": _log_int(rng, 4, 128),
                    "fractions": rng.randint(2, 16), "count": _log_int(rng, 8, 64)}
        return {"kind": kind, "llms": llms, "gpus": rng.randint(4, 20),
                "fractions": rng.randint(4, 10), "count": _log_int(rng, 1, 4)}
    if kind == "stats":
        shape = rng.choice(["beam", "rag"])
        return {"kind": kind, "shape": shape, "traces": _log_int(rng, 200, 20000),
                "order": rng.choice(["logged", "shuffled"])}
    return {"kind": kind, "config": rng.choice([1, 2, 4]), "count": _log_int(rng, 16, 1000)}


# ---- inputs ----------------------------------------------------------------------------------

def _options(c):
    return len(TP_SETS[c["tp"] - 2]) * len(SHARE_SETS[c["shares"] - 1]) * c["replicas"]


def _profiles(case, seed):
    """Profile tables of the case's workflows and, per query, instance, budget and the target
    as a fraction of the largest sustainable rate (ppm)."""
    kind, s = case["kind"], int(seed) % (1 << 31)
    if kind == "pruned":
        # As the scheduler micro-benchmark: up to 8 shares spread over 1..F, F units per GPU.
        F, n = case["fractions"], case["count"]
        shares = sorted({max(1, round(F * (k + 1) / min(F, 8))) for k in range(min(F, 8))})
        b = make_custom(s, case["llms"], (1, 2, 4, 8), shares, 4, 8, case["gpus"], count=n,
                        frac_den=F, param_range=(1e9, 70e9), alpha=0.5)
        return b, np.arange(n), b["G"], b["u_ppm"]
    if "config" in case:
        n = case.get("count", 1)
        b = make_batch(case["config"], [s * 5000 + i for i in range(n)])
        return b, np.arange(n), b["G"], b["u_ppm"]
    n = case.get("instances", 1)
    b = make_custom(s, case["llms"], TP_SETS[case["tp"] - 2], SHARE_SETS[case["shares"] - 1],
                    case["replicas"], case["points"], case["gpus"], count=n,
                    frac_tp=case["frac_tp"])
    count = case.get("count", 1) if kind != "split" else n
    rng = np.random.default_rng([s, 3])
    inst = np.arange(count) % n
    G = np.full(count, case["gpus"])
    if kind == "batch":                     # the sweep's budgets, up to the case's
        G = rng.integers(max(1, case["gpus"] // 2), case["gpus"] + 1, count)
    return b, inst, G.astype(np.uint32), rng.integers(100_000, 900_001, count)


def _targets(ctx, inst, G, ppm):
    tmax = ctx.max_throughput(G, instances=inst)
    return np.asarray([target_from_tmax(int(u), int(t)) for u, t in zip(ppm, tmax)],
                      dtype=np.uint32)


def _traces(case, seed):
    """Recorded requests as workloads/traces.py draws them (beam: rounds of 3 generator calls,
    then 1 to 3 verifier calls; rag: embed, rerank 5 to 20 documents, one time in three or so
    again, generate), drawn for all requests at once: (LLMs, offsets, llm, start, end)."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    R = case["traces"]

    def uniform(lo, hi, *size):
        return torch.randint(lo, hi, size, generator=g, device=dev)

    def duration(mean, *size):
        z = torch.randn(*size, generator=g, device=dev, dtype=torch.float64)
        return torch.clamp(torch.exp(0.5 * z + float(np.log(mean)) - 0.125).round(), min=1).long()

    # One row per round of a request; columns are the round's calls: LLM, start and end relative
    # to the round, used or not.
    if case["shape"] == "beam":
        llms, rounds = 2, uniform(8, 282, R)
        n = int(rounds.sum())
        gs = uniform(0, 2000, n, 3)
        ge = gs + duration(300_000, n, 3)
        k = torch.tensor([1, 2, 2, 2, 2, 2, 3, 3, 3, 3], device=dev)[uniform(0, 10, n)]
        vs = ge.max(1, keepdim=True).values + uniform(100, 5000, n, 1) + uniform(0, 1000, n, 3)
        ve = vs + duration(80_000, n, 3)
        used = torch.cat([torch.ones(n, 3, dtype=torch.bool, device=dev),
                          torch.arange(3, device=dev)[None] < k[:, None]], 1)
        start, end = torch.cat([gs, vs], 1), torch.cat([ge, ve], 1)
        llm = torch.tensor([0, 0, 0, 1, 1, 1], device=dev).expand(n, 6)
    else:
        llms = 3
        rounds = 1 + (torch.rand(R, generator=g, device=dev) < 0.3).long()
        n = int(rounds.sum())
        last = torch.zeros(n, dtype=torch.bool, device=dev)
        last[torch.cumsum(rounds, 0) - 1] = True
        es = torch.zeros(n, 1, dtype=torch.long, device=dev)
        ee = duration(10_000, n, 1)
        k = uniform(5, 21, n)
        rs = ee + uniform(2000, 20_000, n, 1) + uniform(0, 500, n, 20)
        re = rs + duration(30_000, n, 20)
        rerank = torch.arange(20, device=dev)[None] < k[:, None]
        qs = torch.where(rerank, re, 0).max(1, keepdim=True).values + uniform(100, 2000, n, 1)
        qe = qs + duration(2_000_000, n, 1)
        used = torch.cat([torch.ones(n, 1, dtype=torch.bool, device=dev), rerank, last[:, None]], 1)
        start, end = torch.cat([es, rs, qs], 1), torch.cat([ee, re, qe], 1)
        llm = torch.tensor([0] + [1] * 20 + [2], device=dev).expand(n, 22)
    span = torch.where(used, end, 0).max(1).values + uniform(100, 5000, n)
    owner = torch.repeat_interleave(torch.arange(R, device=dev), rounds)
    before = torch.cumsum(span, 0) - span
    first = torch.cumsum(rounds, 0) - rounds
    base = uniform(0, 1 << 40, R)[owner] + before - before[first][owner]
    start, end = start + base[:, None], end + base[:, None]
    order = torch.argsort(torch.where(used, end, torch.iinfo(torch.int64).max), dim=1, stable=True)
    kept = used.gather(1, order)
    start, end, llm = (a.gather(1, order)[kept] for a in (start, end, llm))
    counts = torch.zeros(R, dtype=torch.long, device=dev).index_add_(0, owner, used.sum(1))
    offsets = torch.zeros(R + 1, dtype=torch.long, device=dev)
    offsets[1:] = torch.cumsum(counts, 0)
    if case["order"] == "shuffled":
        trace = torch.repeat_interleave(torch.arange(R, device=dev), counts)
        p = torch.argsort(trace * (1 << 31) + uniform(0, 1 << 31, len(trace)))
        start, end, llm = start[p], end[p], llm[p]
    return llms, offsets, llm.to(torch.int32).contiguous(), start.contiguous(), end.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "stats":
        return {"kind": kind, "ctx": alp.StatsContext(), "traces": _traces(case, seed)}
    batch, inst, G, ppm = _profiles(case, seed)
    inst = inst.astype(np.uint32)
    ctx = alp.Context(batch)
    st = {"kind": kind, "ctx": ctx, "inst": inst, "G": G}
    if kind == "tmax":
        return st
    if kind == "split":                     # targets at an even share of the pool
        st["total"], st["policy"] = case["gpus"], case["policy"]
        G = np.maximum(1, G // len(G)).astype(np.uint32)
    st["lam"] = _targets(ctx, inst, G, ppm)
    if kind == "place":
        st["found"] = ctx.search_batch(G, st["lam"])
    if kind == "queue":
        st["q"] = [torch.from_numpy(a.view(np.int32)).cuda() for a in (G, st["lam"], inst)]
        st["out"] = torch.zeros(len(G) * alp.RESULT_DTYPE.itemsize, dtype=torch.uint8,
                                device="cuda")
    return st


# ---- one pass --------------------------------------------------------------------------------

def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "stats":
        return ctx.compute(*state["traces"]).view(np.uint64)
    G, inst = state["G"], state["inst"]
    if kind == "tmax":
        return ctx.max_throughput(G, instances=inst)
    lam = state["lam"]
    if kind == "search":
        return np.frombuffer(ctx.search(0, int(G[0]), int(lam[0])), dtype=np.uint32)
    if kind == "queue":
        ctx.search_batch_async(state["q"][0], state["q"][1], state["out"], instances=state["q"][2])
        return state["out"]
    if kind == "batch":
        return ctx.search_batch(G, lam, instances=inst).view(np.uint32)
    if kind == "split":
        plan, gpus, found = ctx.allocate_workflows(lam, state["total"], state["policy"])
        out = {"plan": np.frombuffer(plan, dtype=np.uint32)}
        return out if gpus is None else {**out, "gpus": gpus, "found": found.view(np.uint32)}
    if kind == "pruned":
        return ctx.search_pruned(G, lam).view(np.uint32)
    return ctx.place(state["found"], G).view(np.uint32)


def work(case):
    """Searches: every candidate's budget test and latency minimum (two operations), the profile
    tables read once and one 48-byte record per query.  Statistics: 20 bytes per call."""
    kind = case["kind"]
    if kind == "stats":
        calls = case["traces"] * (762 if case["shape"] == "beam" else 19)
        return {"bytes": 20 * calls + 8 * case["traces"], "flops": 10 * calls}
    if "config" in case:
        cfg = CONFIGS[case["config"]]
        llms, curves = cfg.num_llms, len(cfg.tp_values) * len(cfg.frac_q)
        options, points = curves * cfg.max_replicas, cfg.num_points
    elif kind == "pruned":
        llms, curves = case["llms"], 4 * min(8, case["fractions"])
        options, points = curves * 4, 8
    else:
        llms, options, points = case["llms"], _options(case), case["points"]
        curves = options // case["replicas"]
    count = case.get("count", 1)
    tables = case.get("instances", count) * llms * (curves * (8 * points + 1) + 16)
    if kind == "split":
        count = case["instances"] * (case["gpus"] + 1)
    per_query = {"place": 48 + 272 + 4, "tmax": 12, "pruned": 12 + 64}.get(kind, 12 + 48)
    flops = {"place": 16 * 64, "tmax": llms * options * 16, "pruned": llms * options * 16}
    return {"bytes": (0 if kind == "place" else tables) + per_query * count,
            "flops": count * flops.get(kind, 2 * options ** llms)}


def tolerance(case):
    return "exact"


# ---- plain statements ------------------------------------------------------------------------

def _terms(b, i, lam):
    """Instance i's option terms at target lam, each [LLM][option]: deployable, sustains the
    target, latency contribution, saturation rate, share units."""
    sp = b["space"]
    tp, fq = np.asarray(sp["tp"], np.int64), np.asarray(sp["fq"], np.int64)
    D, K, Q = int(sp["D"]), int(sp["K"]), int(sp["Q"])
    d = np.arange(1, D + 1)
    tpq = (tp[:, None] * fq[None, :]).reshape(-1)
    out = []
    for m in range(int(sp["M"])):
        n, p, W = int(b["n"][i, m]), int(b["p"][i, m]), int(b["W"][i, m])
        ok = (b["allowed"][i, m].reshape(-1) != 0) & (W * Q <= tpq * int(b["H"]))
        rate = b["rate"][i, m].reshape(-1, K).astype(np.int64)
        lat = b["lat"][i, m].reshape(-1, K).astype(np.int64)
        r = (-(-(lam * n) // (1000 * d)))[None, :]
        k = (rate[:, None, :] < r[:, :, None]).sum(2)
        hi, lo = np.clip(k, 0, K - 1), np.clip(k - 1, 0, K - 1)
        row = np.arange(len(rate))[:, None]
        r0, r1, l0, l1 = rate[row, lo], rate[row, hi], lat[row, lo], lat[row, hi]
        w = np.maximum(1, r1 - r0)
        at = np.clip(r, r0, r0 + w)
        ell = np.where(k == 0, lat[:, :1], (l0 * (w - (at - r0)) + l1 * (at - r0)) // w)
        tau = np.minimum(1000 * d[None, :] * rate[:, -1:] // n, 0xFFFFFFFF)
        out.append((np.repeat(ok, D), (r <= rate[:, -1:]).reshape(-1), (ell * n // p).reshape(-1),
                    tau.reshape(-1), (tpq[:, None] * d[None, :]).reshape(-1)))
    return [np.stack(a) for a in zip(*out)]


def _tmax(terms, cap):
    ok, _, _, tau, u = terms
    best = 0
    for t in np.unique(tau[ok]):
        need = np.where(ok & (tau >= t), u, 1 << 40).min(1).sum()
        best = int(t) if need <= cap else best
    return best


def _best(terms, cap):
    """Lowest latency within cap share units and its lowest index, by suffix tables: the least
    latency of the LLMs m.. within each number of units."""
    ok, thr, c, _, u = terms
    M, O = c.shape
    none = 1 << 60
    cost = np.where(ok & thr, c, none)
    cap = min(int(cap), int(u.max()) * M)
    left = np.arange(cap + 1)[None, :] - u[:, :, None]              # [LLM][option][units]
    best, pick = np.zeros(cap + 1, np.int64), []
    for m in range(M - 1, -1, -1):
        total = np.where(left[m] >= 0, cost[m][:, None] + best[np.maximum(left[m], 0)], none)
        pick.insert(0, total.argmin(0))                             # the lowest option on ties
        best = np.minimum(total.min(0), none)
    if best[cap] >= none:
        return None
    options, at = [], cap
    for m in range(M):
        options.append(int(pick[m][at]))
        at -= int(u[m][options[-1]])
    return int(best[cap]), options


def _record(b, terms, cap):
    """alp_result_t of a query as 12 words."""
    rec = np.zeros(1, dtype=alp.RESULT_DTYPE)[0]
    found = _best(terms, cap)
    if found is None:
        rec["index"], rec["status"] = alp.NO_INDEX, alp.ALP_INFEASIBLE
        return np.frombuffer(rec, dtype=np.uint32)
    L, options = found
    sp, M, x = b["space"], len(options), 0
    nf, D = len(sp["fq"]), int(sp["D"])
    for o in options:
        x = x * nf * len(sp["tp"]) * D + o
    m, o = np.arange(M), np.asarray(options)
    rec["index"], rec["latency_us"] = x, L
    rec["throughput_milli"] = terms[3][m, o].min()
    rec["gpu_units"] = terms[4][m, o].sum()
    rec["tp"][:M] = np.asarray(sp["tp"])[o // D // nf]
    rec["frac_units"][:M] = np.asarray(sp["fq"])[o // D % nf]
    rec["replicas"][:M] = o % D + 1
    return np.frombuffer(rec, dtype=np.uint32)


def _exact_stats(case, seed):
    llms, offsets, llm, start, end = _traces(case, seed)
    R = len(offsets) - 1
    group = torch.repeat_interleave(torch.arange(R, device=llm.device), offsets.diff()) * llms + llm
    low = torch.full((R * llms,), 1 << 62, device=llm.device).scatter_reduce_(
        0, group, start, "amin")[group]
    s, e = start - low, end - low                       # below 2^32, so groups stay apart
    p = torch.argsort((group << 36) + s)
    group, s, e = group[p], s[p] + (group[p] << 36), e[p] + (group[p] << 36)
    reach = torch.cummax(e, 0).values
    before = torch.cat([s[:1], reach[:-1]])
    active = torch.clamp(e - torch.maximum(s, before), min=0)
    out = np.zeros(llms, dtype=alp.STATS_DTYPE)
    for m in range(llms):
        sel = group % llms == m
        calls, busy, act = int(sel.sum()), int((e - s)[sel].sum()), int(active[sel].sum())
        out[m] = (calls * 1000 // R, busy * 1000 // act if act else 1000, calls, busy, act)
    return out.view(np.uint64)


def exact(case, seed):
    kind = case["kind"]
    if kind == "stats":
        return _exact_stats(case, seed)
    if kind in ("split", "pruned", "place"):
        return None                         # decisions, not sums: compared as they are
    batch, inst, G, ppm = _profiles(case, seed)
    Q, words = int(batch["space"]["Q"]), []
    for i, g, u in zip(inst, G, ppm):
        top = _tmax(_terms(batch, i, 1), Q * int(g))
        if kind == "tmax":
            words.append(top)
        else:
            words.append(_record(batch, _terms(batch, i, target_from_tmax(int(u), top)),
                                 Q * int(g)))
    if kind == "tmax":
        return np.asarray(words, dtype=np.uint32)
    words = np.concatenate(words)
    return torch.from_numpy(words.view(np.uint8)) if kind == "queue" else words
