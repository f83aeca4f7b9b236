"""The packed 16-bit scan against the knapsack DP and the masked scan, on an MI355X: option counts
around the tiles' remainders, the signed and unsigned 16-bit ranges to their ends and the first space
beyond them (which the masked scan keeps; the plan says which scan a space takes), two to eight LLMs, lanes' indices beyond 32 bits, and
launch overrides that take every work distribution (whole rows, tiles in turn, waves sharing a
tile by rows or records).  Integers throughout: results are equal, ties to the lowest index."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from dp_knapsack import dp_argmin
from workloads import make_custom, target_from_tmax

pytestmark = pytest.mark.gpu

TP4 = (1, 2, 4, 8)
Q4 = (1, 2, 3, 4)
# seed, M, tp, shares, D, frac_tp, G, instances, queries, launches (blocks, threads; 0 = automatic)
SPACES = [
    (201, 4, TP4, (1, 2, 4), 2, False, 12, 2, 4, [(0, 0), (1, 64), (5, 256), (24, 128), (9, 1024)]),
    (202, 3, (1, 2, 4, 8, 16), (4,), 13, False, 20, 2, 12, [(0, 0), (1, 64), (40, 512)]),   # O = 65
    (203, 3, (1, 2, 4), (1, 2, 4), 7, False, 12, 3, 9, [(0, 0), (3, 192), (64, 1024)]),     # O = 63
    (204, 3, TP4, Q4, 8, False, 16, 2, 64, [(0, 0), (2, 512), (7, 64)]),                    # O = 128
    (205, 3, (1, 2), (4,), 1, False, 4, 1, 3, [(0, 0)]),                                    # O = 2
    (206, 4, TP4, Q4, 11, False, 40, 1, 2, [(0, 0)]),             # (U + 1) S = 27,181: signed
    (207, 3, TP4, Q4, 12, False, 40, 2, 8, [(0, 0), (3, 256)]),   # 32,340: unsigned
    (208, 3, TP4, Q4, 16, False, 48, 2, 8, [(0, 0)]),             # 57,456: unsigned, O = 256
    (209, 3, TP4, Q4, 11, True, 40, 2, 8, [(0, 0)]),              # 62,128: unsigned
    (210, 3, TP4, Q4, 12, True, 40, 1, 8, [(0, 0)]),              # 73,920: masked
    (211, 2, TP4, (1, 2, 4), 16, False, 24, 3, 600, [(0, 0), (2, 128)]),                    # O = 192
    (212, 5, TP4, (2, 4), 3, False, 32, 2, 5, [(0, 0), (1, 64), (100, 256), (331, 1024)]),  # O = 24
    (213, 6, (1, 2), (2, 4), 3, False, 16, 1, 2, [(0, 0), (1, 448), (13, 128)]),            # O = 12
    (214, 8, (1, 2), (4,), 1, False, 12, 2, 2, [(0, 0), (1, 64), (11, 64)]),                # O = 2
    (215, 8, TP4, (2, 4), 3, False, 48, 1, 1, [(0, 0)]),          # 24^8: lanes' indices over 2^32
]


@pytest.fixture(scope="module")
def alp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_15186_amd import alp as binding
    binding.lib()
    return binding


def _queries(alp, ctx, b, instances, count, G):
    rng = np.random.default_rng([2604, 15186, 91, count, G])
    inst = (np.arange(count) % instances).astype(np.uint32)
    budget = rng.integers(0, G + 1, count).astype(np.uint32)
    budget[:instances] = G
    tmax = ctx.max_throughput(budget, instances=inst)
    u = rng.integers(1, 1_000_001, count)
    u[0] = 1_000_000
    lam = np.asarray([target_from_tmax(int(p), int(t)) for p, t in zip(u, tmax)], np.uint32)
    if count > 1:
        lam[-1] = tmax[-1] + 1                                   # infeasible
    return inst, budget, lam


def _check(alp, b, instances, count, G, launches, dp_queries=12):
    Q = int(b["space"]["Q"])
    with alp.Context(b) as ctx:
        inst, budget, lam = _queries(alp, ctx, b, instances, count, G)
        outs = []
        for blocks, threads in launches:
            ctx.set_launch(0, blocks, threads)
            outs.append(ctx.search_batch(budget, lam, instances=inst))
            assert outs[-1].tobytes() == outs[0].tobytes(), (blocks, threads)
            assert ctx.search_batch(budget, lam, instances=inst).tobytes() == outs[0].tobytes()
        if ctx.num_candidates < 1 << 34:
            ctx.set_launch(1)                                    # the masked scan
            assert ctx.search_batch(budget, lam, instances=inst).tobytes() == outs[0].tobytes()
        for k in sorted({int(v) for v in np.linspace(0, count - 1, min(count, dp_queries))}):
            o = oracle.Instance(b, int(inst[k]))
            terms = [[(t["ok"] and t["thr_ok"], t["c"], t["u"]) for t in row]
                     for row in oracle.option_terms(o, int(lam[k]))]
            want = dp_argmin(terms, Q * int(budget[k]))
            r = outs[0][k]
            if want is None:
                assert int(r["status"]) == alp.ALP_INFEASIBLE and int(r["index"]) == alp.NO_INDEX
            else:
                assert (int(r["index"]), int(r["latency_us"])) == want, (k, want)
                ev = oracle.evaluate(o, int(budget[k]), int(lam[k]), want[0])
                assert (int(r["throughput_milli"]), int(r["gpu_units"])) == (ev["T"], ev["U"])


@pytest.mark.parametrize("spec", SPACES, ids=[f"seed{s[0]}" for s in SPACES])
def test_matches_the_dp_and_the_masked_scan(alp, spec):
    seed, M, tps, fqs, D, frac_tp, G, instances, count, launches = spec
    b = make_custom(seed, M, tps, fqs, D, 5, G, count=instances, frac_tp=frac_tp,
                    deny_prob=0.0 if frac_tp else 0.05)
    _check(alp, b, instances, count, G, launches)


@pytest.mark.parametrize("seed,M,D", [(221, 4, 2), (222, 3, 8), (223, 5, 2)])
def test_equal_latencies_keep_the_lowest_index(alp, seed, M, D):
    """Every feasible candidate ties (equal terms share a rank): lane, wave, block and item ends
    all take the lowest index."""
    b = make_custom(seed, M, TP4, (1, 2, 4) if D == 2 else Q4, D, 1, 16, count=2)
    for m in range(M):
        b["lat"][:, m] = 1000 * (m + 1)
    b["n"][:] = 1000
    b["p"][:] = 1000
    _check(alp, b, 2, 10, 16, [(0, 0), (1, 64), (6, 256), (50, 1024)])


def test_device_queries_and_a_growing_batch(alp):
    """Queued batches with an out-of-range instance, one item in many blocks and then many items:
    the counters left by one launch serve the next."""
    import torch
    b = make_custom(231, 4, TP4, Q4, 4, 8, 24, count=3)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.uint32).view(np.int32)).cuda()  # noqa: E731
    with alp.Context(b) as ctx:
        inst, budget, lam = _queries(alp, ctx, b, 3, 40, 24)
        ref = ctx.search_batch(budget, lam, instances=inst)
        for n in (1, 40, 7, 1):
            bad = inst[:n].copy()
            bad[-1] = 3 if n > 1 else bad[-1]
            out = torch.zeros(n * alp.RESULT_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
            for _ in range(3):
                ctx.search_batch_async(dev(budget[:n]), dev(lam[:n]), out, instances=dev(bad))
            torch.cuda.synchronize()
            got = alp.results_from_device(out, n)
            last = n - 1 if n > 1 else n
            assert got[:last].tobytes() == ref[:last].tobytes()
            if n > 1:
                assert int(got[-1]["status"]) == alp.ALP_EINVAL


def _range(b):
    """(U + 1) S of the space's tables: S the most usable options of the last LLM, U the most units
    of any usable option in multiples of the shares' greatest common divisor."""
    sp = b["space"]
    tp, fq, Q, D = (sp["tp"].astype(np.int64), sp["fq"].astype(np.int64), int(sp["Q"]), int(sp["D"]))
    tpq = tp[:, None] * fq[None, :]
    fits = b["W"].astype(object)[:, :, None, None] * Q <= tpq.astype(object) * int(b["H"])
    usable = b["allowed"].astype(bool) & fits.astype(bool)
    S = int(usable[:, -1].sum(axis=(1, 2)).max()) * D
    U = int((usable * tpq).max()) * D // int(np.gcd.reduce(fq))
    return (max(U, 1) + 1) * max(S, 1)


@pytest.mark.parametrize("spec", SPACES, ids=[f"seed{s[0]}" for s in SPACES])
def test_the_plan_takes_the_scan_of_the_range(alp, spec):
    seed, M, tps, fqs, D, frac_tp, G, instances, count, launches = spec
    b = make_custom(seed, M, tps, fqs, D, 5, G, count=instances, frac_tp=frac_tp,
                    deny_prob=0.0 if frac_tp else 0.05)
    v = _range(b)
    with alp.Context(b) as ctx:
        for blocks, threads in launches:
            ctx.set_launch(0, blocks, threads)
            form = int(ctx.scan_plan(count)["form"])
            if M == 2 and len(tps) * len(fqs) * D <= 128:
                continue
            assert form == (alp.SCAN_PACKED if v < 0x7C00 else alp.SCAN_PACKED_WIDE) \
                if v <= 0xFFFF else form in (alp.SCAN_MASKED, alp.SCAN_MASKED_ONE_LAUNCH), v
        ctx.set_launch(1)
        assert int(ctx.scan_plan(count)["form"]) in (alp.SCAN_MASKED, alp.SCAN_MASKED_ONE_LAUNCH)


def test_both_distributions_occur(alp):
    seen = set()
    for seed, M, tps, fqs, D, frac_tp, G, instances, count, launches in SPACES:
        b = make_custom(seed, M, tps, fqs, D, 5, G, count=instances, frac_tp=frac_tp)
        with alp.Context(b) as ctx:
            for blocks, threads in launches:
                ctx.set_launch(0, blocks, threads)
                p = ctx.scan_plan(count)
                seen.add((int(p["form"]) >= alp.SCAN_PACKED, int(p["whole_rows"])))
    assert {(True, 0), (True, 1)} <= seen


# tensor parallel sizes, share units of 16, replicas, denied pairs of the last LLM, (U + 1) S
ENDS = [
    ((1, 2, 4), (1, 11), 12, 1, 31_740),                                         # signed
    ((1, 2, 3, 5, 8, 13, 21, 33), (1, 2, 4, 6, 9, 11, 13, 15), 1, 0, 31_744),    # unsigned, 0x7C00
    ((1, 2, 11), (1, 2, 3, 5, 7, 14), 5, 1, 65_535),                             # unsigned, the last
    ((1, 2, 3, 4, 5, 7, 11), (1, 2, 3, 4, 5), 6, 2, 65_538),                     # masked
]


@pytest.mark.parametrize("k", range(len(ENDS)))
def test_ends_of_the_ranges(alp, k):
    """Every option deployable but a few pairs of the last LLM, so that (U + 1) S is known; a budget
    that only the largest options together exceed, and smaller ones."""
    tps, fqs, D, denied, value = ENDS[k]
    G = 3 * max(tps) * max(fqs) * D // 16
    b = make_custom(241 + k, 3, tps, fqs, D, 5, G, count=2, frac_den=16, frac_tp=True)
    b["W"][:] = 1
    b["allowed"][:] = 1
    for i in range(denied):
        b["allowed"][:, -1, 0, i] = 0
    assert _range(b) == value
    want = alp.SCAN_PACKED if value < 0x7C00 else alp.SCAN_PACKED_WIDE
    with alp.Context(b) as ctx:
        form = int(ctx.scan_plan(16)["form"])
        assert form == want if value <= 0xFFFF else form < alp.SCAN_PACKED
    _check(alp, b, 2, 16, G, [(0, 0), (3, 192), (16, 1024)])


def test_a_large_batch_stays_within_a_launch(alp):
    """The plan's threads are below 2^32 (a launch's limit) for batches up to 2^25 searches."""
    for seed, M, tps, fqs, D in ((251, 3, (1, 2), (4,), 1), (252, 4, TP4, (2, 4), 2),
                                 (253, 3, (1, 2, 4, 8, 16), (2, 4), 13), (254, 5, (1, 2), (4,), 2),
                                 (255, 4, (1, 2, 4), (1, 2, 3, 4), 4)):
        b = make_custom(seed, M, tps, fqs, D, 5, 16, count=1)
        with alp.Context(b) as ctx:
            for count in (1 << 22, 4_300_000, 6_200_000, 1 << 23, 9_000_000, 1 << 24, 1 << 25):
                p = ctx.scan_plan(count)
                assert count * int(p["blocks_per_item"]) * int(p["threads_per_block"]) < 1 << 32, \
                    (seed, count, p)
