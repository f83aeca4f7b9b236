"""The pruned search's enumeration against the oracle at the edges of its tables and prefixes, on an
MI355X: option tables at and beyond what a block holds in LDS (with and without the ordering), one
share unit per GPU, one to eight LLMs, several blocks per item and many items in a batch."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from workloads import make_custom, target_from_tmax

pytestmark = pytest.mark.gpu

# seed, M, share units per GPU, budgets, flags
POINTS = [
    (301, 1, 4, (0, 3, 16), (0, 3)),
    (302, 2, 16, (128, 127, 1), (0, 1, 2, 3)),        # 2,048 units (the most): table in memory
    (303, 3, 8, (120, 7), (0, 3)),                    # 960 units: in memory
    (304, 3, 10, (82, 81), (1, 3)),                   # 820 units: the most a block holds in LDS
    (310, 3, 10, (83, 82), (1, 3)),                   # beyond
    (305, 4, 1, (40, 13, 3, 4), (0, 1, 2, 3)),        # one unit per GPU
    (306, 4, 16, (10, 1), (2, 3)),
    (307, 5, 3, (11, 5), (0, 1, 2, 3)),
    (308, 7, 2, (9, 3), (0, 3)),
    (309, 8, 2, (8,), (1, 3)),
    (311, 4, 16, (21, 5), (0, 1)),                    # 336 units: in memory, more blocks
    (312, 5, 16, (8,), (2,)),                         # 128 units: in memory without the ordering
]


@pytest.fixture(scope="module")
def alp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_15186_amd import alp as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("point", POINTS, ids=[f"seed{p[0]}" for p in POINTS])
def test_matches_the_oracle(alp, point):
    seed, M, Q, budgets, flag_sets = point
    fq = sorted({max(1, round(Q * k / 4)) for k in range(1, 5)})
    b = make_custom(seed, M, (1, 2, 4, 8), fq, 8, 4, max(budgets), count=2, frac_den=Q, alpha=0.7)
    inst = np.asarray([0, 1] * len(budgets), np.uint32)
    G = np.repeat(np.asarray(budgets, np.uint32), 2)
    objs = [oracle.Instance(b, 0), oracle.Instance(b, 1)]
    lam = [max(1, target_from_tmax(300_000, oracle.tmax(objs[i], int(g))) // (1 + k % 3))
           for k, (i, g) in enumerate(zip(inst, G))]
    with alp.Context(b) as ctx:
        for flags in flag_sets:
            want = [oracle.pruned(objs[i], int(g), int(v), flags) for i, g, v in zip(inst, G, lam)]
            for reps in (1, 40):                      # several blocks per item, then many items
                out = ctx.search_pruned(np.tile(G, reps), np.tile(lam, reps), flags,
                                        instances=np.tile(inst, reps))
                for k, r in enumerate(out):
                    w = want[k % len(want)]
                    got = (int(r["vectors"]), int(r["unpruned"]))
                    assert got == (w["vectors"], w["unpruned"]), (flags, k)
                    if w["x"] is None:
                        assert int(r["best"]["status"]) == alp.ALP_INFEASIBLE
                    else:
                        assert (int(r["best"]["index"]), int(r["best"]["latency_us"])) == \
                            (w["x"], w["L"]), (flags, k)


def test_more_queries_than_a_launch_of_whole_blocks_holds(alp):
    """2^23 queries: 512 threads for each would be 2^32, more than a launch holds."""
    b = make_custom(321, 1, (1, 2), (2, 4), 2, 4, 8, count=2, alpha=0.7)
    count, period = 1 << 23, 1 << 10
    G = (np.arange(period) % 9).astype(np.uint32)
    inst = (np.arange(period) % 2).astype(np.uint32)
    lam = np.full(period, 100, np.uint32)
    with alp.Context(b) as ctx:
        want = ctx.search_pruned(G, lam, 3, instances=inst)
        rep = count // period
        got = ctx.search_pruned(np.tile(G, rep), np.tile(lam, rep), 3, instances=np.tile(inst, rep))
        assert (got.reshape(rep, period) == want).all()
        w = oracle.pruned(oracle.Instance(b, 1), 3, 100, 3)
        assert (int(want[3]["best"]["index"]), int(want[3]["vectors"])) == \
            (alp.NO_INDEX if w["x"] is None else w["x"], w["vectors"])


def test_the_table_time_is_that_of_tables_in_memory(alp):
    """820 ordered units are the most a block holds in LDS: no table kernel, and no time for one."""
    b = make_custom(331, 3, (1, 2, 4, 8), (2, 5, 10), 8, 4, 83, count=1, frac_den=10, alpha=0.7)
    with alp.Context(b) as ctx:
        ctx.set_timing(1)
        for G, in_memory in ((82, False), (83, True), (82, False)):
            ctx.search_pruned(np.asarray([G], np.uint32), np.asarray([10], np.uint32), 1,
                              instances=np.asarray([0], np.uint32))
            terms, enumeration, table, _ = ctx.kernel_times()
            assert terms > 0 and enumeration > 0 and (table > 0) == in_memory
