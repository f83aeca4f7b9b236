"""Largest reachable throughput against the oracle at the edges of the kernel's waves and LDS, on an
MI355X: one to eight LLMs (odd and even), fewer and more options than a wave has lanes, as many as
leave one wave to a block, budgets where nothing fits, and items that do not fill the last block."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from workloads import make_custom

pytestmark = pytest.mark.gpu

# seed, M, tensor parallel sizes, share units (of 16 per GPU), replicas
POINTS = [
    (401, 1, (1,), (16,), 1),                                          # one option
    (402, 2, (1, 2, 4, 8), (4, 8, 12, 16), 4),                         # 64: one per lane
    (403, 3, (1, 2, 4, 8, 16), (4, 8, 16), 13),                        # 195
    (404, 4, (1, 2, 4, 8, 16, 32, 64), (1, 5, 16), 3),                  # 63
    (405, 5, (1, 2, 4, 8), (2, 4, 6, 8, 10, 12, 14, 16), 16),          # 512, the most
    (406, 7, (1, 2, 4, 8), (2, 4, 6, 8, 10, 12, 16), 16),              # 448: one wave to a block
    (407, 8, (1, 2, 4), (1, 8, 16), 16),                               # 144
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
    seed, M, tps, fqs, D = point
    b = make_custom(seed, M, tps, fqs, D, 4, 64, count=3, frac_den=16, alpha=0.7)
    G = np.asarray([0, 1, 3, 16, 64, 1024, 2000], np.uint32)
    inst = np.resize(np.asarray([0, 1, 2], np.uint32), len(G))
    want = [oracle.tmax(oracle.Instance(b, int(i)), int(g)) for i, g in zip(inst, G)]
    with alp.Context(b) as ctx:
        for reps in (1, 37):
            got = ctx.max_throughput(np.tile(G, reps), instances=np.tile(inst, reps))
            assert np.array_equal(np.asarray(got, np.uint64), np.tile(np.asarray(want, np.uint64), reps))


def test_results_take_four_bytes_an_item(alp, monkeypatch):
    """A context that has returned 3,000 search records (48 bytes each) holds a result buffer for
    36,000 throughputs: with the queries' buffers there, no allocation is needed."""
    b = make_custom(411, 2, (1, 2), (2, 4), 2, 4, 8, count=1)
    G = (np.arange(36_000) % 9).astype(np.uint32)
    inst = np.zeros(36_000, np.uint32)
    with alp.Context(b) as ctx:
        want = np.tile(ctx.max_throughput(G[:9], instances=inst[:9]), 4_000)
        ctx.search_batch(G[:3_000], np.ones(3_000, np.uint32), instances=inst[:3_000])
        ctx.search_pruned(G, np.ones(36_000, np.uint32), instances=inst)
        monkeypatch.setenv("ALP_TEST_FAIL_ALLOC", "1")
        assert ctx.max_throughput(G, instances=inst).tolist() == want.tolist()


def test_searches_after_throughputs_pin_no_more_memory(alp, monkeypatch):
    """The throughputs that set a search's target and the searches that follow share one buffer."""
    b = make_custom(412, 2, (1, 2), (2, 4), 2, 4, 8, count=1)
    G = np.full(1_000, 8, np.uint32)
    inst = np.zeros(1_000, np.uint32)
    with alp.Context(b) as other:
        want = other.search_batch(G, np.ones(1_000, np.uint32), instances=inst)
    with alp.Context(b) as ctx:
        ctx.max_throughput(G, instances=inst)
        out = ctx.search_pruned(G, np.ones(1_000, np.uint32), instances=inst)   # device buffers
        assert len(out) == 1_000
        one = ctx.search(0, 8, 1)
        assert one.tobytes() == want[0].tobytes()
        monkeypatch.setenv("ALP_TEST_FAIL_ALLOC", "1")
        assert ctx.search(0, 8, 1).tobytes() == want[0].tobytes()
        try:
            got = ctx.search_batch(G, np.ones(1_000, np.uint32), instances=inst)
        except alp.AlpError as err:                   # the scan's own device buffers only
            assert err.status == alp.ALP_ENOMEM and "results" not in str(err)
        else:
            assert got.tobytes() == want.tobytes()
