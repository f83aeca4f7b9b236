"""Placements of spaces whose replicas fill part of a record's 128 slots, all of them, or end
inside a lane's share: every slot against the oracle, those past the replicas "not placed"."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from workloads import make_custom

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def alp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_15186_amd import alp as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("M,D", [(1, 1), (1, 8), (1, 9), (3, 5), (4, 16), (5, 13), (8, 16)])
def test_every_slot(alp, M, D):
    rng = np.random.default_rng([M, D])
    b = make_custom(70 + M, M, (1, 2), (1, 4), D, 1, 8, count=1, frac_den=4)
    count = 300
    tp = rng.choice([1, 2], (count, M))
    q = rng.choice([1, 4], (count, M))
    d = rng.integers(1, D + 1, (count, M))
    d[::7] = D                                          # the space's most replicas
    G = rng.choice([1, 8, 15, 16, 17, 40, 64], count).astype(np.uint32)
    with alp.Context(b) as ctx:
        for n in (count, 5, count):                     # a call after a larger and a smaller one
            res = np.zeros(n, dtype=alp.RESULT_DTYPE)
            res["tp"][:, :M], res["frac_units"][:, :M], res["replicas"][:, :M] = \
                tp[:n], q[:n], d[:n]
            out = ctx.place(res, G[:n])
            for i in range(n):
                a = [[int(v) for v in x[i]] for x in (tp, q, d)]
                want = oracle.place(4, int(G[i]), *a)
                got = out[i]
                k = sum(a[2])
                assert (int(got["status"]) == 0) == want["placed"]
                assert (int(got["replicas"]), int(got["gpus_used"]), int(got["nodes_used"])) == \
                    (want["replicas"], want["gpus_used"], want["nodes_used"])
                assert [int(v) for v in got["slot"][:k]] == want["slot"]
                assert (got["slot"][k:] == 0xFFFF).all()
