"""The statistics' launch sequences on one context, on an MI355X: the sweep, the switch to the direct
sort and back, long traces found by the kernels and then expected, traces longer than the last
direct call's, and offsets that only the kernels see.  Every result equals the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from workloads.traces import make_traces

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def alp():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_15186_amd import alp as binding
    binding.lib()
    return binding


def _shuffle(tr, seed):
    rng = np.random.default_rng(seed)
    off = tr["offsets"].astype(np.int64)
    perm = np.concatenate([lo + rng.permutation(hi - lo) for lo, hi in zip(off[:-1], off[1:])])
    return {**tr, **{k: tr[k][perm] for k in ("llm", "start", "end")}}


def _joined(tr, per):
    """The traces joined `per` at a time (longer traces of the same calls)."""
    return {**tr, "offsets": np.append(tr["offsets"][:-1:per], tr["offsets"][-1:])}


def _same(ctx, tr):
    args = (tr["M"], tr["offsets"], tr["llm"], tr["start"], tr["end"])
    got, want = ctx.compute(*args), oracle.trace_stats(*args)
    for f in want.dtype.names:
        assert [int(v) for v in got[f]] == [int(v) for v in want[f]], f


def _one_start(tr):
    """Every trace moved to the same start, so that joined traces span a few minutes."""
    off = tr["offsets"].astype(np.int64)
    first = np.repeat(np.minimum.reduceat(tr["start"], off[:-1]), np.diff(off))
    return {**tr, "start": tr["start"] - first, "end": tr["end"] - first}


@pytest.mark.parametrize("shape,R,per", [("rag", 700, 40), ("beam", 90, 1), ("beam", 200, 3)])
def test_one_context_takes_every_path(alp, shape, R, per):
    logged = make_traces(shape, R, 31)
    mixed = _shuffle(logged, 1)
    longer = _shuffle(_joined(_one_start(logged), per), 2)   # beam, 3 at a time: some beyond 2,048
    with alp.StatsContext(0) as ctx:
        for tr in (logged, mixed, mixed, longer, mixed, longer, longer, logged, logged, mixed,
                   longer, logged, longer):
            _same(ctx, tr)


@pytest.mark.parametrize("offsets", [[0, 100, 10], [0, 4, 3, 10], [5, 10], [0, 12, 11, 10],
                                     [3, 2, 1], [0, 5, (1 << 63), 10]])
def test_bad_offsets_are_refused_and_leave_the_context_working(alp, offsets):
    """The call arrays hold offsets[-1] entries."""
    good = make_traces("rag", 50, 3)
    calls = int(offsets[-1])
    rng = np.random.default_rng(4)
    start = rng.integers(0, 1000, calls).astype(np.uint64)
    bad = (3, np.asarray(offsets, np.uint64), np.zeros(calls, np.uint32), start, start + 5)
    with alp.StatsContext(0) as ctx:
        for order in (good, _shuffle(good, 5)):           # from the sweep, then the direct sort
            for _ in range(2):
                _same(ctx, order)
            for _ in range(2):
                with pytest.raises(alp.AlpError) as err:
                    ctx.compute(*bad)
                long = offsets[1] + (1 << 24) < offsets[2] if len(offsets) > 3 else False
                assert err.value.status == (alp.ALP_ERANGE if long else alp.ALP_EINVAL)
            _same(ctx, order)


@pytest.mark.parametrize("sized", [True, False], ids=["sized", "unsized"])
@pytest.mark.parametrize("offsets", [[0, 10, 5, 1000], [0, 1000], [0, 3, 11, 11], [4, 1000, 2, 9]])
def test_offsets_beyond_the_call_arrays_are_refused(alp, offsets, sized):
    """Lists whose last (or any) offset lies beyond the arrays' ten calls.  The arrays are the front
    of longer ones, whose further calls belong to an LLM out of range: a call read there would be
    one more reason for EINVAL, never a fault.  Without the arrays' length only a malformed list
    can be refused, and only before anything is read."""
    import torch
    good = make_traces("rag", 50, 3)
    off = torch.tensor(offsets, dtype=torch.int64, device="cuda")
    llm = torch.full((2000,), 7, dtype=torch.int32, device="cuda")
    llm[:10] = 0
    start = torch.arange(2000, dtype=torch.int64, device="cuda")
    end = start + 5
    with alp.StatsContext(0) as ctx:
        for order in (good, _shuffle(good, 5)):           # from the sweep, then the direct sort
            for _ in range(2):
                _same(ctx, order)
            if sized:
                with pytest.raises(alp.AlpError) as err:
                    ctx.compute(1, off, llm[:10], start[:10], end[:10])
                assert err.value.status == alp.ALP_EINVAL
                assert "offset" in str(err.value)
            elif offsets != sorted(offsets) or offsets[0]:
                out = np.zeros(1, alp.STATS_DTYPE)
                st = alp.lib().alp_trace_stats(ctx._ctx, 1, len(offsets) - 1, off.data_ptr(),
                                               llm.data_ptr(), start.data_ptr(), end.data_ptr(),
                                               out.ctypes.data)
                assert st == alp.ALP_EINVAL and "offsets" in alp.last_error()
            _same(ctx, order)


def test_without_the_arrays_length_the_result_is_the_same(alp):
    """alp_trace_stats and alp_trace_stats_sized agree, call by call, on one context each."""
    import torch
    logged = make_traces("beam", 60, 8)
    longer = _joined(_one_start(logged), 4)
    with alp.StatsContext(0) as a, alp.StatsContext(0) as b:
        for tr in (logged, _shuffle(logged, 1), longer, _shuffle(longer, 2), logged):
            dev = [torch.from_numpy(np.ascontiguousarray(tr[k], t).view(s)).cuda() for k, t, s in
                   (("offsets", np.uint64, np.int64), ("llm", np.uint32, np.int32),
                    ("start", np.uint64, np.int64), ("end", np.uint64, np.int64))]
            out = np.zeros(tr["M"], alp.STATS_DTYPE)
            st = alp.lib().alp_trace_stats(a._ctx, tr["M"], len(tr["offsets"]) - 1,
                                           *(t.data_ptr() for t in dev), out.ctypes.data)
            assert st == alp.ALP_OK
            assert out.tobytes() == b.compute(tr["M"], *dev).tobytes()
            _same(a, tr)


@pytest.mark.parametrize("R", [1 << 24, 3 << 23])
def test_more_traces_than_a_launch_holds_threads_for(alp, R):
    """2^24 traces and more (256 threads for each would be 2^32 or more) out of end order, the
    longest of 1,030 calls: 1,024 copies and more of the same traces, so the sums are multiples of
    the oracle's and n and p the same."""
    import torch
    T = 1 << 13
    rng = np.random.default_rng(2 ** 24)
    n = rng.integers(2, 4, T)                             # out of end order: sorted directly
    n[5], n[77], n[1234] = 1030, 600, 0
    off = np.concatenate([[0], np.cumsum(n)]).astype(np.int64)
    calls = int(off[-1])
    end = np.empty(calls, np.int64)
    for lo, hi in zip(off[:-1], off[1:]):
        end[lo:hi] = np.sort(rng.integers(100_000, 1 << 27, hi - lo))[::-1]
    start = end - rng.integers(1, 100_000, calls)
    llm = rng.integers(0, 2, calls).astype(np.int32)
    want = oracle.trace_stats(2, off.astype(np.uint64), llm.astype(np.uint32),
                              start.astype(np.uint64), end.astype(np.uint64))
    K = R // T
    base = torch.arange(K, dtype=torch.int64, device="cuda").repeat_interleave(T) * calls
    offsets = torch.empty(R + 1, dtype=torch.int64, device="cuda")
    offsets[:R] = base + torch.from_numpy(off[:-1]).cuda().repeat(K)
    offsets[R] = K * calls
    dev = [torch.from_numpy(v).cuda().repeat(K) for v in (llm, start, end)]
    with alp.StatsContext(0) as ctx:
        for _ in range(3):                                # the sweep, then the direct sort
            got = ctx.compute(2, offsets, *dev)
            for f in ("calls", "busy_us", "active_us"):
                assert [int(v) for v in got[f]] == [K * int(v) for v in want[f]], f
            for f in ("n_milli", "p_milli"):
                assert got[f].tolist() == want[f].tolist(), f


def test_the_time_is_the_kernels_alone(alp):
    """A context that expects long traces reads the offsets first: four million of them on the
    host take many times the kernels' time, and none of that is in it."""
    import time

    import torch
    R = 1 << 22
    dev = [torch.zeros(n, dtype=t, device="cuda") for n, t in
           ((R + 1, torch.int64), (3000, torch.int32), (3000, torch.int64), (3000, torch.int64))]
    dev[0][R // 2:] = 3000                                # one long trace, the others empty
    dev[3] += torch.arange(3000, device="cuda")
    with alp.StatsContext(0) as ctx:
        ctx.set_timing(True)
        ctx.compute(1, *dev)                              # finds the long trace: two launches
        kernels, call = [], []
        for _ in range(3):
            t = time.perf_counter()
            ctx.compute(1, *dev)
            call.append(1e3 * (time.perf_counter() - t))
            kernels.append(ctx.time_ms())
        assert 0 < min(kernels) < 0.5 * min(call), (kernels, call)
        dev[0][R // 2:] = 2000                            # none is long any more, nor in order
        ctx.compute(1, *dev)
        ctx.compute(1, *dev)
        assert 0 < ctx.time_ms() < min(call)


def test_a_context_goes_back_to_the_sweep_on_sparse_traces_in_order(alp):
    """Three empty traces beside every logged one, after shuffled traces: the context that sorts
    directly finds most in order and sweeps again, as a new context does from its first call."""
    logged = make_traces("beam", 3000, 7)
    sparse = {**logged, "offsets": np.repeat(logged["offsets"], [4] * 3000 + [1])}

    def kernel_ms(ctx):
        ms = []
        for _ in range(6):
            _same(ctx, sparse)
            ms.append(ctx.time_ms())
        return min(ms)

    with alp.StatsContext(0) as new, alp.StatsContext(0) as used:
        for ctx in (new, used):
            ctx.set_timing(True)
        for _ in range(2):
            _same(used, _shuffle(logged, 1))
        want, got = kernel_ms(new), kernel_ms(used)
        assert got < 1.5 * want, (got, want)          # a call: 36 us swept, 112 sorted


def test_the_first_direct_sort_launches_only_the_groups_it_needs(alp):
    """2^22 traces of two calls, the later one logged first: the call after the sweep takes no
    longer than the next one (a launch of groups for traces that are not there takes milliseconds)."""
    import torch
    R = 1 << 22
    offsets = 2 * torch.arange(R + 1, dtype=torch.int64, device="cuda")
    llm = torch.zeros(2 * R, dtype=torch.int32, device="cuda")
    start = torch.tensor([500, 100], dtype=torch.int64, device="cuda").repeat(R)
    with alp.StatsContext(0) as warm:                     # every kernel loaded
        for _ in range(3):
            warm.compute(1, offsets, llm, start, start + 50)
    ms = []
    with alp.StatsContext(0) as ctx:
        ctx.set_timing(True)
        for _ in range(4):
            got = ctx.compute(1, offsets, llm, start, start + 50)
            ms.append(ctx.time_ms())
            assert [int(v) for v in got[0]] == [2000, 1000, 2 * R, 100 * R, 100 * R]
    assert ms[1] < 2 * min(ms[2:]), ms                    # 4.9 and 1.8 ms with every group launched
