"""nb_sync reports calls of one context that overlapped on the device, also
when their launches are too small to touch the work queue's counters: the first
kernel of a call that shares memory of the context with its last one steps the
queue's in-flight word, the last one steps it back."""
import itertools
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _overlapped_value():
    src = open(os.path.join(ROOT, "paper_1409_5474_amd", "csrc", "work_queue.h")).read()
    return int(re.search(r"kOverlapped = (0x[0-9a-f]+)u", src).group(1), 16)


def _final(events, limit):
    """The word after a sequence of first steps (+1) and steps back (-1), by the wrapping
    increment (old >= 1 ? 0 : old + 1) and decrement (old == 0 or old > limit ?
    limit : old - 1)."""
    x = 0
    for e in events:
        if e > 0:
            x = 0 if x >= 1 else x + 1
        else:
            x = limit if x == 0 or x > limit else x - 1
    return x


def _sequences(n):
    """All orders of n starts and n ends in which no end comes before its start."""
    for at in itertools.combinations(range(2 * n), n):
        ev = [-1] * (2 * n)
        for a in at:
            ev[a] = 1
        if min(np.cumsum(ev)) >= 0:
            yield ev


def test_in_flight_word_is_zero_exactly_when_no_launches_overlapped():
    limit = _overlapped_value()
    for n in range(1, 8):
        for ev in _sequences(n):
            apart = max(np.cumsum(ev)) == 1
            assert (_final(ev, limit) == 0) == apart, ev


def test_in_flight_word_stays_set_through_later_launches():
    limit = _overlapped_value()
    rng = np.random.default_rng(1)
    for ev in _sequences(4):
        if max(np.cumsum(ev)) > 1:
            for later in (1, 2, 3, int(rng.integers(4, 500))):
                assert _final(ev + [1, -1] * later, limit) != 0, (ev, later)


@pytest.fixture(scope="module")
def streams():
    # one pair for the module: a process has four hardware queues, and streams
    # beyond them share one
    import torch
    return [torch.cuda.Stream(), torch.cuda.Stream()]


@pytest.mark.gpu
@pytest.mark.parametrize("second", ["devcount", "small_step"])
def test_sync_reports_overlapping_calls_without_queue_counters(streams, second):
    # a launch of one workgroup and some milliseconds on one stream, and on
    # another the same or a small system's block step.  The two launches share
    # only the slot that holds their split (one for both), so the results are
    # right and only the report shows the overlap; the block step shares
    # nothing, and there is nothing to report.
    import torch
    import paper_1409_5474_amd as nb
    import synth
    from paper_1409_5474_amd.integrator import BlockIntegrator
    c = nb.Context(0, "fp64", load_tuning=False)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    n, k = 262144, 256
    c.tune_add("fp64", n, 0, 2 ** 31 - 1, 1, 1, 1)  # one work item: one workgroup, no j-split
    p, q = synth.plummer(n, 2), synth.plummer(500, 3)
    P, V, M, act = t(p.pos), t(p.vel), t(p.mass), t(np.arange(k, dtype=np.int32))
    cnt = torch.tensor([k], dtype=torch.int32, device="cuda")
    outs = [[torch.zeros((k, 3), dtype=torch.float64, device="cuda"),
             torch.zeros((k, 3), dtype=torch.float64, device="cuda"),
             torch.zeros(k, dtype=torch.float64, device="cuda")] for _ in range(2)]
    bi = BlockIntegrator(c, t(q.pos), t(q.vel), t(q.mass), 1e-3)
    start = [getattr(bi, a).clone() for a in ("pos", "vel", "acc", "jerk", "t_tick", "level", "sched")]

    def first():
        c.forces_devcount(P, V, M, act, cnt, k, 1e-3, *outs[0])

    def other():
        if second == "devcount":
            c.forces_devcount(P, V, M, act, cnt, k, 1e-3, *outs[1])
        else:
            bi.step()

    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(2)]

    def go(apart):
        for a, x in zip(("pos", "vel", "acc", "jerk", "t_tick", "level", "sched"), start):
            getattr(bi, a).copy_(x)
        torch.cuda.synchronize()
        for s, e, f in zip(streams, ev, (first, other)):
            c.set_stream(s)
            e[0].record(s)
            with torch.cuda.stream(s):
                f()
            e[1].record(s)
            if apart:
                torch.cuda.synchronize()
        torch.cuda.synchronize()
        return [x.clone() for x in outs[0] + outs[1] + [bi.pos, bi.vel, bi.t_tick, bi.level, bi.sched]]

    ref = go(apart=True)
    c.sync()
    got = go(apart=False)
    for a, b in zip(ref, got):
        assert torch.equal(a, b)
    if not ev[0][0].elapsed_time(ev[1][1]) < ev[0][0].elapsed_time(ev[0][1]) + 0.5 * ev[1][0].elapsed_time(ev[1][1]):
        c.close()
        pytest.skip("the two streams ran one after the other here")
    if second == "devcount":
        with pytest.raises(nb.NbodyError, match="overlapped"):
            c.sync()
    c.sync()
    # reported once; later calls, one after another, are clean
    go(apart=True)
    c.sync()
    c.close()
