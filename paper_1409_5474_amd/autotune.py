"""Autotuner for the force kernel's launch shape.

For each precision and each active-set bucket it times every built
(K, L) shape over a range of j-subset counts S with ``nb_time_forces`` (HIP
events on the context stream); a second stage times the two fastest shapes
with every other j-tile length T and workgroup size WG built for them.  The
winner is stored as a table entry (K, L, T, WG, work-item target = S x
i-blocks) covering the active counts between the geometric midpoints of
neighbouring buckets; the library derives S from that target with the
paper's saturation rule, identically for host-count and device-count
launches.  ``tune_batch_forces`` and ``tune_batch_steps`` tune the batched
kernel (the latter inside graph-replayed block steps).

A block step launches one kernel per distinct shape of the table (each
returns at once unless the device-held count falls in its range), so every
shape run costs about one empty launch in every step.  After the sweep, a
run of buckets takes a neighbouring run's shape when that costs it at most
``launch_ms`` at each of its buckets: a step's count falls in one bucket, so
the switch loses at most that much in a step and always saves one launch.
A single bucket likewise takes another shape when that alone saves a launch
(e.g. a shape of one kernel family where its fastest keeps two families
apart).

    python -m paper_1409_5474_amd.autotune --n 65536 262144 --out tuning.json

``--rounds`` (``tune_rounds``) instead times every range of active counts on
two systems with whole numbers of work items per compute unit; the shipped
table's entries with ``rep_n`` come from it.

Entries tuned on up to 4096 particles hold for such systems only where they
beat the library's small-system launch at every bucket; otherwise they start
at N = 4097.

``load(ctx, path)`` installs a saved table into a context.
"""
import argparse
import json
import math
import os
import sys
import time
import warnings

import numpy as np
import torch

# (K, L); L = 0 is the scalar j-path (i-parallel, j-records through the scalar cache)
SHAPES = [(1, 1), (1, 4), (1, 16), (1, 64), (1, 256), (2, 1), (2, 4), (2, 16), (4, 1), (4, 4), (1, 0), (2, 0), (3, 0), (4, 0)]
BUCKETS = [1, 8, 64, 256, 1024, 4096, 16384, 65536, 262144]
DEFAULT_TABLE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "tuning_gfx950.json")
TILE, WG = 256, 256
# Up to this many particles a system without a table entry takes one launch of
# its own (the library's kSmallDirect), which no (K, L) names: any entry that
# holds for such a system switches it off for every active count.
SMALL_SYSTEM = 4096
# Second stage: the j-tile length T and workgroup size WG the library builds
# besides (256, 256), per (K, L) (see nb_set_launch).
TILE_WG = {(1, 1): [(128, 256), (128, 128), (64, 64)], (1, 4): [(128, 256), (128, 128), (64, 64)],
           (1, 16): [(128, 256), (128, 128), (64, 64)], (2, 1): [(128, 256), (128, 128), (64, 64)],
           (2, 4): [(128, 256), (128, 128), (64, 64)], (1, 0): [(256, 128)], (2, 0): [(256, 128)]}


# j-split counts tried: every S up to 8, then steps of about a quarter.  The
# time is not monotone in S (items are handed out from a queue, and how the
# last items fall across the compute units matters), so powers of two alone
# miss good values.
_S_STEPS = [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 128, 160, 192, 256]


def _s_candidates(n, n_act, K, L, num_cus, tile=TILE, wg=WG):
    ib = (wg // max(L, 1)) * K
    n_iblk = -(-n_act // ib)
    max_s = -(-n // tile)
    out = {0}
    for s in _S_STEPS:
        if s > max_s or n_iblk * s > 32 * num_cus:
            break
        out.add(s)
    return sorted(out), n_iblk


def _full(sh):
    """(K, L) or (K, L, T, WG) -> (K, L, T, WG)."""
    return tuple(sh) if len(sh) == 4 else (sh[0], sh[1], TILE, WG)


def _shape_str(sh):
    K, L, tl, wg = _full(sh)
    return f"K={K} L={L} T={tl} WG={wg}"


def _midpoints(buckets):
    lo = [0]
    for a, b in zip(buckets[:-1], buckets[1:]):
        lo.append(int(math.floor(math.sqrt(a * b))) + 1)
    hi = [x - 1 for x in lo[1:]] + [2 ** 31 - 1]
    return list(zip(lo, hi))


# cost of one empty force launch in a graph-replayed block step (measured
# 3.5-5 us per launch on MI355X; the smaller figure keeps the merge safe)
LAUNCH_MS = 0.003


def _family(sh):
    """The library's family_of: the LDS kernel family holding a shape (0: none)."""
    K, L, tl, wg = _full(sh)
    if tl != TILE or wg != WG or L < 1:
        return 0
    if K == 1 and L in (1, 4, 16, 64, 256):
        return 1
    if K == 2 and L in (1, 4, 16):
        return 2
    if K == 4 and L == 4:
        return 4
    return 0


def _cover(a, b):
    """The library's family_cover."""
    if not a or not b:
        return 0
    if a == b or b == 1:
        return a
    if a == 1:
        return b
    return 0


def _launch_runs(choice):
    """Runs of buckets that share one device-count launch: the same shape, or
    shapes one kernel family holds.  Returns [(family or None, [buckets])]."""
    runs = []
    for b, sh in enumerate(choice):
        if runs:
            fam, bs = runs[-1]
            if choice[bs[-1]] == sh and fam is None:
                bs.append(b)
                continue
            joint = _cover(fam if fam else _family(choice[bs[-1]]), _family(sh))
            if joint:
                runs[-1] = (joint, bs + [b])
                continue
        runs.append((None, [b]))
    return runs


def _merge_buckets(choice, times, launch_ms):
    """One bucket at a time: a bucket takes another of its timed shapes when
    that lowers the number of launch runs at a cost of at most launch_ms
    (the cheapest such change first, repeated until none fits) -- e.g. the
    one bucket whose shape keeps two kernel families from sharing a launch."""
    choice = list(choice)
    while True:
        n_runs = len(_launch_runs(choice))
        best = None
        for b, t in enumerate(times):
            for sh, ms in t.items():
                pen = ms - t[choice[b]]
                if sh == choice[b] or pen > launch_ms or (best is not None and pen >= best[0]):
                    continue
                if len(_launch_runs(choice[:b] + [sh] + choice[b + 1:])) < n_runs:
                    best = (pen, b, sh)
        if best is None:
            return choice
        choice[best[1]] = best[2]


def _merge_shapes(choice, times, launch_ms):
    """choice[b]: the shape of bucket b; times[b]: {shape: best ms}.  Returns
    the choice after merging launch runs into neighbours (see module doc): a
    run whose buckets all take the shape of the neighbouring run's nearest
    bucket at a cost of at most launch_ms each saves one launch per step;
    then single buckets as in _merge_buckets, and again until neither
    changes anything.  Every change saves a launch and costs a bucket at
    most launch_ms, so no bucket loses more than the launches saved."""
    while True:
        merged = _merge_runs(choice, times, launch_ms)
        merged = _merge_buckets(merged, times, launch_ms)
        if merged == list(choice):
            return merged
        choice = merged


def _merge_runs(choice, times, launch_ms):
    choice = list(choice)
    while True:
        runs = _launch_runs(choice)
        best = None
        for r, (_, bs) in enumerate(runs):
            for q in (r - 1, r + 1):
                if not 0 <= q < len(runs):
                    continue
                other = choice[runs[q][1][-1] if q < r else runs[q][1][0]]
                if not all(other in times[b] for b in bs):
                    continue
                pen = max(times[b][other] - times[b][choice[b]] for b in bs)
                if pen <= launch_ms and (best is None or pen < best[0]):
                    best = (pen, bs, other)
        if best is None:
            return choice
        for b in best[1]:
            choice[b] = best[2]


def _graph_ms(ctx, call, calls=20, replays=8):
    """Milliseconds of one call, replayed back to back from a graph (short
    launches issued one by one are timed at the host's rate)."""
    call()
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx.set_stream(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        for _ in range(calls):
            call()
    best = math.inf
    for _ in range(replays):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        with torch.cuda.stream(stream):
            graph.replay()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) * 1e3 / calls)
    ctx.set_stream(None)
    return best


def _small_n_min(n, default_ms, shape_ms):
    """The smallest N that entries tuned on n <= SMALL_SYSTEM particles should
    hold for: n when their shapes beat the small-system launch at every bucket,
    else the first N that does not take it."""
    return n if all(s < d for d, s in zip(default_ms, shape_ms)) else SMALL_SYSTEM + 1


def tune(ctx, n, precisions=("fp64", "mixed", "mixed_ds"), buckets=BUCKETS, seed=2, reps=3, log=print,
         launch_ms=LAUNCH_MS):
    import synth
    dev = ctx.device
    p = synth.plummer(n, seed)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    P, V, M = t(p.pos), t(p.vel), t(p.mass)
    eps2 = 2.0 ** -16
    num_cus = torch.cuda.get_device_properties(dev).multi_processor_count
    bks = [b for b in buckets if b <= n]
    ranges = _midpoints(bks)
    entries = []
    for prec in precisions:
        ctx.set_precision(prec)
        times, best_of = [], []
        for b in bks:
            act = torch.from_numpy(np.linspace(0, n - 1, b).astype(np.int32)).to(dev)
            acc = torch.empty((b, 3), dtype=torch.float64, device=dev)
            jerk = torch.empty_like(acc)
            pot = torch.empty(b, dtype=torch.float64, device=dev)
            per_shape = {}
            for K, L in SHAPES:
                if K > 1 and b < 64 * K:
                    continue
                svals, n_iblk = _s_candidates(n, b, K, L, num_cus)
                for S in svals:
                    r = reps if b * n < 2 ** 32 else max(1, reps - 1)
                    ms = ctx.time_forces(K, L, S, P, V, M, act, eps2, acc, jerk, pot, reps=r)
                    if (K, L) not in per_shape or ms < per_shape[(K, L)][0]:
                        per_shape[(K, L)] = (ms, S, n_iblk)
            # second stage: the two fastest shapes with every other (T, WG)
            # built for them, at j-splits around their best (scaled to keep
            # the work-item count)
            base = sorted(per_shape.items(), key=lambda kv: kv[1][0])[:2]
            for (K, L), (ms0, S0, _) in base:
                for tl, wg in TILE_WG.get((K, L), []):
                    svals, n_iblk = _s_candidates(n, b, K, L, num_cus, tl, wg)
                    ib0 = (WG // max(L, 1)) * K
                    ib = (wg // max(L, 1)) * K
                    centre = max(1, round(S0 * (-(-b // ib0)) / max(1, -(-b // ib)))) if S0 else 0
                    near = sorted({0} | {v for v in svals if centre and centre / 2 <= v <= centre * 2})
                    for S in near:
                        ms = ctx.time_forces(K, L, S, P, V, M, act, eps2, acc, jerk, pot, reps=reps, T=tl, WG=wg)
                        key = (K, L, tl, wg)
                        if key not in per_shape or ms < per_shape[key][0]:
                            per_shape[key] = (ms, S, n_iblk)
            times.append({sh: v[0] for sh, v in per_shape.items()})
            best_of.append(per_shape)
            sh, v = min(per_shape.items(), key=lambda kv: kv[1][0])
            log(f"# {prec} N={n} n_active={b}: fastest {_shape_str(sh)} S={v[1]} {v[0]:.5f} ms")
        fastest = [min(t, key=t.get) for t in times]
        choice = _merge_shapes(fastest, times, launch_ms)
        n_min = n
        if n <= SMALL_SYSTEM:
            plain = type(ctx)(dev.index or 0, prec, load_tuning=False)
            default_ms, shape_ms = [], []
            for i, b in enumerate(bks):
                act = torch.from_numpy(np.linspace(0, n - 1, b).astype(np.int32)).to(dev)
                out = (torch.empty((b, 3), dtype=torch.float64, device=dev),
                       torch.empty((b, 3), dtype=torch.float64, device=dev),
                       torch.empty(b, dtype=torch.float64, device=dev))
                call = lambda: plain.forces(P, V, M, act, eps2, *out)
                plain.set_launch(0)
                default_ms.append(_graph_ms(plain, call))
                K, L, tl, wg = _full(choice[i])
                plain.set_launch(K, L, best_of[i][choice[i]][1], tl, wg)
                shape_ms.append(_graph_ms(plain, call))
            plain.close()
            n_min = _small_n_min(n, default_ms, shape_ms)
            log(f"# {prec} N={n}: small-system launch {[round(x, 5) for x in default_ms]} ms, "
                f"tuned shapes {[round(x, 5) for x in shape_ms]} ms: entries from N = {n_min}")
        for i, (b, (lo, hi)) in enumerate(zip(bks, ranges)):
            K, L, tl, wg = _full(choice[i])
            ms, S, n_iblk = best_of[i][choice[i]]
            items = S * n_iblk if S else 0
            e = dict(prec=prec, n_min=n_min, act_min=lo, act_max=hi, K=K, L=L, T=tl, WG=wg, items=items,
                     ms=round(ms, 5), rep_n_active=b, gint=round(b * n / ms / 1e6, 2))
            if n_min != n:
                e["rep_n"] = n
            if choice[i] != fastest[i]:
                fK, fL, fT, fW = _full(fastest[i])
                e["fastest"] = dict(K=fK, L=fL, T=fT, WG=fW, ms=round(times[i][fastest[i]], 5))
            entries.append(e)
            log(json.dumps(e))
    return entries


# Tables in whole rounds: the smallest N of each table and the two systems it
# is timed on, the work items tried (per compute unit: a unit is busy to the end
# with its share, so what counts is how many whole items that is), and the
# active counts at which a new range may start.
ROUND_TABLES = {4097: (6000, 13000), 16385: (22000, 50000), 65536: (65536, 150000), 262144: (262144, 600000)}
ROUND_ITEMS = [1, 2, 3, 4, 5, 6, 8, 10, 12, 14, 16, 20, 24, 32, 48, 64, 96]
ROUND_EDGES = [0, 3, 23, 61, 128, 256, 513, 1024, 2049, 4096, 8193, 16384, 32769, 65536, 131073]
# all-active counts from here on keep the entry of the table they start from:
# few, large items win in sustained runs, which one timed call does not show
ROUND_KEEP = 65536
PARTIAL_ROWS = 16384 * 256  # S x rows that stay within the fixed scratch (56 bytes a row)


def _round_ranges(points, starts=()):
    """Ranges of active counts: those that start where the present entries do,
    and others where ROUND_EDGES are a third away from all of them."""
    lo = sorted({0, *starts} | {c for c in ROUND_EDGES
                                if all(max(c, b, 1) > 1.35 * max(min(c, b), 1) for b in starts)})
    lo = [c for c in lo if c < points[-1]]
    return list(zip(lo, [c - 1 for c in lo[1:]] + [2 ** 31 - 1]))


def _round_counts(lo, hi, points):
    """The (N, active count) a range is timed at: a quarter and three quarters of
    its way on a logarithmic scale; all particles in the last range."""
    out = []
    for n, f in zip(points, (0.25, 0.75)):
        a, b = max(lo, 1), min(hi, n)
        if b >= a:
            out.append((n, n if hi == 2 ** 31 - 1 else max(1, int(round(a * (b / a) ** f)))))
    return out


def _round_pick(times):
    """The entry of a range from {(K, L, T, items): [ms, ...]}: the smallest
    geometric mean; a shape of a kernel family (which shares a device-count
    launch) within 2 %, and of these the fewest partial sums within 0.7 %."""
    mean = {k: math.exp(sum(map(math.log, v)) / len(v)) for k, v in times.items()}
    fam = {k: m for k, m in mean.items() if _family((k[0], k[1], k[2], WG))}
    pool = fam if fam and min(fam.values()) < 1.02 * min(mean.values()) else mean
    top = 1.007 * min(pool.values())
    return min((k for k in pool if pool[k] <= top), key=lambda k: (k[3] * (WG // max(k[1], 1)) * k[0], pool[k]))


def _round_merge(times, loss=1.015):
    """Neighbouring ranges share an entry where that costs none of them more than
    `loss`: [(first, last, entry)]."""
    mean = lambda r, k: math.exp(sum(map(math.log, times[r][k])) / len(times[r][k]))
    own = [_round_pick(t) for t in times]
    out, i = [], 0
    while i < len(times):
        j, entry = i, own[i]
        while j + 1 < len(times):
            span = range(i, j + 2)
            fits = [k for k in times[i] if all(k in times[r] and mean(r, k) <= loss * mean(r, own[r]) for r in span)]
            if not fits:
                break
            entry, j = min(fits, key=lambda k: sum(math.log(mean(r, k)) for r in span)), j + 1
        out.append((i, j, entry))
        i = j + 1
    return out


def tune_rounds(ctx, n_min, points, old, precisions=("fp64", "mixed", "mixed_ds"), log=print):
    """Entries from N = n_min on in whole rounds of work items per compute unit.
    FP64 takes any shape; the mixed policies keep the lane split and the tile of
    the context's present choice, so that the composition of their float sums
    stays.  The context holds the table to start from, `old` its entries."""
    import synth
    dev = ctx.device
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    put = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    bodies = {n: synth.plummer(n, 2) for n in points}
    bodies = {n: (put(p.pos), put(p.vel), put(p.mass)) for n, p in bodies.items()}
    eps2, entries = 2.0 ** -16, []
    lanes = lambda K, L, T: (max(L, 1), T if L >= 1 else TILE)
    for prec in precisions:
        ctx.set_precision(prec)
        ranges, times, kept = [], [], []
        mine = [o for o in old if o.get("kind", 0) == 0 and o["prec"] == prec and o["n_min"] == n_min]
        for lo, hi in _round_ranges(points, [o["act_min"] for o in mine]):
            held = [o for o in mine if o["act_min"] <= lo <= o["act_max"]]
            if min(n_min, lo) >= ROUND_KEEP and held:
                kept.append(dict(held[-1], act_min=lo, act_max=hi))
                continue
            at = _round_counts(lo, hi, points)
            K0, L0, _, T0, _ = ctx.get_shape(max(at[0][0], n_min), at[0][1])
            t = {}
            for n, a in at:
                act = torch.from_numpy(np.linspace(0, n - 1, a).astype(np.int32)).to(dev)
                out = (torch.empty((a, 3), dtype=torch.float64, device=dev),
                       torch.empty((a, 3), dtype=torch.float64, device=dev),
                       torch.empty(a, dtype=torch.float64, device=dev))
                done = {}
                reps = max(2, int(2 ** 33 / (n * a)) if n * a > 2 ** 26 else 20)
                for K, L in SHAPES:
                    T = TILE if prec == "fp64" else T0
                    if (prec != "fp64" and lanes(K, L, T) != lanes(K0, L0, T0)) or (K > 1 and a < 32 * K):
                        continue
                    if (T != TILE and (T, WG) not in TILE_WG.get((K, L), [])) or (L <= 0 and L0 > 0):
                        continue
                    if prec == "fp64" and L > 4 and n * a > 2 ** 30:
                        continue
                    ib = (WG // max(L, 1)) * K
                    blocks, tiles = -(-a // ib), -(-n // T)
                    for g in ROUND_ITEMS:
                        S = max(1, min(tiles, g * cus // blocks))
                        if g * cus * ib > PARTIAL_ROWS or (g > 4 and blocks > 2 * cus * g):
                            continue
                        if (K, L, S) not in done:
                            done[K, L, S] = ctx.time_forces(K, L, S, *bodies[n], act, eps2, *out, reps=reps, T=T, WG=WG)
                        t.setdefault((K, L, T, g * cus), []).append(done[K, L, S])
            t = {k: v for k, v in t.items() if len(v) == len(at)}
            ranges.append((lo, hi, at))
            times.append(t)
            best = _round_pick(t)
            log(f"# {prec} N >= {n_min}, {lo} to {hi} active, timed at {at}: {best} {[round(x, 5) for x in t[best]]} ms")
        for i, j, (K, L, T, items) in _round_merge(times):
            n, a = ranges[j][2][0]
            ms = times[j][K, L, T, items][0]
            entries.append(dict(prec=prec, n_min=n_min, act_min=ranges[i][0], act_max=ranges[j][1], K=K, L=L, T=T,
                                WG=WG, items=items, ms=round(ms, 5), rep_n=n, rep_n_active=a,
                                gint=round(a * n / ms / 1e6, 2)))
        entries += kept
    return entries


# Shapes of the batched force kernel (L = 0: scalar j-path)
BATCH_SHAPES = [(1, 1), (1, 4), (1, 16), (1, 64), (2, 1), (2, 4), (2, 16), (1, 0), (2, 0)]
# kind 1 (nbody_forces_batch) keys: mean active rows per system, timed on
# all-active batches of equal systems of this size
BATCH_BUCKETS = [128, 256, 512, 1024, 2048, 4096, 8192, 16384]
# kind 2 (batched block steps) keys: mean system size, timed as
# graph-replayed block steps over one synchronisation interval
STEP_SHAPES = [(1, 1), (1, 4), (1, 16), (1, 64), (1, 0), (2, 0)]
STEP_BUCKETS = [256, 1024, 4096]


def _equal_batch(size, total, seed):
    import synth
    return synth.cluster_batch(seed=seed, n_clusters=max(1, total // size), n_min=size, n_max=size)


def _wall_ms(fn, reps):
    fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) * 1e3 / reps


def tune_batch_forces(ctx, precisions=("fp64", "mixed", "mixed_ds"), buckets=BATCH_BUCKETS, total=1 << 19,
                      reps=3, log=print):
    """Kind 1 entries: the fastest batched shape for nbody_forces_batch on
    all-active batches of `total` bodies in equal systems of each size (the
    whole call: work list, force kernel and chunk sums)."""
    dev = ctx.device
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    entries = []
    ranges = _midpoints(list(buckets))
    for size, (lo, hi) in zip(buckets, ranges):
        b = _equal_batch(size, total, 11)
        P, V, M = t(b.pos), t(b.vel), t(b.mass)
        n = int(b.offsets[-1])
        act = t(np.arange(n, dtype=np.int32))
        acc = torch.empty((n, 3), dtype=torch.float64, device=dev)
        jerk = torch.empty_like(acc)
        pot = torch.empty(n, dtype=torch.float64, device=dev)
        inter = float(np.sum(b.sizes.astype(np.float64) ** 2))
        for prec in precisions:
            ctx.set_precision(prec)
            best = None
            for K, L in BATCH_SHAPES:
                ctx.tune_clear()
                ctx.tune_add_batch(prec, 1, 1, 2 ** 40, K, L)
                ms = _wall_ms(lambda: ctx.forces_batch(b.offsets, b.eps2, P, V, M, act, b.offsets, acc, jerk, pot),
                              reps)
                if best is None or ms < best[0]:
                    best = (ms, K, L)
            ms, K, L = best
            e = dict(kind=1, prec=prec, key_min=lo, key_max=hi, K=K, L=L, ms=round(ms, 4), rep_size=size,
                     gint=round(inter / ms / 1e6, 1))
            entries.append(e)
            log(json.dumps(e))
    ctx.tune_clear()
    return entries


def tune_batch_steps(ctx, precisions=("fp64", "mixed", "mixed_ds"), buckets=STEP_BUCKETS, total=1 << 18, log=print):
    """Kind 2 entries: the fastest shape for graph-replayed batched block steps
    over one synchronisation interval (dt_max = 1/16) of `total` bodies in
    equal Plummer systems of each size, after a first interval that sizes the
    buffers and captures the graphs."""
    from .integrator import BlockIntegrator
    dev = ctx.device
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
    entries = []
    ranges = _midpoints(list(buckets))
    for size, (lo, hi) in zip(buckets, ranges):
        b = _equal_batch(size, total, 12)
        for prec in precisions:
            ctx.set_precision(prec)
            best = None
            for K, L in STEP_SHAPES:
                ctx.tune_clear()
                ctx.tune_add_batch(prec, 2, 1, 2 ** 40, K, L)
                bi = BlockIntegrator(ctx, t(b.pos), t(b.vel), t(b.mass), b.eps2, 0.01, 1.0 / 16, 30,
                                     offsets=b.offsets)
                bi.run_until(1.0 / 16, graph_steps=16)
                torch.cuda.synchronize()
                s0 = bi.steps
                t0 = time.perf_counter()
                bi.run_until(2.0 / 16, graph_steps=16)
                torch.cuda.synchronize()
                ms = (time.perf_counter() - t0) * 1e3
                if best is None or ms < best[0]:
                    best = (ms, K, L, bi.steps - s0)
                del bi
            ms, K, L, steps = best
            e = dict(kind=2, prec=prec, key_min=lo, key_max=hi, K=K, L=L, ms=round(ms, 3), rep_size=size,
                     steps=int(steps))
            entries.append(e)
            log(json.dumps(e))
    ctx.tune_clear()
    return entries


def forces_source_hash(files=("forces.hip",)):
    """sha256 of the source the table was measured on: the force kernels, or
    with KERNEL_SOURCES also the work queue and the argument structures."""
    import hashlib
    h = hashlib.sha256()
    for name in files:
        with open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


KERNEL_SOURCES = ("forces.hip", "work_queue.h", "nb_internal.h")


def save(entries, path, meta=None):
    doc = {"format": 1, "meta": meta or {}, "entries": entries}
    with open(path, "w") as f:
        json.dump(doc, f, indent=1)


def table_path():
    """The launch table a new context installs: the file named by the
    environment variable NB_TUNE_CACHE when it is set, non-empty and exists
    (the autotuner writes there by default); else the shipped table for this
    GPU when it exists (with a warning when NB_TUNE_CACHE names a missing
    file: the cache has not been written yet); else None."""
    env = os.environ.get("NB_TUNE_CACHE", "")
    if env:
        if os.path.exists(env):
            return env
        warnings.warn(f"NB_TUNE_CACHE names {env}, which does not exist yet; using the shipped table",
                      stacklevel=2)
    return DEFAULT_TABLE if os.path.exists(DEFAULT_TABLE) else None


# The last table read: (the file's path and state, its entries).  Every context
# installs a table, and reading it takes longer than the rest of a context's
# creation; one that is rewritten is read again.
_last_table = (None, None)


def _table_entries(path):
    global _last_table
    st = os.stat(path)
    state = (os.path.abspath(path), st.st_ino, st.st_size, st.st_mtime_ns)
    held, entries = _last_table
    if held != state:
        with open(path) as f:
            entries = json.load(f)["entries"]
        _last_table = (state, entries)
    return entries


def load(ctx, path=DEFAULT_TABLE):
    """Install a saved table into a context (entries in file order)."""
    entries = _table_entries(path)
    single = [e for e in entries if e.get("kind", 0) == 0]
    for e in sorted(single, key=lambda e: e["n_min"]):
        ctx.tune_add(e["prec"], e["n_min"], e["act_min"], e["act_max"], e["K"], e["L"], e["items"],
                     e.get("T", 0), e.get("WG", 0))
    for e in entries:
        if e.get("kind", 0) in (1, 2):
            ctx.tune_add_batch(e["prec"], e["kind"], e["key_min"], e["key_max"], e["K"], e["L"])
    return len(entries)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--n", type=int, nargs="+", default=None, help="system sizes to tune (default: 65536 262144)")
    ap.add_argument("--prec", nargs="+", default=["fp64", "mixed", "mixed_ds"])
    ap.add_argument("--out", default=os.environ.get("NB_TUNE_CACHE") or "tuning.json",
                    help="table to write (default: $NB_TUNE_CACHE, else tuning.json)")
    ap.add_argument("--reps", type=int, default=3)
    ap.add_argument("--max-active", type=int, default=0,
                    help="largest active-set bucket to time (0: up to N); the top bucket's range then covers every larger count")
    ap.add_argument("--append", default="", help="start from the entries of this table")
    ap.add_argument("--rounds", action="store_true",
                    help="retune the tables in whole rounds (those of --n, else all), starting from --append "
                         "(default: the shipped table); this made the shipped table's entries with rep_n")
    ap.add_argument("--batch", action="store_true", help="also tune the batched kernel (nbody_forces_batch)")
    ap.add_argument("--batch-steps", action="store_true", help="also tune the batched block steps")
    ap.add_argument("--batch-only", action="store_true", help="tune only the batched kernel (no --n sweep)")
    ap.add_argument("--batch-forces-only", action="store_true",
                    help="retune only the batched kernel's entries (nbody_forces_batch); keep every other entry")
    args = ap.parse_args()
    if args.n is None:
        args.n = [] if args.rounds else [65536, 262144]
    sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    import paper_1409_5474_amd as nb
    ctx = nb.Context(0, "fp64", load_tuning=False)
    t0 = time.time()
    entries = []
    if args.append:
        with open(args.append) as f:
            entries = json.load(f)["entries"]
    buckets = [b for b in BUCKETS if not args.max_active or b <= args.max_active]
    say = lambda m: print(m, flush=True)
    props = torch.cuda.get_device_properties(0)

    def checkpoint():
        # the table so far, after every stage (a long run keeps what it finished)
        save(entries, args.out, meta={"device": props.name, "gcn_arch": getattr(props, "gcnArchName", ""),
                                      "cus": props.multi_processor_count, "seconds": round(time.time() - t0, 1),
                                      "forces_hip_sha256": forces_source_hash(),
                                      "kernel_sources_sha256": forces_source_hash(KERNEL_SOURCES)})

    if args.rounds:
        args.append = args.append or DEFAULT_TABLE
        with open(args.append) as f:
            entries = json.load(f)["entries"]
        load(ctx, args.append)
        for n in [n for n in ROUND_TABLES if n in args.n] or list(ROUND_TABLES):
            old = [e for e in entries if e.get("kind", 0) == 0 and e["n_min"] == n]
            new = tune_rounds(ctx, n, ROUND_TABLES[n], old, args.prec, log=say)
            entries = [e for e in entries if not (e.get("kind", 0) == 0 and e["n_min"] == n and e["prec"] in args.prec)]
            entries = new + entries
            checkpoint()
            print(f"# table from N={n} done after {time.time() - t0:.0f} s", flush=True)
    elif args.batch_only:
        entries = [e for e in entries if e.get("kind", 0) == 0]
    elif args.batch_forces_only:
        args.batch = True
    else:
        for n in sorted(args.n):
            # an earlier run's entries for this N
            entries = [e for e in entries if e.get("kind", 0) != 0 or
                       not (e["n_min"] == n or (e["n_min"] > n and e.get("rep_n") == n))]
            entries += tune(ctx, n, args.prec, buckets=buckets, reps=args.reps, log=say)
            checkpoint()
            print(f"# N={n} done after {time.time() - t0:.0f} s", flush=True)
    if args.batch or args.batch_only:
        entries = [e for e in entries if e.get("kind", 0) != 1]
        entries += tune_batch_forces(ctx, args.prec, reps=args.reps, log=say)
        checkpoint()
        print(f"# batched forces done after {time.time() - t0:.0f} s", flush=True)
    if args.batch_steps or args.batch_only:
        entries = [e for e in entries if e.get("kind", 0) != 2]
        entries += tune_batch_steps(ctx, args.prec, log=say)
        checkpoint()
        print(f"# batched block steps done after {time.time() - t0:.0f} s", flush=True)
    checkpoint()
    print(f"wrote {args.out} ({len(entries)} entries)", flush=True)


if __name__ == "__main__":
    main()
