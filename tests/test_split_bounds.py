"""The j-split rule of the force launches against the space reserved for its
partial sums, on the library's own host functions (no GPU call): a
device-count launch reserves host_split_rows for every count up to its
regime's top before it knows the count, and the kernels then write
S x n_active rows.  A split of more i-blocks than the item target would write
past them."""
import ctypes

import numpy as np
import pytest


def _functions():
    import paper_1409_5474_amd as nb
    lib = nb.library()
    choose, rows = lib._ZN2nb13host_choose_SEliili, lib._ZN2nb15host_split_rowsEliili
    for f, res in ((choose, ctypes.c_int), (rows, ctypes.c_int64)):
        f.restype = res
        f.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    return choose, rows


def _counts(top, IB, target, rng):
    """Every kind of count up to top: the smallest, around whole i-blocks, around
    as many i-blocks as the target has items, and the largest."""
    near = [1, 2, IB - 1, IB, IB + 1, (target - 1) * IB, target * IB, target * IB + 1, (target + 1) * IB,
            target * IB * 5 // 3, 2 * target * IB, 3 * target * IB + 1, top - 1, top]
    near += [int(x) for x in np.exp(rng.uniform(0, np.log(max(top, 2)), 40))]
    return sorted({d for d in near if 1 <= d <= top})


@pytest.mark.parametrize("tile", [64, 128, 256])
@pytest.mark.parametrize("IB", [1, 4, 16, 64, 128, 256, 512, 1024])
def test_partial_sums_fit_the_reserved_rows(IB, tile):
    choose, rows = _functions()
    rng = np.random.default_rng(IB * 1000 + tile)
    for _ in range(60):
        n = int(np.exp(rng.uniform(0, np.log(4e6))))
        target = int(rng.choice([1, 2, 3, 255, 256, 257, 1024, 4096, 8192, 24576, int(np.exp(rng.uniform(0, 11)))]))
        top = max(1, int(n * rng.choice([1.0, 1.0, 0.3, 2.0])))
        room = rows(top, IB, target, n, tile)
        for d in _counts(top, IB, target, rng):
            S = choose(d, IB, target, n, tile)
            assert 1 <= S <= max(1, -(-n // tile))
            assert S == 1 or S * d <= room, (d, IB, target, n, tile, S, room)


def test_more_blocks_than_the_target_are_not_split():
    # the split's items already exceed the target: no partial sums, no second kernel
    choose, rows = _functions()
    for IB in (1, 4, 256, 512):
        for target in (1, 256, 1024, 8192):
            for blocks in (target + 1, target + 100, 2 * target, 5 * target + 3):
                assert choose(blocks * IB, IB, target, 10 ** 7, 256) == 1
    assert rows(10 ** 6, 256, 1, 10 ** 6, 256) == 0


def test_split_stays_at_or_below_the_saturation_rule():
    # ceil(target / i-blocks) chunks saturate the device; the rule takes that
    # many or one fewer, so it never needs more space than it
    choose, _ = _functions()
    rng = np.random.default_rng(3)
    for _ in range(3000):
        IB, target = int(rng.choice([4, 64, 256, 512])), int(np.exp(rng.uniform(0, 10)))
        n = int(np.exp(rng.uniform(0, np.log(4e6))))
        d = int(np.exp(rng.uniform(0, np.log(4e6))))
        b, tiles = -(-d // IB), -(-n // 256)
        up = max(1, min(-(-target // b), tiles))
        assert up - 1 <= choose(d, IB, target, n, 256) <= up, (d, IB, target, n)


def test_capped_target_is_the_largest_that_fits():
    import paper_1409_5474_amd as nb
    fit = nb.library()._ZN2nb14host_fit_itemsEliilil
    fit.restype, fit.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64,
                                               ctypes.c_int, ctypes.c_int64]
    _, rows = _functions()
    rng = np.random.default_rng(8)
    for _ in range(3000):
        IB, target = int(rng.choice([1, 4, 64, 256, 512])), int(np.exp(rng.uniform(0, 10)))
        n = int(np.exp(rng.uniform(0, np.log(4e6))))
        top = max(1, int(n * rng.uniform(0.01, 1)))
        cap = int(np.exp(rng.uniform(0, 18))) if rng.random() < 0.9 else 2 ** 62
        t = fit(top, IB, target, n, 256, cap)
        assert 1 <= t <= target and rows(top, IB, t, n, 256) <= cap
        # the next target reserves more, unless the number of tiles bounds both
        assert t == target or rows(top, IB, t + 1, n, 256) > cap or rows(top, IB, target, n, 256) <= cap


def test_sixth_order_partial_sums_fit_the_reserved_rows():
    # both lane splits (one and four lanes per row), at every target the cap may leave
    import paper_1409_5474_amd as nb
    split = nb.library()._ZN2nb13forces6_splitEliil
    split.restype, split.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    _, rows = _functions()
    rng = np.random.default_rng(6)
    for _ in range(1500):
        n = int(np.exp(rng.uniform(0, np.log(1e6))))
        top = max(1, int(n * rng.choice([1.0, 0.2])))
        slots = int(rng.choice([32, 768, 1024]))
        target = int(rng.choice([1, 2, 5, 64, slots, 4 * slots, 8 * slots]))
        room = rows(top, 256, target, n, 256)
        for d in _counts(top, 64, target, rng):
            S = split(d, slots, target, n)
            assert S == 1 or S * d <= room, (d, slots, target, n, S, room)
            assert S == 1 or target > 1


@pytest.mark.gpu
@pytest.mark.parametrize("n,cap", [(1000, 100000), (20011, 1 << 20), (20011, 0)])
def test_sixth_order_splits_fit_the_workspace_cap(monkeypatch, n, cap):
    # forces and block steps run under a cap with the split that fits it
    import torch
    import paper_1409_5474_amd as nb
    import synth
    from paper_1409_5474_amd.integrator import BlockIntegrator6
    p = synth.plummer(n, 4)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    P, V, M = t(p.pos), t(p.vel), t(p.mass)
    act = t(np.arange(0, n, 7, dtype=np.int32))
    results = []
    for limit in (None, cap):
        if limit is not None:
            monkeypatch.setenv("NB_MAX_WORKSPACE_BYTES", str(limit))
        c = nb.Context(0, "fp64")
        r = list(c.forces6(P, V, -P, M, act, 1e-3))
        bi = BlockIntegrator6(c, P.clone(), V.clone(), M, 1e-3, 0.15, 1.0 / 16, 24, 0.01)
        for _ in range(3):
            bi.step()
        c.sync()
        used = c.workspace_bytes()
        results.append((r + [bi.pos, bi.vel], [bi.t_tick, bi.level]))
        c.close()
    assert used <= cap
    for a, b in zip(results[0][0], results[1][0]):
        # as above: the order of at most 80 chunks' double sums
        assert torch.linalg.norm(a - b) <= 100 * 80 * 2.0 ** -53 * torch.linalg.norm(a)
    for a, b in zip(results[0][1], results[1][1]):
        assert torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("prec,n,cap", [("fp64", 9620, 6 << 20), ("fp64", 22000, 1 << 20), ("mixed_ds", 65536, 4 << 20),
                                        ("mixed", 16384, 0)])
def test_automatic_splits_fit_the_workspace_cap(prec, n, cap):
    # under NB_MAX_WORKSPACE_BYTES every automatic call of the fourth-order
    # forces runs with the split that fits, from the host's count and the
    # device's; the sums differ from an uncapped context's in their order only
    import os
    import subprocess
    import sys
    code = r"""
import os, sys, numpy as np, torch
sys.path.insert(0, %r)
import paper_1409_5474_amd as nb, synth
prec, n, cap = %r, %d, %d
p = synth.plummer(n, 3)
t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
P, V, M = t(p.pos), t(p.vel), t(p.mass)
sets = [t(np.arange(0, n, max(1, n // k), dtype=np.int32)) for k in (3, 500, 2000)]
def go():
    c = nb.Context(0, prec)
    out = []
    for act in sets:
        out.append(c.forces(P, V, M, act, 1e-4))
        out.append(c.forces_ij(P, V, M, P, V, act, 1e-4))
        full = torch.zeros(n, dtype=torch.int32, device="cuda")
        full[:len(act)] = act
        o = (torch.empty((n, 3), dtype=torch.float64, device="cuda"), torch.empty((n, 3), dtype=torch.float64, device="cuda"),
             torch.empty(n, dtype=torch.float64, device="cuda"))
        c.forces_devcount(P, V, M, full, torch.tensor([len(act)], dtype=torch.int32, device="cuda"), n, 1e-4, *o)
        out.append([x[:len(act)] for x in o])
    torch.cuda.synchronize()
    c.sync()
    return out, c.workspace_bytes()
free, _ = go()
os.environ["NB_MAX_WORKSPACE_BYTES"] = str(cap)
capped, used = go()
worst = 0.0
for a, b in zip(free, capped):
    for x, y in zip(a, b):
        worst = max(worst, float(torch.linalg.norm(x - y) / torch.linalg.norm(x)))
# beside the capped workspace: the scalar path's j-records (up to 48 bytes), under a cap of their own
print("USED", used, used <= cap + (0 if prec == "fp64" else 48 * (n + 1)), worst)
""" % (os.path.dirname(os.path.dirname(os.path.abspath(__file__))), prec, n, cap)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert "USED" in r.stdout, (r.stdout, r.stderr[-2000:])
    used, ok, worst = r.stdout.split("USED")[1].split()
    assert ok == "True", r.stdout
    # double sums of at most 256 chunks in another order (the pairs and, in the
    # mixed policies, the float runs are the same), of terms that cancel to no
    # less than a hundredth
    assert float(worst) <= 100 * 256 * 2.0 ** -53, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("shape,items", [((1, 64), 300), ((1, 256), 700), ((2, 4), 20)])
def test_device_count_with_more_blocks_than_items(shape, items):
    # counts below and above `items` i-blocks: the device-count launch gives the
    # bits of the host-count one
    import torch
    import paper_1409_5474_amd as nb
    import synth
    n = 5000
    ib = 256 // shape[1] * shape[0]
    p = synth.plummer(n, 12)
    t = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    P, V, M, act = t(p.pos), t(p.vel), t(p.mass), t(np.arange(n, dtype=np.int32))
    with_table = nb.Context(0, "fp64", load_tuning=False)
    with_table.tune_add("fp64", 1, 0, 2 ** 31 - 1, *shape, items)
    for na in (ib * items // 2, ib * items, ib * items + 1, min(n, 2 * ib * items + 3), n):
        if na > n:
            continue
        ref = with_table.forces(P, V, M, act[:na].contiguous(), 1e-3)
        out = (torch.empty((n, 3), dtype=torch.float64, device="cuda"),
               torch.empty((n, 3), dtype=torch.float64, device="cuda"),
               torch.empty(n, dtype=torch.float64, device="cuda"))
        with_table.forces_devcount(P, V, M, act, torch.tensor([na], dtype=torch.int32, device="cuda"), n, 1e-3, *out)
        torch.cuda.synchronize()
        for a, b in zip(ref, out):
            assert torch.equal(a, b[:na]), na
    with_table.sync()
    with_table.close()
