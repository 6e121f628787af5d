"""GPU tests of calls that the fast paths take only in part: batches with a set
that ends the call, sets that no polygon thins, sets that are refused. Hull
index lists are integer results: the bar is equality."""
import sys

import numpy as np
import pytest

import oracle
from paper_1501_04706_amd import sqh, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "gpu tests need a HIP device"
    h = sqh.Hull(0)
    yield h
    h.close()


def say(msg):
    print(f"[case] {msg}", file=sys.stderr, flush=True)


def hull(xy):
    return [int(v) for v in oracle.c_hull(xy)]


def batch(H, parts):
    import torch
    off = np.zeros(len(parts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in parts])
    xy = np.concatenate(parts, 0).astype(np.float32)
    out, out_off = H.hull_batched(torch.from_numpy(xy).cuda(), torch.from_numpy(off).cuda())
    out, out_off = out.cpu().numpy(), out_off.cpu().numpy()
    return [[int(v) for v in out[out_off[s]:out_off[s + 1]]] for s in range(len(parts))]


@pytest.mark.parametrize("where", ["small", "big", "both"])
def test_bad_sets_among_many(H, where):
    # sets flagged while other workgroups of the same launch start or wait
    say(f"bad sets among many: {where}")
    rng = np.random.default_rng(3)
    sizes = [int(v) for v in np.exp(rng.uniform(np.log(8), np.log(20_000), 1500))]
    parts = [workloads.make(("square", "disk", "circle")[i % 3], n, i) for i, n in enumerate(sizes)]
    good = [hull(p) for p in parts]
    pick = [i for i, n in enumerate(sizes) if (n <= 1024 if where == "small" else n > 1024 if where == "big" else True)]
    bad = list(parts)
    for i in pick[::7]:
        bad[i] = bad[i].copy()
        bad[i][len(bad[i]) // 2, i % 2] = np.nan if i % 3 else np.inf
    for _ in range(3):
        with pytest.raises(sqh.SqhError) as e:
            batch(H, bad)
        assert e.value.code == sqh.SQH_EINVAL
        assert batch(H, parts) == good


@pytest.mark.parametrize("mode", [sqh.SQH_FP32_FILTER, sqh.SQH_FP32_SEMISTATIC, sqh.SQH_FP64_ONLY])
@pytest.mark.parametrize("n,scale", [(70_001, 3e38), (300_000, 1e25), (1_500_000, 1e28)])
def test_products_overflow(H, n, scale, mode):
    # the area of nearly every point is no float32 number: bounds that are NaN
    import torch
    say(f"products overflow: n={n} scale={scale} mode={mode}")
    H.set_precision(mode)
    try:
        for kind in ("square", "disk"):
            xy = (workloads.make(kind, n, 5).astype(np.float64) * scale).astype(np.float32)
            t = torch.from_numpy(xy).cuda()
            for _ in range(2):  # (the second call enqueues as many passes as the first one took)
                assert [int(v) for v in H.hull(t).cpu().numpy()] == hull(xy), kind
    finally:
        H.set_precision(sqh.SQH_FP32_FILTER)


def timed_hull(H, xy):
    """(hull, launches, stats) with per-launch timing on."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(xy, dtype=np.float32)).cuda()
    H.set_launch_timing(True)
    try:
        H.hull(t)
        got = [int(v) for v in H.hull(t).cpu().numpy()]
        return got, H.launch_times(), H.stats()
    finally:
        H.set_launch_timing(False)


@pytest.mark.parametrize("n", [6000, 70_000, 400_000])
@pytest.mark.parametrize("kind", ["circle", "two thirds"])
def test_times_cover_the_whole_call(H, kind, n):
    # rings (the sieve's kernels, then the ring kernels), and a set that the
    # sieve leaves to the general or the streaming path
    say(f"times: {kind} n={n}")
    xy = workloads.circle(n, 4)
    if kind != "circle":
        xy[::2] = workloads.disk(len(xy[::2]), 5) * np.float32(0.9)
    got, launches, st = timed_hull(H, xy)
    assert got == hull(xy)
    names = [k for k, _ in launches]
    assert "k_polygon" in names and len(set(names)) > 3, names
    assert ("k_ring_emit" in names) == (kind == "circle"), names
    # the events also see the gaps around a kernel: a tenth of room
    assert st["ms_total"] >= 0.9 * sum(ms for _, ms in launches), (st["ms_total"], launches)
def around_its_box(n):
    """A quarter of a circle whose sampled places all hold one inner point, so
    that no polygon is found and the ring kernels take the box's centre, which
    lies on the chord: they cut, sort and join, and then have to refuse."""
    t = np.linspace(0.0, np.pi / 2, n)
    xy = np.stack([np.cos(t), np.sin(t)], 1)
    xy[0], xy[-1] = [1, 0], [0, 1]
    xy = xy[np.random.default_rng(n).permutation(n)]
    ends = [np.array([1.0, 0.0]), np.array([0.0, 1.0])]
    for r in range(128):  # the sample of one workgroup: 128 runs of 8 points
        q = min(r * n // 128, n - 8)
        xy[q:q + 8] = [0.6, 0.6]
    # the box's sample is every n / 8192th point: the two ends among them
    q = [int(i * n // 8192) for i in (11, 4099)]
    assert all(not np.array_equal(xy[i], [0.6, 0.6]) for i in q)
    xy[q] = ends
    return xy.astype(np.float32)


@pytest.mark.parametrize("n", [40_000, 90_001])
def test_refused_ring_writes_nothing(H, n):
    import torch
    say(f"refused ring n={n}")
    xy = around_its_box(n)
    want = hull(xy)
    assert len(want) > 1024
    t = torch.from_numpy(xy).cuda()
    out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    H.set_launch_timing(True)
    try:
        got = H.hull(t, out=out)
        names = [k for k, _ in H.launch_times()]
    finally:
        H.set_launch_timing(False)
    assert [int(v) for v in got.cpu().numpy()] == want
    assert bool((out[len(want):] == -7).all())
    # the ring kernels ran to their end, and another path followed
    assert names.index("k_ring_emit") < len(names) - 1, names


@pytest.mark.parametrize("case", ["square", "rim", "refused"])
def test_prefiltered_subset_is_not_made_twice(H, case):
    # a subset of which the sieve's polygon keeps between a quarter and three
    # quarters, and one whose ring is refused: both go on from the subset
    say(f"pre-filtered subset: {case}")
    if case == "square":
        xy = workloads.square(20_000_000, 0)  # 4176 points are left
    elif case == "rim":
        xy = np.concatenate([workloads.circle(50_000, 3), workloads.disk(950_000, 4) * np.float32(0.95)])
        xy = xy.astype(np.float32)[np.random.default_rng(1).permutation(1_000_000)]
    else:
        # (extents below the ring kernels' range)
        xy = workloads.circle(300_000, 5) * np.float32(1e-20)
    H.set_prefilter(sqh.SQH_PREFILTER_OCTAGON)
    try:
        got, launches, st = timed_hull(H, xy)
    finally:
        H.set_prefilter(sqh.SQH_PREFILTER_NONE)
    names = [k for k, _ in launches]
    assert got == hull(xy)
    assert st["prefilter_points"] > 4096 and st["ms_prefilter"] > 0
    assert names.count("k_pre_keep") == 1 and "k_prefilter" not in names, names
    assert ("k_hull<prefiltered>" in names) == (case == "refused"), names
    assert st["ms_total"] >= 0.9 * sum(ms for _, ms in launches), (st["ms_total"], launches)


def copies(n, k, seed=1):
    t = np.random.default_rng(seed).integers(0, k, n) * (2 * np.pi / k)
    return np.stack([np.cos(t), np.sin(t)], 1).astype(np.float32)


def thin_sets(n):
    rng = np.random.default_rng(n)
    a = rng.permutation(n).astype(np.float32)
    heap = workloads.circle(n, 9)
    heap[rng.random(n) < 0.6] = heap[17]
    yield "one position", np.full((n, 2), 0.5, np.float32)
    yield "two positions", np.float32([[1, 2], [-3, 0.5]])[rng.integers(0, 2, n)]
    yield "line", np.stack([a, 2 * a], 1)
    yield "copies of three", copies(n, 3)
    yield "copies of 150", copies(n, 150)
    yield "copies of 600", copies(n, 600)
    yield "heap", heap
    # most points in one direction from the centre, in 4000 places
    far = np.concatenate([workloads.circle(n - n // 2, 3), (workloads.circle(n // 2, 4) * 1e-3 + [0.9, 0.0])])
    yield "cluster", far[rng.permutation(n)].astype(np.float32)


@pytest.mark.parametrize("n", [4097, 30_000, 65_536, 262_144, 262_145, 600_001])
def test_sets_that_no_polygon_thins(H, n):
    # copies of a few points, and points on a line: no wave and no workgroup
    # may be left with a share of the set (200K copies of three points took the
    # ring kernels 85 ms, 2M 0.9 s)
    for name, xy in thin_sets(n):
        say(f"no polygon: {name} n={n}")
        got, launches, st = timed_hull(H, xy)
        assert got == hull(xy), name
        names = [k for k, _ in launches]
        if name.startswith("copies of") or "position" in name or name == "line":
            assert "k_ring_pocket" not in names or name == "copies of 600", (name, names)
        # (a wave that sorts a thousand copies takes a millisecond)
        assert dict(launches).get("k_ring_pocket", 0.0) < 1.5, (name, launches)


def awkward_sets():
    """Sets that the batch kernels refuse, one by one."""
    rng = np.random.default_rng(8)
    rim = np.concatenate([workloads.circle(54_000, 3), workloads.disk(246_000, 4) * np.float32(0.95)])
    heap = workloads.circle(90_000, 5)
    heap[rng.random(len(heap)) < 0.6] = heap[11]
    a = rng.permutation(200_000).astype(np.float32)
    return {"rim": rim[rng.permutation(len(rim))].astype(np.float32), "heap": heap,
            "small heap": heap[rng.permutation(90_000)[:25_000]], "line": np.stack([a, 2 * a], 1), "copies": copies(200_000, 3), "large": workloads.disk((1 << 20) + 1, 6)}


AWKWARD = list(awkward_sets()) + ["all", "most"]


def around_awkward(which):
    sets = awkward_sets()
    some = list(sets.values()) if which in ("all", "most") else [sets[which]]
    few = [workloads.make(("square", "disk", "circle", "grid")[i % 4], n, i)
           for i, n in enumerate([1, 7, 64, 900, 1024, 1025, 4097, 20_000, 30_000, 60_000] * (1 if which == "most" else 12))]
    few += [np.zeros((0, 2), np.float32)]
    at = len(few) // 2
    return few[:at] + some[:1] + few[at:] + some[1:] + few[:3], [id(s) for s in some]


@pytest.mark.parametrize("which", AWKWARD)
def test_batch_with_awkward_sets(H, which):
    # only the refused sets take the general path, unless they are most of it
    import torch
    say(f"batch with awkward sets: {which}")
    parts, odd = around_awkward(which)
    want = [hull(p) for p in parts]
    H.set_launch_timing(True)
    try:
        got = batch(H, parts)
        names = [k for k, _ in H.launch_times()]
        times = dict(H.launch_times())
    finally:
        H.set_launch_timing(False)
    # (3 ms where one workgroup had a refused set of 25000 points for itself)
    assert which != "small heap" or times["k_hull<plain>"] < 2.2, times
    for s, w in enumerate(want):
        assert got[s] == w, (s, len(parts[s]))
    assert names[0] == "k_batch" and "k_hull<plain>" in names, names
    assert ("k_refused" in names) == (which != "most"), names
    # a short output: the offsets and the total are whole, nothing is written past it
    off = np.zeros(len(parts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in parts])
    xy = torch.from_numpy(np.concatenate(parts, 0).astype(np.float32)).cuda()
    flat = [v for w in want for v in w]
    out = torch.full((len(flat),), -7, dtype=torch.int32, device="cuda")
    out_off = torch.empty(len(parts) + 1, dtype=torch.int64, device="cuda")
    ws = H.workspace(len(xy), len(parts))
    rc, h = sqh.sqh_hull_batched(H.ctx, xy, torch.from_numpy(off).cuda(), len(parts), len(xy), out, out_off,
                                 len(flat) - 9, ws, ws.numel())
    assert rc == sqh.SQH_ECAPACITY and h == len(flat) and int(out_off[-1]) == h
    assert [int(v) for v in out.cpu().numpy()] == flat[:-9] + [-7] * 9
    # a bad point in a refused set, and in one that is not
    for s in (next(i for i, p in enumerate(parts) if id(p) in odd), 3):
        z = [p.copy() for p in parts]
        z[s][len(z[s]) // 2, 1] = np.nan
        with pytest.raises(sqh.SqhError) as e:
            batch(H, z)
        assert e.value.code == sqh.SQH_EINVAL


@pytest.mark.parametrize("which", AWKWARD)
def test_engine_step_with_awkward_requests(H, which):
    say(f"engine step with awkward requests: {which}")
    parts, odd = around_awkward(which)
    bad = workloads.disk(30_000, 3)
    bad[7, 0] = np.inf
    parts = parts + [bad]
    want = [None if p is bad else hull(p) for p in parts]
    E = H.engine(1 << 23, 256, 1 << 22)
    try:
        for passes in (32, 16, 32):
            for i, p in enumerate(parts):
                assert E.admit(p, i)
            E.launch(passes)
            assert E.admit(parts[2], 999)  # (into the other half while the step runs)
            E.finish()
            for _ in range(64):  # (a step of 16 passes may leave residents)
                if E.status()["resident"] + E.status()["staged"] == 0:
                    break
                E.step(passes)
            got = dict(iter(E.poll, None))
            for i, w in enumerate(want):
                assert (got[i] is None) if w is None else ([int(v) for v in got[i]] == w), (passes, i, len(parts[i]))
            assert [int(v) for v in got[999]] == want[2]
            assert E.status()["free_slots"] == E.slots
    finally:
        E.close()


def test_autotune_times_the_shapes_it_stores(H):
    # the shapes are those of the persistent kernel, which the local kernels
    # spare most calls: it has to be the one that is timed, and an entry from a
    # batch must not take a large single set off its path
    import torch
    say("autotune on a batch, a small set and a large one")
    rng = np.random.default_rng(4)
    parts = [workloads.make(("square", "disk", "circle")[i % 3], int(n), i)
             for i, n in enumerate(rng.integers(500, 30_000, 70))]
    off = np.zeros(len(parts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in parts])
    bxy, boff = torch.from_numpy(np.concatenate(parts, 0)).cuda(), torch.from_numpy(off).cuda()
    xy = workloads.square(1_000_000, 3)
    t = torch.from_numpy(xy).cuda()
    assert H.tuning() == '{"entries": []}'
    H.set_launch_timing(True)
    try:
        for args in ((bxy, boff), (t[:20_000],)):
            text = H.autotune(*args, reps=1)
            names = [k for k, _ in H.launch_times()]  # of the last candidate
            assert names == ["k_reset", "k_hull<plain>"], names
            assert '"stream": 0' not in text, text
            assert [int(v) for v in H.hull(t).cpu().numpy()] == hull(xy)
            assert "k_sieve_solve" in [k for k, _ in H.launch_times()]
        text = H.autotune(t, reps=3)
        assert text.count("log2n") == 3
        # 0.09 ms past the sieve, at least 0.25 on the persistent kernel
        assert '"log2n": 19' in text and '"stream": 0' not in text, text
    finally:
        H.set_launch_timing(False)
        H.set_tuning('{"entries": []}')
    assert batch(H, parts) == [hull(p) for p in parts]


@pytest.mark.parametrize("lobes", [2, 5, 40])
@pytest.mark.parametrize("n", [30_000, 300_000])
def test_stars(H, n, lobes):
    # lobes around the centre: whole wedges between them empty, so that the join
    # has to go over the ring at once (0.81 ms at five lobes of 300K points)
    say(f"star of {lobes} lobes n={n}")
    t = np.random.default_rng(lobes).random(n) * 2 * np.pi
    r = 1 + 0.3 * np.cos(lobes * t)
    got, launches, _ = timed_hull(H, np.stack([r * np.cos(t), r * np.sin(t)], 1).astype(np.float32))
    assert got == hull(np.stack([r * np.cos(t), r * np.sin(t)], 1).astype(np.float32))
    assert dict(launches).get("k_ring_join", 0.0) < 0.7, launches


@pytest.mark.parametrize("mode", [sqh.SQH_FP32_FILTER, sqh.SQH_FP64_ONLY])
@pytest.mark.parametrize("n", [500, 4000, 35_000])
def test_overflowing_areas_are_elected_by_bounds(H, n, mode):
    # where float32 has no bounds for an area, float64 has: few points challenge
    # their child's leader exactly (all of them did: 25 ms a batch at 35K points)
    rng = np.random.default_rng(n)
    t = rng.random(n) * 2 * np.pi
    two = np.stack([np.cos(t), np.sin(t)], 1) * np.where(rng.random(n) < 0.5, 1.0, 1e-2)[:, None]
    two[rng.random(n) < 0.5] += [3.0, 1.0]
    H.set_precision(mode)
    try:
        for name, unit in (("circles", two), ("disk", workloads.disk(n, 3)), ("square", workloads.square(n, 4))):
            for scale in (2.0 ** -98, 2.0 ** -70, 1.0, 2.0 ** 62, 2.0 ** 90, 2.0 ** 125):
                say(f"areas by float64 bounds: {name} n={n} scale={scale:.3g} mode={mode}")
                xy = (unit.astype(np.float64) * scale).astype(np.float32)
                want = hull(xy)
                assert batch(H, [xy, workloads.square(2000, 1), xy[:7]])[0] == want
                if n <= 4096:
                    import torch
                    assert [int(v) for v in H.hull(torch.from_numpy(xy).cuda()).cpu().numpy()] == want
                    # (copies and near ties aside; every point of every pass before)
                    assert H.stats()["cmp_exact"] <= 50 + n // 4, H.stats()["cmp_exact"]
    finally:
        H.set_precision(sqh.SQH_FP32_FILTER)


def test_copies_that_the_second_polygon_keeps(H):
    # 2M points in 340 places: some 50 thousand copies of the hull's vertices pass
    # both polygons, and one workgroup solved them 4096 at a time (1.5 ms), each
    # time electing among hundreds of copies by position
    rng = np.random.default_rng(7)
    n = 2_000_000
    places = rng.random((340, 2)).astype(np.float32)
    xy = places[rng.integers(0, 340, n)]
    xy[rng.random(n) < 0.28] = [0.5, 0.4375]
    say(f"copies past both polygons n={n}")
    got, launches, st = timed_hull(H, xy)
    assert got == hull(xy)
    assert dict(launches)["k_rest"] < 0.5, launches
    assert 4096 < st["first_survivors"] <= 65536
