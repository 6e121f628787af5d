"""GPU parity of the workgroup-local kernels (small sets in LDS, sets past the
sieve, batches, rings in pockets) against the oracle: at the sizes where a
thread, a workgroup, the LDS or a launch shape is exactly full, on inputs the
sample does not represent, and on the error paths. Hull index lists are
integer results: the bar is equality."""
import sys

import numpy as np
import pytest

import oracle
from oracle import hull_exact as he
from paper_1501_04706_amd import sqh, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "gpu tests need a HIP device"
    h = sqh.Hull(0)
    yield h
    h.close()


def gpu(H, xy):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(xy, dtype=np.float32).reshape(-1, 2)).to("cuda")
    return [int(v) for v in H.hull(t).cpu().numpy()]


def want(xy):
    return he.hull(xy) if len(xy) < 300 else [int(v) for v in oracle.c_hull(xy)]


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 255, 257, 1023, 1024, 1025, 4095, 4096, 4097, 12287, 16385, 65535])
def test_sizes(H, n):
    print(f"[case] local n={n}", file=sys.stderr, flush=True)
    for kind in ("square", "disk", "circle", "grid"):
        xy = workloads.make(kind, n, n + 5)
        for mode in (sqh.SQH_FP32_FILTER, sqh.SQH_FP32_SEMISTATIC, sqh.SQH_FP64_ONLY):
            H.set_precision(mode)
            try:
                assert gpu(H, xy) == want(xy), (kind, mode)
            finally:
                H.set_precision(sqh.SQH_FP32_FILTER)


def shapes(n):
    rng = np.random.default_rng(n)
    d = workloads.disk(n, 7)
    yield "sorted by x", d[np.argsort(d[:, 0], kind="stable")]
    yield "far from the origin", (d + np.float32([4096.0, -9000.0])).astype(np.float32)
    yield "large", (d * np.float32(3e37)).astype(np.float32)
    yield "products overflow", (d * np.float32(3e38)).astype(np.float32)
    yield "tiny", (d * np.float32(1e-30)).astype(np.float32)
    yield "one position", np.full((n, 2), 0.25, np.float32)
    yield "vertical", np.stack([np.zeros(n), rng.integers(0, 50, n)], 1).astype(np.float32)
    yield "collinear", np.stack([np.arange(n) % 701, 2 * (np.arange(n) % 701)], 1).astype(np.float32)
    yield "vertical sides", np.stack([rng.integers(0, 2, n), rng.random(n)], 1).astype(np.float32)
    # growing outwards: what a prefix or a sample certifies keeps changing
    t = np.arange(n) * 2.399963
    r = 1.0 + np.arange(n) / n
    yield "spiral", np.stack([r * np.cos(t), r * np.sin(t)], 1).astype(np.float32)
    # the sample's stride falls on one half plane only
    s = np.where((np.arange(n) % 16 == 0)[:, None], d * np.float32(0.01), d)
    yield "stride", s.astype(np.float32)
    x = rng.permutation(n) - n // 2
    yield "parabola", np.stack([x, x.astype(np.float64) ** 2 / n], 1).astype(np.float32)


@pytest.mark.parametrize("n", [1000, 4000, 4100, 30000])
def test_shapes(H, n):
    for name, xy in shapes(n):
        print(f"[case] local shape {name} n={n}", file=sys.stderr, flush=True)
        assert gpu(H, xy) == [int(v) for v in oracle.c_hull(xy)], name


@pytest.mark.parametrize("n", [700, 4000, 50_000])
def test_errors_and_capacity(H, n):
    import torch
    xy = workloads.disk(n, 3)
    expect = [int(v) for v in oracle.c_hull(xy)]
    for bad in (np.nan, np.inf, -np.inf):
        for at in (0, n // 2 + 1, n - 1):
            for col in (0, 1):
                z = xy.copy()
                z[at, col] = bad
                with pytest.raises(sqh.SqhError) as e:
                    gpu(H, z)
                assert e.value.code == sqh.SQH_EINVAL
    t = torch.from_numpy(xy).cuda()
    ws = H.workspace(n, 1)
    out = torch.full((len(expect) + 8,), -7, dtype=torch.int32, device="cuda")
    rc, h = sqh.sqh_hull(H.ctx, t, n, out, 5, ws, ws.numel())
    assert rc == sqh.SQH_ECAPACITY and h == len(expect)
    assert [int(v) for v in out.cpu().numpy()] == expect[:5] + [-7] * (len(expect) + 3)
    rc, h = sqh.sqh_hull(H.ctx, t, n, out, out.numel(), ws, ws.numel())
    assert rc == sqh.SQH_OK and [int(v) for v in out.cpu().numpy()] == expect + [-7] * 8
    rc, h = sqh.sqh_hull(H.ctx, t, n, out, out.numel(), ws, 16)
    assert rc == sqh.SQH_ENOMEM


@pytest.mark.parametrize("n", [100_000, 100_001, 1_500_000, 1_500_001])
def test_sieve_sizes(H, n):
    """Both sides of the sieve's launch shapes; what its sample misses, keeps
    whole (copies) or cannot use (flat sets), more points left than one
    workgroup takes, and non-finite coordinates wherever they are."""
    rng = np.random.default_rng(n)
    cases = [c for c in shapes(n) if c[0] not in ("parabola", "large", "tiny")]
    tri = np.float32([[0, 0], [1, 0], [0.25, 1]])
    cases += [("copies of three points", tri[rng.integers(0, 3, n)]),
              ("flat", (workloads.disk(n, 2) * np.float32([1.0, 1e-6])).astype(np.float32)),
              ("outer tenth copied", np.where((rng.random(n) < 0.1)[:, None], tri[rng.integers(0, 3, n)],
                                              workloads.disk(n, 3) * np.float32(0.1) + np.float32(0.4)).astype(np.float32)),
              ("grid", workloads.grid(n, 4, side=64))]
    for name, xy in cases:
        print(f"[case] sieve {name} n={n}", file=sys.stderr, flush=True)
        assert gpu(H, xy) == [int(v) for v in oracle.c_hull(xy)], name
    d = workloads.disk(n, 5) * np.float32(0.5)
    for at in (0, n // 3, n - 1):
        z = d.copy()
        z[at, 1] = np.nan
        with pytest.raises(sqh.SqhError) as e:
            gpu(H, z)
        assert e.value.code == sqh.SQH_EINVAL


def rings(n):
    """Sets most of whose points are hull vertices, and their awkward relatives."""
    rng = np.random.default_rng(n)
    c = workloads.circle(n, n)
    yield "circle", c
    yield "sorted", c[np.argsort(c[:, 0], kind="stable")]
    yield "flat", (c * np.float32([1.0, 1e-4])).astype(np.float32)
    yield "far from the origin", (c + np.float32([31.0, -17.0])).astype(np.float32)
    yield "copies", workloads.circle(max(1, n // 3), 5)[rng.integers(0, max(1, n // 3), n)]
    t = rng.integers(0, 5000, n) * 0.00125
    yield "few directions", np.stack([np.cos(t), np.sin(t)], 1).astype(np.float32)
    t = np.where(rng.random(n) < 0.8, rng.random(n) * 0.3, rng.random(n) * 6.28)
    yield "uneven", np.stack([np.cos(t), np.sin(t)], 1).astype(np.float32)
    x = rng.permutation(n) - n // 2
    yield "parabola", np.stack([x, x.astype(np.float64) ** 2 / n], 1).astype(np.float32)
    two = np.concatenate([c[: n // 2], c[n // 2:] + np.float32([5.0, 1.0])])  # arcs that meet at reflex nodes
    yield "two circles", two[rng.permutation(n)]
    yield "most of two circles", np.concatenate([c[: n - n // 8], (c[n - n // 8:] * np.float32(0.5) + np.float32([1.2, 0.0]))])


@pytest.mark.parametrize("n", [4097, 6001, 40_000, 65535])
def test_single_rings(H, n):
    for name, xy in rings(n):
        print(f"[case] ring {name} n={n}", file=sys.stderr, flush=True)
        assert gpu(H, xy) == [int(v) for v in oracle.c_hull(xy)], name


@pytest.mark.parametrize("n", [65536, 65537, 300_001, 1_000_003])
def test_large_rings(H, n):
    """Rings over the whole chip: wedges of every size, one that empties, a
    pocket's points in several loads, centres that are no inner point."""
    rng = np.random.default_rng(n)
    sets = list(rings(n))
    c = workloads.circle(n, 9)
    heap = c.copy()
    heap[rng.random(n) < 0.6] = c[17]  # copies: more of one point than a wave sorts
    arc = rng.random(n) * 1.5
    half = np.stack([np.cos(2 * arc), np.sin(2 * arc)], 1).astype(np.float32)
    half[:5] = [[-1, -0.5], [1, -0.5], [0, -0.75], [-0.5, -0.625], [0.5, -0.625]]
    sets += [("heap", heap), ("half", half), ("quarter", np.stack([np.cos(arc), np.sin(arc)], 1).astype(np.float32)),
             ("beyond its frame", c + np.float32([300.0, 0.0])), ("tiny", c * np.float32(1e-20)),
             ("filled", (c * np.where(np.arange(n) % 3, rng.random(n), 1.0)[:, None]).astype(np.float32))]
    for name, xy in sets:
        print(f"[case] large ring {name} n={n}", file=sys.stderr, flush=True)
        assert gpu(H, xy) == [int(v) for v in oracle.c_hull(xy)], name


def test_large_ring_errors(H):
    import torch
    c = workloads.circle(200_000, 3)
    h = len(oracle.c_hull(c))
    z = c.copy()
    z[123_457, 1] = np.inf
    with pytest.raises(sqh.SqhError) as e:
        gpu(H, z)
    assert e.value.code == sqh.SQH_EINVAL
    d = torch.from_numpy(c).cuda()
    out = torch.full((h + 8,), -7, dtype=torch.int32, device="cuda")
    with pytest.raises(sqh.SqhError) as e:
        H.hull(d, out=out[: h - 1])
    assert e.value.code == sqh.SQH_ECAPACITY
    assert out[h - 1 :].cpu().tolist() == [-7] * 9
    assert gpu(H, c) == [int(v) for v in oracle.c_hull(c)]


@pytest.mark.parametrize("n", [1, 2, 255, 2047, 4097, 8193, 30_001, 65_537, 400_003])
@pytest.mark.parametrize("mode", [sqh.SQH_PREFILTER_QUAD, sqh.SQH_PREFILTER_OCTAGON])
def test_prefiltered_subsets(H, n, mode):
    """The subset by every route (one workgroup, the sieve, the ring kernels),
    its indices, and copies whose lowest index must win."""
    rng = np.random.default_rng(n)
    sets = [(k, workloads.make(k, n, n + 3)) for k in ("square", "disk", "grid", "circle")]
    sets += [("copies", workloads.circle(max(1, n // 3), 7)[rng.integers(0, max(1, n // 3), n)]),
             ("line", np.stack([np.arange(n)] * 2, 1).astype(np.float32)[rng.permutation(n)]),
             ("overflow", workloads.square(n, 2) * np.float32(3e38)),
             ("half and half", np.concatenate([workloads.circle(n - n // 2, 3), workloads.disk(n // 2, 4) * np.float32(1.01)])
              .astype(np.float32)[rng.permutation(n)])]
    H.set_prefilter(mode)
    try:
        for name, xy in sets:
            print(f"[case] pre-filtered {name} n={n} mode={mode}", file=sys.stderr, flush=True)
            assert gpu(H, xy) == want(xy), name
            assert 0 <= H.stats()["prefilter_points"] <= n
    finally:
        H.set_prefilter(sqh.SQH_PREFILTER_NONE)


@pytest.mark.parametrize("n", [1024, 4096, 4097, 20_000, 160_000, 700_000])
def test_batches(H, n):
    """Every kind of set in one batch, with empty sets and a ragged last one:
    each size class, rings in pockets, sieved sets."""
    import torch
    print(f"[case] batch of sets of about {n}", file=sys.stderr, flush=True)
    parts = [np.zeros((0, 2), np.float32)] + [xy for _, xy in rings(n)][:10 if n < 500_000 else 2]
    parts += [workloads.make(k, m, 3) for k in ("square", "disk", "grid") for m in (n, max(1, n // 7))]
    parts += [workloads.circle(m, 4) for m in (1, 2, 3, 65)] + [np.zeros((0, 2), np.float32)]
    off = np.zeros(len(parts) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in parts])
    xy = np.concatenate(parts, 0).astype(np.float32)
    out, out_off = H.hull_batched(torch.from_numpy(xy).cuda(), torch.from_numpy(off).cuda())
    out, out_off = out.cpu().numpy(), out_off.cpu().numpy()
    for s, p in enumerate(parts):
        assert [int(v) for v in out[out_off[s]:out_off[s + 1]]] == [int(v) for v in oracle.c_hull(p)], s


def test_batch_errors(H):
    import torch
    parts = [workloads.disk(500, 1), workloads.circle(30_000, 2), workloads.disk(30_000, 3)]
    off = np.zeros(4, np.int64)
    off[1:] = np.cumsum([len(p) for p in parts])
    xy = np.concatenate(parts, 0)
    off_d = torch.from_numpy(off).cuda()
    want = [int(v) for p in parts for v in oracle.c_hull(p)]
    for at in (3, 500 + 17, 30_000, 30_500 + 29_999):  # each kind of set, on and off its sample
        z = xy.copy()
        z[at, 0] = np.nan
        with pytest.raises(sqh.SqhError) as e:
            H.hull_batched(torch.from_numpy(z).cuda(), off_d)
        assert e.value.code == sqh.SQH_EINVAL
    for bad in ([0, 500, 400, len(xy)], [1, 500, 600, len(xy)], [0, 500, 600, len(xy) - 1], [0, -5, 600, len(xy)]):
        with pytest.raises(sqh.SqhError) as e:
            H.hull_batched(torch.from_numpy(xy).cuda(), torch.tensor(bad, dtype=torch.int64, device="cuda"))
        assert e.value.code == sqh.SQH_EINVAL
    # a short output: the offsets and the total are whole, nothing is written past it
    ws = H.workspace(len(xy), 3)
    cap = len(want) - 100
    out = torch.full((len(want),), -7, dtype=torch.int32, device="cuda")
    out_off = torch.empty(4, dtype=torch.int64, device="cuda")
    rc, h = sqh.sqh_hull_batched(H.ctx, torch.from_numpy(xy).cuda(), off_d, 3, len(xy), out, out_off, cap, ws, ws.numel())
    assert rc == sqh.SQH_ECAPACITY and h == len(want)
    assert [int(v) for v in out.cpu().numpy()] == want[:cap] + [-7] * 100
    assert int(out_off[3]) == len(want)


def serve(E, reqs, passes, per_step=10 ** 6):
    """Admits as room allows, per_step requests at most before each step."""
    import torch
    copy = torch.cuda.Stream()
    got, nxt, inflight = {}, 0, False
    for _ in range(1000):
        for _ in range(per_step):
            if nxt == len(reqs) or not E.admit(reqs[nxt], nxt, stream=copy):
                break
            nxt += 1
        if inflight:
            E.finish()
            for tag, hull in iter(E.poll, None):
                got[tag] = hull
        if len(got) >= len(reqs):
            return got
        inflight = E.launch(passes)
    raise AssertionError("the engine does not finish")


@pytest.mark.parametrize("hi,per_step", [(3000, 7), (90_000, 10 ** 6), (1_400_000, 4)])
def test_engine_steps_of_many_passes(H, hi, per_step):
    """Steps on the local kernels: every size class, requests of more than a
    million points, bad and empty ones, one that the local kernels leave
    (a quarter of a circle), and a step of few passes in between."""
    rng = np.random.default_rng(hi)
    sizes = [1, 2, 63, 64, 65, 1024, 1025, 4096, 4097, hi, hi - 1] + [int(v) for v in rng.integers(1, hi, 14)]
    kinds = ("square", "disk", "circle", "grid")
    reqs = [workloads.make(kinds[i % 4], n, i) for i, n in enumerate(sizes)]
    if hi > 1 << 20:
        reqs += [workloads.circle((1 << 20) + 1, 3), workloads.disk((1 << 20) + 2, 4), workloads.square(1_600_001, 5)]
    bad = workloads.disk(hi, 6)
    bad[hi // 2, 1] = np.nan
    t = rng.random(hi) * 1.5
    reqs += [bad, np.zeros((0, 2), np.float32), workloads.disk(777, 8), np.stack([np.cos(t), np.sin(t)], 1).astype(np.float32)]
    for left in (False, True):
        rs = reqs if left else reqs[:-1]
        want_ = [None if not np.all(np.isfinite(xy)) else [int(v) for v in oracle.c_hull(xy)] for xy in rs]
        E = H.engine(1 << 23, 64, 1 << 22)
        try:
            for passes in (32, 16, 2):
                print(f"[case] engine hi={hi} passes={passes} left={left}", file=sys.stderr, flush=True)
                got = serve(E, rs, passes, per_step)
                for i, w in enumerate(want_):
                    assert (got[i] is None) if w is None else ([int(v) for v in got[i]] == w), (passes, i, len(rs[i]))
                st = E.status()
                assert st["free_slots"] == E.slots and st["resident"] == 0
            # a request in the table from a step of few passes, then local steps
            assert E.admit(workloads.circle(100_000, 1), 900)
            E.step(1)
            assert E.status()["resident"] == 1
            got = serve(E, rs[:9], 32)
            assert 900 in got and [int(v) for v in got[8]] == want_[8]
        finally:
            E.close()
