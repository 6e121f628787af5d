"""GPU parity of the workgroup-local hulls (sets of up to 65535 points on one
workgroup) against the oracle: at the sizes where a thread, a workgroup or
the LDS is exactly full, on inputs the sample does not represent, and on the
error paths. Hull index lists are integer results: the bar is equality."""
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
