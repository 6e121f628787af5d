"""Workloads of the library as its users call it, for timing.

Point sets are the synthetic recipes of ``workloads.py`` (uniform square and
disk, jittered circle, integer grid with duplicates and collinear borders),
drawn on the GPU from the seed. Every case goes through the Python binding's
public calls and returns the hull sizes and the program's own output buffer
(filled with -1 beforehand: the library writes nothing past the hull).

A case is a dict: ``entry`` (which call), ``kind`` and ``n`` for one point
set, ``sets`` / ``lo`` / ``hi`` / ``total`` for a batch, ``requests`` / ``lo``
/ ``hi`` for the serving engine.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1501_04706_amd import sqh

KINDS = ("square", "disk", "circle", "grid")
MIX = ("square", "disk", "circle")  # the kinds of batches and request streams
HULL_CAP = 1 << 16  # output entries a single hull's program allocates (the largest circle here has about 40,000 vertices)
ROW_CAP = 1 << 15   # ... and per request of a stream


def listed():
    return [
        # the smallest sets a request stream holds: one call's latency
        {"name": "single_1k_square", "entry": "hull", "kind": "square", "n": 1000},
        # a set of the size of a few tiles, ragged
        {"name": "single_20k_disk", "entry": "hull", "kind": "disk", "n": 20011},
        # the paper's smallest set, through the entry point that takes no workspace
        {"name": "noalloc_100k_square", "entry": "noalloc", "kind": "square", "n": 100_000},
        # a program that keeps x and y apart, an ordinary size
        {"name": "soa_1m_disk", "entry": "soa", "kind": "disk", "n": 1_000_003},
        # the paper's largest set: the benchmark's default workload
        {"name": "single_20m_square", "entry": "hull", "kind": "square", "n": 20_000_000},
        # a round cloud: hundreds of hull points, half the points past the first split
        {"name": "single_20m_disk", "entry": "hull", "kind": "disk", "n": 20_000_000},
        # adversarial: nearly every point within a few ulps of the hull, tens of thousands of vertices
        {"name": "single_5m_circle", "entry": "hull", "kind": "circle", "n": 4_999_999},
        # quantised scanner data: duplicates, long collinear runs on the border
        {"name": "single_20m_grid", "entry": "hull", "kind": "grid", "n": 20_000_000},
        # the paper's first mode (extreme points discard the interior first), octagon form
        {"name": "octagon_5m_disk", "entry": "octagon", "kind": "disk", "n": 5_000_000},
        # many small objects at once (collision shapes, clusters): 512 sets of 64 to 4096 points
        {"name": "batch_512_small", "entry": "batch", "sets": 512, "lo": 64, "hi": 4096, "total": 0},
        # the batched benchmark: 4096 sets of widely different sizes, 64M points in all
        {"name": "batch_4096_64m", "entry": "batch", "sets": 4096, "lo": 64, "hi": 1 << 20, "total": 64_000_000},
        # a saturated request stream from host memory through the serving engine
        {"name": "serving_96", "entry": "serving", "requests": 96, "lo": 1000, "hi": 4_000_000},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))) | rng.randrange(2)


def draw(rng):
    family = rng.choice(("single", "single", "single", "batch", "serving"))
    if family == "single":
        entry = rng.choice(("hull", "hull", "hull", "noalloc", "soa", "octagon"))
        kind = rng.choice(KINDS)
        top = {"noalloc": sqh.SQH_NOALLOC_MAX_POINTS - 1, "hull": 20_000_000, "soa": 10_000_000,
               "octagon": 10_000_000}[entry]
        if kind == "circle":
            top = min(top, 5_000_000)
        return {"entry": entry, "kind": kind, "n": _log_int(rng, 1000, top - 1)}
    if family == "batch":
        sets = _log_int(rng, 16, 4095)
        hi = _log_int(rng, 1024, 1 << 20)
        mean = (hi - 64) / math.log(hi / 64)
        total = 64_000_000 if sets * mean > 40_000_000 else 0
        return {"entry": "batch", "sets": sets, "lo": 64, "hi": hi, "total": total}
    return {"entry": "serving", "requests": rng.randrange(8, 96), "lo": 1000, "hi": _log_int(rng, 20_000, 3_900_000)}


# ---- inputs ----

def _points(kind, n, gen):
    """The recipes of workloads.py on the device; (n, 2) float32."""
    dev = gen.device

    def u(m):
        return torch.rand(m, dtype=torch.float64, device=dev, generator=gen)

    if kind == "square":
        return torch.rand((n, 2), dtype=torch.float32, device=dev, generator=gen)
    if kind == "grid":
        side, nb = 4096, n - int(round(0.3 * n))
        base = torch.randint(0, side, (nb, 2), device=dev, generator=gen, dtype=torch.int32)
        # 2 % of the base points on a border (the points are i.i.d.: any of them will do)
        ns = int(0.02 * nb)
        edge = torch.randint(0, 4, (ns,), device=dev, generator=gen)
        base[:ns, 0] = torch.where(edge == 0, 0, torch.where(edge == 1, side - 1, base[:ns, 0]))
        base[:ns, 1] = torch.where(edge == 2, 0, torch.where(edge == 3, side - 1, base[:ns, 1]))
        dups = base[torch.randint(0, nb, (n - nb,), device=dev, generator=gen)]
        pts = torch.cat([base, dups], 0)
        return pts[torch.randperm(n, device=dev, generator=gen)].to(torch.float32).contiguous()
    th = 2.0 * math.pi * u(n)
    r = torch.sqrt(u(n)) if kind == "disk" else 1.0 + 1e-6 * (2.0 * u(n) - 1.0)
    return torch.stack([r * torch.cos(th), r * torch.sin(th)], 1).to(torch.float32).contiguous()


def _sizes(count, lo, hi, rng):
    return np.floor(np.exp(math.log(lo) + rng.random(count) * (math.log(hi) - math.log(lo)))).astype(np.int64)


def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen


def _prepare_batch(case, seed):
    # sizes come from the case alone, points and kinds from the seed: every
    # seed gives the same amount of work
    sizes = _sizes(case["sets"], case["lo"], case["hi"], np.random.default_rng(case["sets"] * 7919 + case["hi"]))
    if case["total"]:
        sizes = np.maximum(case["lo"], np.floor(sizes * (case["total"] / sizes.sum()))).astype(np.int64)
    gen = _generator(seed)
    which = np.random.default_rng(seed).permutation(np.arange(case["sets"]) % len(MIX))
    off = np.zeros(case["sets"] + 1, dtype=np.int64)
    off[1:] = np.cumsum(sizes)
    xy = torch.empty((int(off[-1]), 2), dtype=torch.float32, device="cuda")
    # one draw per kind, dealt to that kind's sets
    owner = torch.repeat_interleave(torch.from_numpy(which).cuda(), torch.from_numpy(sizes).cuda())
    for k, kind in enumerate(MIX):
        at = (owner == k).nonzero().squeeze(1)
        xy[at] = _points(kind, at.numel(), gen)
    H = sqh.Hull(0)
    H.workspace(int(off[-1]), case["sets"])
    out = torch.full((int(off[-1]),), -1, dtype=torch.int32, device="cuda")
    return {"entry": "batch", "H": H, "xy": xy, "off": torch.from_numpy(off).cuda(), "out": out}


def _serving_requests(case):
    rng = np.random.default_rng(case["requests"] * 104729 + case["hi"])
    sizes = _sizes(case["requests"], case["lo"], case["hi"], rng)
    return sizes, rng.integers(0, len(MIX), size=case["requests"])


def _prepare_serving(case, seed):
    sizes, kinds = _serving_requests(case)
    gen = _generator(seed)
    # one pinned pool per kind; a request is a window into one
    pools = []
    for kind in MIX:
        pool = torch.empty((case["hi"], 2), dtype=torch.float32, pin_memory=True)
        pool.copy_(_points(kind, case["hi"], gen))
        pools.append(pool)
    starts = np.floor(np.random.default_rng(seed).random(len(sizes)) * (case["hi"] - sizes + 1)).astype(np.int64)
    reqs = [pools[int(k)][int(s):int(s) + int(n)] for k, s, n in zip(kinds, starts, sizes)]
    H = sqh.Hull(0)
    stage = 1 << 24
    return {"entry": "serving", "H": H, "E": H.engine(1 << 25, 1024, stage), "copy": torch.cuda.Stream(),
            "reqs": reqs, "pools": pools, "rows": np.full((len(reqs), ROW_CAP), -1, dtype=np.int32),
            "counts": np.zeros(len(reqs), dtype=np.int64)}


def prepare(case, seed):
    if case["entry"] == "batch":
        return _prepare_batch(case, seed)
    if case["entry"] == "serving":
        return _prepare_serving(case, seed)
    n = case["n"]
    xy = _points(case["kind"], n, _generator(seed))
    H = sqh.Hull(0)
    state = {"entry": case["entry"], "H": H, "xy": xy, "n": n,
             "out": torch.full((min(n, HULL_CAP),), -1, dtype=torch.int32, device="cuda")}
    if case["entry"] == "soa":
        state["x"], state["y"] = xy[:, 0].contiguous(), xy[:, 1].contiguous()
        H.ws = torch.empty(sqh.sqh_workspace_bytes_soa(n), dtype=torch.uint8, device="cuda")
    elif case["entry"] != "noalloc":
        H.workspace(n, 1)
    if case["entry"] == "octagon":
        H.set_prefilter(sqh.SQH_PREFILTER_OCTAGON)
    return state


# ---- one pass ----

def _serve(state):
    """Every request admitted as room allows (copies on their own stream,
    overlapping the running step), steps until all hulls are back."""
    E, reqs, rows, counts = state["E"], state["reqs"], state["rows"], state["counts"]
    left, nxt, inflight = len(reqs), 0, False
    while left:
        while nxt < len(reqs) and E.admit(reqs[nxt], nxt, stream=state["copy"]):
            nxt += 1
        if inflight:
            E.finish()
            while True:
                r = E.poll()
                if r is None:
                    break
                tag, hull = r
                counts[tag] = len(hull)
                rows[tag, :len(hull)] = hull
                left -= 1
        inflight = E.launch(32)
    if inflight:
        E.finish()
    return {"hulls": rows, "counts": counts}


def run(state):
    H, entry, out = state["H"], state["entry"], state["out"] if "out" in state else None
    if entry in ("hull", "octagon"):
        h = H.hull(state["xy"], out=out).numel()
    elif entry == "soa":
        h = H.hull_soa(state["x"], state["y"], out=out).numel()
    elif entry == "noalloc":
        rc, h = sqh.sqh_hull_noalloc(H.ctx, state["xy"], state["n"], out, out.numel())
        if rc != sqh.SQH_OK:
            raise sqh.SqhError(rc, "sqh_hull_noalloc")
    elif entry == "batch":
        hulls, off = H.hull_batched(state["xy"], state["off"], out=out)
        return {"h": hulls.numel(), "offsets": off, "out": out}
    else:
        return _serve(state)
    return {"h": h, "out": out}


def work(case):
    """Each coordinate pair read once, one orientation test (7 operations) per point; the hulls written are small."""
    if case["entry"] == "batch":
        sizes = _sizes(case["sets"], case["lo"], case["hi"], np.random.default_rng(case["sets"] * 7919 + case["hi"]))
        if case["total"]:
            sizes = np.maximum(case["lo"], np.floor(sizes * (case["total"] / sizes.sum()))).astype(np.int64)
        n = int(sizes.sum())
    elif case["entry"] == "serving":
        n = int(_serving_requests(case)[0].sum())
    else:
        n = case["n"]
    return {"bytes": 8 * n, "flops": 7 * n}


def exact(case, seed):
    """Every output is a whole number (indices and counts), held to equality: no value in 64 bits to come near to."""
    return None
