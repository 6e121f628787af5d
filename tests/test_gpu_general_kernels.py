"""The streaming and the persistent kernels under the default precision, with
the workgroup-local kernels off: the tests of both paths again, on the kernels
that they were written for. They still run for what the sieve and the ring
kernels leave, in graphs and in the other precision modes."""
import sys

import numpy as np
import pytest

import oracle
import test_gpu_engine as engine
import test_gpu_graph_tune as tune
import test_gpu_parity as parity
import test_gpu_stream as stream
from paper_1501_04706_amd import sqh, workloads

pytestmark = pytest.mark.gpu

LOCAL = ("k_local", "k_polygon", "k_sieve", "k_ring", "k_rest", "k_batch", "k_pre_", "k_extreme")


class GeneralHull(sqh.Hull):
    """Every call checked: no local kernel, and the streaming kernels where the
    stats say so."""

    def __init__(self, device):
        super().__init__(device)
        self.set_local(False)
        self.set_launch_timing(True)

    def _check(self):
        names = [k for k, _ in self.launch_times()]
        assert names and not any(k.startswith(LOCAL) for k in names), names
        streamed = self.stats()["stream_path"] != 0
        assert ("k_sseed" in names) == streamed and ("k_sfirst<line>" in names) == streamed, names

    def hull(self, *args, **kw):
        out = super().hull(*args, **kw)
        self._check()
        return out

    def hull_soa(self, *args, **kw):
        out = super().hull_soa(*args, **kw)
        self._check()
        return out

    def hull_batched(self, *args, **kw):
        out = super().hull_batched(*args, **kw)
        self._check()
        return out


@pytest.fixture(scope="module")
def H():
    import torch
    assert torch.cuda.is_available(), "gpu tests need a HIP device"
    h = GeneralHull(0)
    yield h
    h.close()


for _mod, _names in ((stream, ("test_stream_matches_general", "test_stream_precision_modes", "test_stream_line_filter_domain",
                               "test_stream_hands_over_to_passes_kernel", "test_stream_degenerate",
                               "test_stream_ignores_memory_past_the_end", "test_stream_pass_count_adapts",
                               "test_soa_input_matches_aos", "test_stream_lds_tail_hand_over")),
                     (tune, ("test_launch_shapes_same_hull", "test_streaming_shapes_same_hull")),
                     (parity, ("test_tile_boundaries", "test_batched_matches_single")),
                     (engine, ("test_engine_alone_equals_oracle", "test_engine_mix_staggered"))):
    for _n in _names:
        globals()[_n] = getattr(_mod, _n)


def test_local_switch(H):
    print("[case] local kernels off and on", file=sys.stderr, flush=True)
    import torch
    xy = workloads.square(300_000, 3)
    t = torch.from_numpy(xy).cuda()
    want = [int(v) for v in oracle.c_hull(xy)]
    assert [int(v) for v in H.hull(t).cpu().numpy()] == want
    st = H.stats()
    assert st["ms_seed"] > 0 and st["ms_split"] > 0 and st["ms_first"] > 0 and st["ms_pass"] > 0
    H.set_local(True)
    try:
        assert [int(v) for v in sqh.Hull.hull(H, t).cpu().numpy()] == want
        assert "k_sieve_solve" in [k for k, _ in H.launch_times()]
    finally:
        H.set_local(False)
    assert sqh.sqh_set_local(0, 1) == sqh.SQH_EINVAL
