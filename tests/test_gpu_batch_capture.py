"""Batched launches recorded in a graph, and on streams that their owner destroys: a
work table belongs to its launch until that has ended, and to a graph for good.
"""
import ctypes

import numpy as np
import pytest

from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu


class Set:
    """n frames, what one call makes of them, and what they should be."""

    def __init__(self, ctx, n, seed, launch):
        import torch

        self.frames = [DeviceFrame(*inputs.g_brain(20 + k % 7, 41 + seed % 5, 100 * seed + k), 8, 4, 0.01,
                                   with_nbr=False) for k in range(n)]
        self.c = [df.as_c() for df in self.frames]
        self.plan = dict(search=1, launch=launch, flags=_lib.KNNF_PLAN_NO_INPUT_CHECK)
        for c in self.c:
            _lib.knnf_filter(ctx, c, dict(search=1, flags=1), current_stream())
        torch.cuda.synchronize()
        self.want = [df.results()[:2] for df in self.frames]
        self.clear()

    def run(self, ctx, stream):
        _lib.knnf_filter_batch(ctx, self.c, self.plan, stream)

    def clear(self):
        for df in self.frames:
            df.clear_outputs()

    def check(self, label):
        for df, want in zip(self.frames, self.want):
            for a, b in zip(df.results()[:2], want):
                assert np.array_equal(a, b), label


@pytest.mark.parametrize("launch", [1, 2], ids=["persistent", "grid"])
@pytest.mark.parametrize("n", [3, 45], ids=["argument", "staged"])
def test_replays_between_other_batches(n, launch):
    import torch

    ctx = _lib.knnf_create(0)
    try:
        rec = [Set(ctx, n, s, launch) for s in range(6)]
        plain = [Set(ctx, n, 20 + s, launch) for s in range(5)]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for x in rec:
                x.run(ctx, current_stream())
        side = torch.cuda.Stream()
        for turn in range(3):
            print(f"replay {turn}", flush=True)
            for x in rec + plain:
                x.clear()
            torch.cuda.synchronize()
            g.replay()
            for k, x in enumerate(plain):
                x.run(ctx, side.cuda_stream if k % 2 else current_stream())
            torch.cuda.synchronize()
            for k, x in enumerate(rec + plain):
                x.check(f"turn {turn}, set {k}")
        assert _lib.knnf_ctx_status(ctx) == _lib.KNNF_OK
    finally:
        _lib.knnf_destroy(ctx)


def test_streams_that_come_and_go():
    import torch

    hip = ctypes.CDLL(_loaded_hip())
    ctx = _lib.knnf_create(0)
    try:
        sets = [Set(ctx, 3 if s % 2 else 45, s, 2) for s in range(4)]
        for turn in range(12):
            s = ctypes.c_void_p()
            assert hip.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
            sets[turn % 4].clear()
            torch.cuda.synchronize()
            sets[turn % 4].run(ctx, s.value)
            assert hip.hipStreamDestroy(s) == 0
            other = sets[(turn + 1) % 4]
            other.run(ctx, current_stream())
            torch.cuda.synchronize()
            sets[turn % 4].check(f"turn {turn}")
            other.check(f"turn {turn}, other")
        assert _lib.knnf_ctx_status(ctx) == _lib.KNNF_OK
    finally:
        _lib.knnf_destroy(ctx)


def _loaded_hip():
    """Path of the HIP runtime that is mapped into this process (torch's)."""
    with open("/proc/self/maps") as f:
        return next(line.split()[-1] for line in f if "libamdhip64.so" in line)
