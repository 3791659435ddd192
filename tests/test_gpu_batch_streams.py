"""Batched launches after the stream of earlier ones is gone: a context's work tables
are reused only when the launch that used them has ended, whatever has become of the
stream it ran on (a closed server's, or a caller's own).
"""
import numpy as np
import pytest

from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream
from paper_2404_10631_amd.serve import HostFrame, Server, replay

pytestmark = pytest.mark.gpu


def batch(ctx, frames, stream):
    _lib.knnf_filter_batch(ctx, [df.as_c() for df in frames], dict(search=1, flags=1), stream)


def test_batches_after_servers():
    import torch

    ctx = _lib.knnf_create(0)
    try:
        data = [inputs.g_brain(40 + k, 61, k) for k in range(3)]
        frames = [DeviceFrame(p, q, 16, 7, 0.01) for p, q in data]
        host = [HostFrame(p, q, 16, 7, 0.01) for p, q in data]
        batch(ctx, frames, current_stream())
        torch.cuda.synchronize()
        want = [df.results() for df in frames]
        for turn in range(4):
            print(f"turn {turn}", flush=True)
            with Server(ctx, 16 << 20) as srv:
                replay(srv, host, [0.0] * len(host))
            # other allocations take the place of what the server's streams held
            side = [torch.cuda.Stream() for _ in range(4)]
            for df in frames:
                df.clear_outputs()
            for k in range(6):
                batch(ctx, frames, side[k % 2].cuda_stream if k % 3 else current_stream())
                torch.cuda.synchronize()
            for df, ref in zip(frames, want):
                for a, b in zip(df.results(), ref):
                    assert np.array_equal(a, b)
            assert _lib.knnf_ctx_status(ctx) == _lib.KNNF_OK
    finally:
        _lib.knnf_destroy(ctx)
