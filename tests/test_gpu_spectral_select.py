"""Cooperative selection of the lambda = 0 kernel, bit-exact against the oracle: K
around what the 64 kept candidates can answer (with and without the band row
outside a query's window), band ends with fewer than 64 candidates on a side, equal
distances inside the kept range (repaired) and across its end (left to the walk),
both in one wavefront, distances at +inf, class counts that take one or several
passes, one-row last workgroups and widths that leave wavefronts part empty.
"""
import numpy as np
import pytest

import oracle
from paper_2404_10631_amd import _lib
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = _lib.knnf_create(0)
    yield c
    _lib.knnf_destroy(c)


def frame(kind, H, W, C, seed):
    rng = np.random.default_rng(seed)
    pc1 = rng.random((H, W)).astype(np.float32)
    if kind == "levels":  # runs of equal distance, longer and shorter than 64
        pc1 = np.where(rng.random((H, W)) < 0.5, np.round(pc1 * 40) / 40, pc1).astype(np.float32)
    elif kind == "pairs":  # many ties of two
        pc1 = (rng.integers(0, H * W // 2, (H, W)) / np.float32(H * W)).astype(np.float32)
    elif kind == "huge":  # distances beyond the binary32 range beside ordinary ones
        pc1[rng.random((H, W)) < 0.02] = np.float32(3e19)
        pc1[rng.random((H, W)) < 0.02] = np.float32(-3e38)
    prob = rng.random((H, W, C)).astype(np.float32)
    return np.ascontiguousarray(pc1), prob


@pytest.mark.parametrize("kind", ["plain", "levels", "pairs", "huge"])
@pytest.mark.parametrize("H,W,K,R,C", [
    (9, 33, 1, 2, 4), (10, 40, 31, 1, 2), (21, 65, 40, 3, 4), (12, 100, 60, 2, 3), (13, 50, 62, 6, 5),
    (8, 70, 63, 4, 4), (8, 70, 64, 4, 4), (5, 31, 40, 9, 16), (7, 1, 4, 5, 7), (3, 1100, 24, 1, 8)])
def test_select(ctx, kind, H, W, K, R, C):
    import torch

    pc1, prob = frame(kind, H, W, C, H * W + K)
    print(f"{kind} {H}x{W} K={K} R={R} C={C}", flush=True)
    ro, rc, rn, rd = oracle.knn_filter(pc1, prob, K, R, 0.0)
    for with_nbr in (True, False):
        df = DeviceFrame(pc1, prob, K, R, 0.0, with_nbr=with_nbr)
        df.clear_outputs()
        _lib.knnf_filter(ctx, df.as_c(), dict(search=1), current_stream())
        torch.cuda.synchronize()
        go, gc, gn, gd = df.results()
        if with_nbr:
            assert np.array_equal(gn, rn)
            assert np.array_equal(gd.view(np.uint32), rd.view(np.uint32))
        assert np.array_equal(gc, rc)
        assert np.array_equal(go.view(np.uint32), ro.view(np.uint32))
