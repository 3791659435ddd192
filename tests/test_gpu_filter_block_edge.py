"""K around the limit of the smaller pass-A block (40 | 41) under every search and tile
shape, where tiles of one launch take different blocks, and persistent batches at K on
both sides of it and at 64.  Bit-exact against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu

TILES = [(1, 8), (1, 16), (2, 4), (2, 8), (4, 4)]


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = _lib.knnf_create(0)
    yield c
    _lib.knnf_destroy(c)


_ref = {}


def frame(K, n=0):
    if (K, n) not in _ref:
        pc1, prob = inputs.g_brain(23 + n, 70 - 3 * n, 60 + n)
        rng = np.random.default_rng(n)
        pc1[rng.random(pc1.shape) < 0.02] += np.float32(0.4)  # outliers: the larger block
        _ref[K, n] = pc1, prob, oracle.knn_filter(pc1, prob, K, 11, 0.01)
    return _ref[K, n]


def run(ctx, K, plan, nframes=0):
    import torch

    print(f"K={K} {plan} frames={nframes}", flush=True)
    refs = [frame(K, n) for n in range(max(nframes, 1))]
    dfs = [DeviceFrame(pc1, prob, K, 11, 0.01, with_nbr=True) for pc1, prob, _ in refs]
    for df in dfs:
        df.clear_outputs()
    if nframes:
        _lib.knnf_filter_batch(ctx, [df.as_c() for df in dfs], plan, current_stream())
    else:
        _lib.knnf_filter(ctx, dfs[0].as_c(), plan, current_stream())
    torch.cuda.synchronize()
    for df, (_, _, ref) in zip(dfs, refs):
        for a, b in zip(df.results(), ref):
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("search", [0, 1])
@pytest.mark.parametrize("K", [39, 40, 41, 42])
def test_block_limit(ctx, K, search, tile):
    run(ctx, K, dict(search=search, tile_rows=tile[0], tile_cols=tile[1], waves=1))


@pytest.mark.parametrize("search", [0, 1])
@pytest.mark.parametrize("K", [40, 41, 64])
def test_persistent_batch(ctx, K, search):
    run(ctx, K, dict(search=search, tile_rows=1, tile_cols=8, waves=1, launch=1), nframes=3)
