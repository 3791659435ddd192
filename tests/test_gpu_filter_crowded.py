"""Tiles whose candidate buffers fill up again and again: small lambda, uniform noise, K
close to 64, few levels, under both searches, every tile shape and both kinds of batch;
windows on both sides of the rule for the whole-window scan; ragged right and lower
edges, other class counts.  Bit-exact against the oracle.  The work counter of the
exhaustive search stays the number of window pairs and block slots.
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


def check(ctx, pc1, prob, K, R, lam, plan, batch=False, with_nbr=True):
    import torch

    df = DeviceFrame(pc1, prob, K, R, lam, with_nbr=with_nbr)
    df.clear_outputs()
    print(f"{pc1.shape} C {prob.shape[2]} K {K} R {R} lambda {lam} {plan} batch {batch}", flush=True)
    if batch:
        _lib.knnf_filter_batch(ctx, [df.as_c()], plan, current_stream())
    else:
        _lib.knnf_filter(ctx, df.as_c(), plan, current_stream())
    torch.cuda.synchronize()
    for a, b in zip(df.results(), reference(pc1, prob, K, R, lam)):
        if a is not None:
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


_ref = {}


def reference(pc1, prob, K, R, lam):
    key = (pc1.tobytes(), prob.tobytes(), K, R, lam)
    if key not in _ref:
        _ref[key] = oracle.knn_filter(pc1, prob, K, R, lam)
    return _ref[key]


def frame(kind, H, W, C=4):
    pc1, prob = inputs.g_unif(H, W, 17, C) if kind != "brain" else inputs.g_brain(H, W, 17, C)
    if kind == "levels":
        pc1 = np.floor(pc1 * 6).astype(np.float32) / 6
    return pc1, prob


@pytest.mark.parametrize("search", [1, 0], ids=["pruned", "exhaustive"])
@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}")
@pytest.mark.parametrize("kind,lam,K", [("unif", 0.01, 64), ("unif", 0.01, 50), ("brain", 1e-4, 40), ("brain", 1e-4, 64),
                                        ("brain", 1e-3, 16), ("levels", 1e-4, 63), ("unif", 0.0, 64)])
def test_searches_and_tiles(ctx, kind, lam, K, tile, search):
    # 23 x 187: windows of up to 4,301 candidates
    pc1, prob = frame(kind, 23, 187)
    check(ctx, pc1, prob, K, 30, lam, dict(search=search, tile_rows=tile[0], tile_cols=tile[1], waves=2))


@pytest.mark.parametrize("launch", [1, 2], ids=["persistent", "grid"])
@pytest.mark.parametrize("search", [1, 0], ids=["pruned", "exhaustive"])
@pytest.mark.parametrize("kind,lam,K", [("unif", 0.01, 64), ("brain", 1e-4, 48), ("levels", 0.0, 60)])
def test_batches(ctx, kind, lam, K, launch, search):
    pc1, prob = frame(kind, 23, 187)
    check(ctx, pc1, prob, K, 30, lam, dict(search=search, launch=launch), batch=True)


@pytest.mark.parametrize("H,W,R", [(9, 131, 3), (40, 61, 14), (64, 5, 40), (1, 300, 0), (19, 230, 18), (5, 66, 2)])
@pytest.mark.parametrize("C,K", [(3, 60), (4, 64), (7, 52)])
def test_shapes_and_classes(ctx, H, W, R, C, K):
    pc1, prob = frame("unif", H, W, C)
    for plan in (dict(search=1), dict(search=1, tile_rows=4, tile_cols=4), dict(search=0)):
        check(ctx, pc1, prob, K, R, 1e-3, plan, with_nbr=C == 4)


@pytest.mark.parametrize("scale", [1.8e19, 6e19])
def test_distances_near_and_beyond_the_largest_finite(ctx, scale):
    pc1, prob = inputs.g_unif(12, 370, 8)
    pc1 = (pc1 * 64).astype(np.int32).astype(np.float32) * np.float32(scale / 32)
    for search in (1, 0):
        check(ctx, pc1, prob, 61, 12, 0.01, dict(search=search))


@pytest.mark.parametrize("kind,lam,K", [("unif", 0.01, 64), ("brain", 1e-4, 64)])
def test_exhaustive_counts_every_pair_once(ctx, kind, lam, K):
    import torch

    H, W, R = 23, 187, 30
    pc1, prob = frame(kind, H, W)
    df = DeviceFrame(pc1, prob, K, R, lam, with_nbr=False)
    c = _lib.knnf_create(0)
    try:
        _lib.knnf_stats_enable(c, True)
        _lib.knnf_filter(c, df.as_c(), dict(search=0), current_stream())
        torch.cuda.synchronize()
        pairs, tiles = _lib.knnf_stats_read(c, True)
    finally:
        _lib.knnf_destroy(c)
    assert tiles == H * -(-W // 8)
    assert pairs == H * W * (H * W) + H * W * 128
