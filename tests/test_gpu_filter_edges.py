"""Filter kernels at the edges of their run-time choices, bit-exact against the
oracle: K around the pass-A block sizes (28 | 29) and the half-size final
selection (32 | 33) up to 64; buffers that overflow (outliers, large K) and are
cut down by a tighter bound; ties that leave no such bound; bounds beyond the
packed keys' range (distances near and at +inf); the four-class Eq. 2 path and
what falls outside it (other class counts, probabilities that are not 16-byte
aligned); frame edges with masked rows and columns.
"""
import numpy as np
import pytest

import oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu

PLANS = [dict(search=1, tile_rows=1, tile_cols=8, waves=1), dict(search=1, tile_rows=2, tile_cols=4, waves=2),
         dict(search=1, tile_rows=1, tile_cols=16, waves=1), dict(search=0, tile_rows=1, tile_cols=8, waves=1),
         dict(search=0, tile_rows=4, tile_cols=4, waves=1)]


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = _lib.knnf_create(0)
    yield c
    _lib.knnf_destroy(c)


def check(ctx, pc1, prob, K, R, lam, plan, label, with_nbr=True, shift=0):
    import torch

    df = DeviceFrame(pc1, prob, K, R, lam, with_nbr=with_nbr)
    if shift:
        flat = torch.zeros(shift + df.prob.numel(), dtype=torch.float32, device="cuda")
        flat[shift:] = df.prob.reshape(-1)
        df.prob = flat[shift:].view(df.prob.shape)
    df.clear_outputs()
    _lib.knnf_filter(ctx, df.as_c(), plan, current_stream())
    torch.cuda.synchronize()
    go, gc, gn, gd = df.results()
    ro, rc, rn, rd = oracle.knn_filter(pc1, prob, K, R, lam)
    if with_nbr:
        assert np.array_equal(gn, rn), f"{label}: neighbours"
        assert np.array_equal(gd.view(np.uint32), rd.view(np.uint32)), f"{label}: distances"
    assert np.array_equal(gc, rc), f"{label}: classes"
    assert np.array_equal(go.view(np.uint32), ro.view(np.uint32)), f"{label}: probabilities"


@pytest.mark.parametrize("plan", PLANS, ids=lambda p: f"s{p['search']}t{p['tile_rows']}x{p['tile_cols']}")
@pytest.mark.parametrize("K", [1, 2, 27, 28, 29, 31, 32, 33, 47, 48, 63, 64])
def test_k_edges(ctx, plan, K):
    pc1, prob = inputs.g_brain(21, 61, 40 + K)
    check(ctx, pc1, prob, K, 9, 0.01, plan, f"K={K}", with_nbr=K % 2 == 0)


@pytest.mark.parametrize("plan", PLANS[:4], ids=lambda p: f"s{p['search']}t{p['tile_rows']}x{p['tile_cols']}")
@pytest.mark.parametrize("K", [16, 40, 60])
def test_outliers_overflow(ctx, plan, K):
    # isolated outliers: their few like-valued neighbours lie far outside the
    # block, so the block's bound lets whole regions through the scan
    pc1, prob = inputs.g_brain(40, 96, 5)
    rng = np.random.default_rng(9)
    at = rng.random(pc1.shape) < 0.03
    pc1[at] += rng.normal(0.0, 0.3, pc1.shape).astype(np.float32)[at]
    check(ctx, pc1, prob, K, 14, 0.01, plan, f"outliers K={K}")


@pytest.mark.parametrize("plan", PLANS, ids=lambda p: f"s{p['search']}t{p['tile_rows']}x{p['tile_cols']}")
@pytest.mark.parametrize("kind", ["constant", "levels", "lambda0"])
def test_ties_without_a_bound(ctx, plan, kind):
    pc1, prob = inputs.g_unif(17, 75, 3)
    if kind == "constant":
        pc1[:] = 0.25
    else:
        pc1 = np.floor(pc1 * 3).astype(np.float32) / 4
    for K in (16, 40, 64):
        check(ctx, pc1, prob, K, 6, 0.0 if kind == "lambda0" else 0.01, plan, f"{kind} K={K}")


@pytest.mark.parametrize("plan", PLANS, ids=lambda p: f"s{p['search']}t{p['tile_rows']}x{p['tile_cols']}")
@pytest.mark.parametrize("scale", [1.8e19, 1.84467e19, 6e19])
def test_distances_near_and_beyond_the_largest_finite(ctx, plan, scale):
    # squares of differences around and past the largest binary32 value
    pc1, prob = inputs.g_unif(9, 40, 8)
    pc1 = (pc1 * 8).astype(np.int32).astype(np.float32) * np.float32(scale / 4)
    for K in (12, 40):
        check(ctx, pc1, prob, K, 3, 0.01, plan, f"scale {scale} K={K}")


@pytest.mark.parametrize("C", [1, 2, 3, 4, 5, 8, 16])
@pytest.mark.parametrize("shift", [0, 1])
def test_class_counts_and_alignment(ctx, C, shift):
    pc1, prob = inputs.g_brain(23, 70, 60 + C, C)
    for K, plan in ((16, PLANS[0]), (40, PLANS[0]), (40, PLANS[2]), (33, PLANS[1])):
        check(ctx, pc1, prob, K, 8, 0.01, plan, f"C={C} K={K}", shift=shift)


@pytest.mark.parametrize("H,W", [(1, 64), (2, 40), (3, 17), (7, 16), (8, 15), (9, 9), (40, 7), (64, 3), (5, 129)])
def test_small_windows(ctx, H, W):
    pc1, prob = inputs.g_unif(H, W, H * 100 + W)
    for R in (0, 2, 7):
        for K in {1, min(16, (min(R + 1, H)) * W), min(64, (min(R + 1, H)) * W)}:
            for plan in (PLANS[0], PLANS[2], PLANS[3]):
                check(ctx, pc1, prob, K, R, 0.01, plan, f"{H}x{W} R={R} K={K}")
