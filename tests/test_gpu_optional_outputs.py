"""Neighbour indices and distances are optional one by one: each is written when it is
asked for, with or without the other, under every search.
"""
import numpy as np
import pytest

import oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("keep", ["none", "nbr", "dist"])
@pytest.mark.parametrize("lam,levels,K,search", [(0.0, 0, 16, 1), (0.0, 5, 16, 1), (0.0, 0, 60, 1), (0.01, 0, 40, 1),
                                                 (0.01, 5, 40, 0)])
def test_each_output_alone(lam, levels, K, search, keep):
    import torch

    pc1, prob = inputs.g_brain(21, 45, 4)
    if levels:  # equal distances
        pc1 = np.floor(pc1 * levels).astype(np.float32) / levels
    df = DeviceFrame(pc1, prob, K, 6, lam)
    df.clear_outputs()
    c = df.as_c()
    if keep != "nbr":
        c.out_nbr = None
    if keep != "dist":
        c.out_dist = None
    print(f"lambda {lam} K {K} search {search}: {keep}", flush=True)
    ctx = _lib.knnf_create(0)
    try:
        _lib.knnf_filter(ctx, c, dict(search=search), current_stream())
        torch.cuda.synchronize()
    finally:
        _lib.knnf_destroy(ctx)
    ro, rc, rn, rd = oracle.knn_filter(pc1, prob, K, 6, lam)
    go, gc, gn, gd = df.results()
    assert np.array_equal(gc, rc) and np.array_equal(go.view(np.uint32), ro.view(np.uint32))
    assert np.array_equal(gn, rn) if keep == "nbr" else np.all(gn == 0x7f7f7f7f)
    untouched = gd.view(np.uint32) == 0x7f7f7f7f
    assert np.array_equal(gd.view(np.uint32), rd.view(np.uint32)) if keep == "dist" else np.all(untouched)
