"""lambda = 0, neighbours of (nearly) equal distance deep in the list: the only pair of a
wavefront's eight queries whose order the packed keys leave open may be the one between
the last lane of a query and the lane before it (candidates 55 and 56 of 64).

One row of many values has such a pair in about one query of 5,000; windows with another
row in the band move it to lower ranks.  Bit-exact against the oracle.
"""
import numpy as np
import pytest

import oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import DeviceFrame, current_stream

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = _lib.knnf_create(0)
    yield c
    _lib.knnf_destroy(c)


def compare(ctx, pc1, prob, K, R):
    import torch

    print(f"{pc1.shape} K={K} R={R}", flush=True)
    df = DeviceFrame(pc1, prob, K, R, 0.0, with_nbr=True)
    df.clear_outputs()
    _lib.knnf_filter(ctx, df.as_c(), None, current_stream())
    torch.cuda.synchronize()
    for a, b in zip(df.results(), oracle.knn_filter(pc1, prob, K, R, 0.0)):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("seed", range(5))
def test_one_row(ctx, seed):
    pc1, prob = inputs.g_unif(1, 6000, 90 + seed)
    compare(ctx, pc1, prob, 60, 0)


@pytest.mark.parametrize("R,K", [(1, 23), (5, 50), (14, 50)])
def test_rows(ctx, R, K):
    pc1, prob = inputs.g_derma(260, 400, R)
    compare(ctx, pc1, prob, K, R)
