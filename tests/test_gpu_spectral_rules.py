"""lambda = 0 around the choice between the selection and the walk (K at its ends, for
windows that drop a large or a small share of the band, both ends of the class and
output rules), and wavefronts whose queries change from the one to the other: bands of
a few levels beside continuous ones.  Bit-exact against the oracle.
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


def check(ctx, pc1, prob, K, R, with_nbr):
    import torch

    df = DeviceFrame(pc1, prob, K, R, 0.0, with_nbr=with_nbr)
    df.clear_outputs()
    print(f"{pc1.shape} C {prob.shape[2]} K {K} R {R} nbr {with_nbr}", flush=True)
    _lib.knnf_filter(ctx, df.as_c(), dict(search=1), current_stream())
    torch.cuda.synchronize()
    for a, b in zip(df.results(), oracle.knn_filter(pc1, prob, K, R, 0.0)):
        if a is not None:
            assert np.array_equal(a.view(np.uint32), b.view(np.uint32))


@pytest.mark.parametrize("R", [0, 1, 2, 7, 40])
def test_neighbour_counts(ctx, R):
    pc1, prob = inputs.g_brain(19, 83, 60 + R)
    rows = 2 * R + 2
    ends = {9, 10, 12, 13, 17, 18, 19, -(-18 * (rows - 1) // rows), 55 - 64 // rows, 56 - 64 // rows, 62, 63}
    for K in sorted(k for k in ends if 1 <= k <= 64):
        check(ctx, pc1, prob, K, R, K % 2 == 0)


@pytest.mark.parametrize("C", [3, 4, 5, 9])
def test_classes(ctx, C):
    pc1, prob = inputs.g_brain(15, 70, 80 + C, C)
    for K in (9, 10, 13, 18, 40):
        check(ctx, pc1, prob, K, 6, False)


@pytest.mark.parametrize("levels", [1, 4, 40, 300])
@pytest.mark.parametrize("part", ["all", "left", "stripes"])
def test_levels_beside_continuous_values(ctx, levels, part):
    pc1, prob = inputs.g_brain(21, 131, 33)
    flat = np.floor(pc1 * levels).astype(np.float32) / np.float32(levels)
    if part == "all":
        pc1 = flat
    elif part == "left":
        pc1[:, :60] = flat[:, :60]
    else:
        pc1[:, ::3] = flat[:, ::3]
    check(ctx, pc1, prob, 24, 7, part == "left")
