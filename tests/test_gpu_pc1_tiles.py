"""The PC1 projection at the edges of its lane layout: band counts around a
piece (4) and around each segment width (32, 64, 128, 256 bands), pixel counts
around a load and a block's step, cubes that are only 4-byte aligned, and more
steps than blocks.

Bar as elsewhere: within one binary32 ulp of the binary64 oracle, minimum 0 and
maximum 1 exactly when normalised.
"""
import numpy as np
import pytest

from oracle import pc1_oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import current_stream

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch

    assert torch.cuda.is_available()
    c = _lib.knnf_create(0)
    yield c
    _lib.knnf_destroy(c)


def call(ctx, cube, mean, vec, normalize, shift):
    import torch

    npix, nb = cube.shape
    flat = torch.zeros(shift + npix * nb, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(cube.reshape(-1)).cuda()
    mv = [torch.from_numpy(a).cuda() for a in (mean, vec)]
    out = torch.full((npix,), float("nan"), device="cuda")
    _lib.knnf_pc1(ctx, flat.data_ptr() + 4 * shift, npix, nb, *(t.data_ptr() for t in mv),
                  out.data_ptr(), normalize, current_stream())
    torch.cuda.synchronize()
    return out.cpu().numpy()


CASES = ([(nb, 515, nb % 4) for nb in (3, 4, 5, 6, 7, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257)]
         + [(nb, n, 0) for nb in (25, 128) for n in (1, 2, 7, 8, 9, 31, 32, 33, 127, 128, 129, 1025)]
         + [(5, 600_001, 1)])


@pytest.mark.parametrize("nb,npix,shift", CASES)
def test_layout_edges(ctx, nb, npix, shift):
    cube, mean, vec = inputs.g_cube(1, npix, nb, 900 + nb + npix, "derma")
    if not np.all(np.isfinite(vec)):
        vec = np.ones_like(vec)
    normalize = (nb + npix) % 3 != 0
    got = call(ctx, cube, mean, vec, normalize, shift)
    ref = pc1_oracle.pc1(cube, mean, vec, normalize)
    assert np.all(np.abs(got.astype(np.float64) - ref) <= np.spacing(np.abs(ref)).astype(np.float64))
    if normalize and npix > 1 and ref.max() > ref.min():
        assert got.min() == 0.0 and got.max() == 1.0


@pytest.mark.parametrize("nb", [6, 33, 100])
def test_infinite_value_stays_in_its_pixel(ctx, nb):
    cube, mean, vec = inputs.g_cube(1, 70, nb, 78, "brain")
    vec = np.abs(vec) + 0.01
    clean = call(ctx, cube, mean, vec, False, 0)
    dirty = cube.copy()
    dirty[20, nb - 1] = np.inf
    got = call(ctx, dirty, mean, vec, False, 0)
    keep = np.arange(70) != 20
    assert np.array_equal(clean[keep].view(np.uint32), got[keep].view(np.uint32))
    assert got[20] == np.inf
