"""The SVM and fused kernels at the edges of their tiles: band counts around a
piece (4), a k-step (16), the short-row variant's limit (64) and a staging of
weights (128); pixel counts around a group (16), a tile (64) and a block (256);
every class count; cubes that are only 4-byte aligned.

Bars as elsewhere: maps within 1e-6 of the binary64 oracle and bitwise equal
between knnf_svm and knnf_svm_pc1, the band within one binary32 ulp.
"""
import numpy as np
import pytest

from oracle import pc1_oracle, svm_oracle
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


def call(ctx, cube, mean, vec, model, C, normalize, shift):
    import torch

    npix, nb = cube.shape
    flat = torch.zeros(shift + npix * nb, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(cube.reshape(-1)).cuda()
    cp = flat.data_ptr() + 4 * shift
    m = [torch.from_numpy(a).cuda() for a in model]
    mv = [torch.from_numpy(a).cuda() for a in (mean, vec)]
    maps, maps2 = (torch.full((npix, C), float("nan"), device="cuda") for _ in range(2))
    band = torch.full((npix,), float("nan"), device="cuda")
    mp = [t.data_ptr() for t in m]
    _lib.knnf_svm(ctx, cp, npix, nb, C, *mp, maps.data_ptr(), current_stream())
    _lib.knnf_svm_pc1(ctx, cp, npix, nb, C, *mp, *(t.data_ptr() for t in mv), maps2.data_ptr(),
                      band.data_ptr(), normalize, current_stream())
    torch.cuda.synchronize()
    return maps.cpu().numpy(), maps2.cpu().numpy(), band.cpu().numpy()


BANDS = [1, 2, 3, 4, 5, 15, 16, 17, 31, 63, 64, 65, 67, 127, 128, 129, 145, 257, 4096]
PIXELS = [1, 15, 16, 17, 63, 64, 65, 255, 257]
CASES = ([(nb, 130, 4, 0) for nb in BANDS] + [(100, n, 4, 0) for n in PIXELS]
         + [(33, n, 3, 1) for n in PIXELS] + [(nb, 81, C, nb % 4) for C in range(2, 9) for nb in (30, 131)])


@pytest.mark.parametrize("nb,npix,C,shift", CASES)
def test_tile_edges(ctx, nb, npix, C, shift):
    cube, mean, vec = inputs.g_cube(1, npix, nb, 700 + nb + npix, "derma")
    model = inputs.g_svm_model(C, nb, 800 + C)
    if not np.all(np.isfinite(vec)):
        vec = np.ones_like(vec)
    normalize = (nb + npix) % 2 == 0
    maps, maps2, band = call(ctx, cube, mean, vec, model, C, normalize, shift)
    ref = svm_oracle.svm_prob(cube, *model, C)
    assert float(np.max(np.abs(maps.astype(np.float64) - ref))) <= 1e-6
    assert np.array_equal(maps.view(np.uint32), maps2.view(np.uint32))
    rb = pc1_oracle.pc1(cube, mean, vec, normalize)
    assert np.all(np.abs(band.astype(np.float64) - rb) <= np.spacing(np.abs(rb)).astype(np.float64))


@pytest.mark.parametrize("nb", [6, 100, 131])
def test_infinite_value_stays_in_its_pixel(ctx, nb):
    # an infinity in a pixel's last band must not reach other pixels, and the
    # raw projection of its own pixel is that infinity (no 0 x infinity)
    cube, mean, vec = inputs.g_cube(1, 40, nb, 77, "brain")
    model = inputs.g_svm_model(4, nb, 5)
    vec = np.abs(vec) + 0.01
    clean = call(ctx, cube, mean, vec, model, 4, False, 0)
    dirty = cube.copy()
    dirty[20, nb - 1] = np.inf
    got = call(ctx, dirty, mean, vec, model, 4, False, 0)
    keep = np.arange(40) != 20
    for a, b in zip(clean, got):
        assert np.array_equal(a[keep].view(np.uint32), b[keep].view(np.uint32))
    assert got[2][20] == np.inf
