"""The fused call's projection is centred band by band: its error is that of the centred
terms, however large the cube's offset is, and a pixel equal to the band averages
projects to zero.

Bound (raw projection): half a binary32 ulp for the rounding of the result, and for the
binary64 sum (bands + 2) * 2^-53 * sum |(x - mean) * vec|, against the sum in extended
precision.
"""
import numpy as np
import pytest

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


def fused(ctx, cube, mean, vec, C, normalize):
    import torch

    npix, nb = cube.shape
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda()
         for a in (cube, *(a.astype(np.float64) for a in (*inputs.g_svm_model(C, nb, 3), mean, vec)))]
    maps = torch.empty((npix, C), device="cuda")
    band = torch.full((npix,), float("nan"), device="cuda")
    _lib.knnf_svm_pc1(ctx, d[0].data_ptr(), npix, nb, C, *(t.data_ptr() for t in d[1:]),
                      maps.data_ptr(), band.data_ptr(), normalize, current_stream())
    torch.cuda.synchronize()
    return band.cpu().numpy()


def sensor_counts(npix, nb, seed, level=60000.0, noise=2.0):
    rng = np.random.default_rng(seed)
    mean = level * (1.0 + rng.normal(0.0, 0.01, nb))
    cube = (mean + rng.normal(0.0, noise, (npix, nb))).astype(np.float32)
    vec = rng.normal(0.0, 1.0, nb)
    return cube, mean, vec / np.linalg.norm(vec)


@pytest.mark.parametrize("C,nb", [(4, 128), (2, 4), (3, 33), (4, 100), (5, 64), (8, 67), (4, 130), (4, 257),
                                  (4, 4096)])
def test_large_offset(ctx, C, nb):
    print(f"C={C} bands={nb}", flush=True)
    cube, mean, vec = sensor_counts(700, nb, nb)
    term = (cube.astype(np.longdouble) - mean) * vec
    ref, mag = term.sum(axis=1), np.abs(term).sum(axis=1)
    got = fused(ctx, cube, mean, vec, C, False).astype(np.longdouble)
    tol = 0.5 * np.spacing(np.abs(ref.astype(np.float32))) + (nb + 2) * 2.0 ** -53 * mag
    assert np.all(np.abs(got - ref) <= tol), float(np.max(np.abs(got - ref) / tol))
    norm = fused(ctx, cube, mean, vec, C, True).astype(np.longdouble)
    span = ref.max() - ref.min()
    want = (ref - ref.min()) / span
    tol = 0.5 * np.spacing(np.abs(want.astype(np.float32))) + 4 * (nb + 4) * 2.0 ** -53 * (mag.max() / span + 1)
    assert np.all(np.abs(norm - want) <= tol), float(np.max(np.abs(norm - want) / tol))


@pytest.mark.parametrize("nb", [4, 7, 64, 100, 128, 131, 300])
def test_pixels_at_the_band_averages(ctx, nb):
    cube, mean, vec = sensor_counts(300, nb, 7 * nb, 0.35, 0.1)
    mean = mean.astype(np.float32).astype(np.float64)
    cube[::3] = mean.astype(np.float32)
    got = fused(ctx, cube, mean, vec, 4, False)
    assert np.all(got[::3] == 0.0)
    assert np.all(got[1::3] != 0.0)
