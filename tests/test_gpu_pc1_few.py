"""The PC1 projection around the change from a thread per pixel to segments (10 | 11
bands) and at band counts beyond 256, with more pixels than one pass of the blocks holds.
Bar: within one binary32 ulp of the binary64 oracle.
"""
import numpy as np
import pytest

from oracle import pc1_oracle
from paper_2404_10631_amd import _lib, inputs
from paper_2404_10631_amd.frames import current_stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nb,npix", [(nb, n) for nb in (8, 9, 10, 11, 12) for n in (1, 63, 515)]
                         + [(9, 300_001), (10, 262_145), (11, 300_001), (256, 30_001), (257, 263_001)])
@pytest.mark.parametrize("normalize", [True, False], ids=["normalised", "raw"])
def test_around_the_change(nb, npix, normalize):
    import torch

    cube, mean, vec = inputs.g_cube(1, npix, nb, nb + npix)
    if not np.all(np.isfinite(vec)):
        vec = np.ones_like(vec)
    d = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (cube, mean, vec)]
    out = torch.full((npix,), float("nan"), device="cuda")
    ctx = _lib.knnf_create(0)
    try:
        _lib.knnf_pc1(ctx, d[0].data_ptr(), npix, nb, d[1].data_ptr(), d[2].data_ptr(), out.data_ptr(),
                      normalize, current_stream())
        torch.cuda.synchronize()
    finally:
        _lib.knnf_destroy(ctx)
    got, ref = out.cpu().numpy(), pc1_oracle.pc1(cube, mean, vec, normalize)
    assert np.all(np.abs(got.astype(np.float64) - ref) <= np.spacing(np.abs(ref)).astype(np.float64))
