"""The two ways a W-stacking image takes the columns of power-of-two layers, on
both sides of the rule that picks one: few columns (the layers transformed side
by side and combined), columns that fill the chip, and one layer, for column
lengths of the short, middle and long kernels, against numpy's FP64 transform
with the bar of the other imaging tests."""
import numpy as np
import pytest

from tests import helpers as H
from tests.test_gpu_imaging_sizes import TOL, _centred, _random

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("npol,layers,nx,ny", [
    (1, 3, 256, 256), (4, 2, 512, 512), (1, 1, 512, 512), (4, 3, 2048, 256), (1, 2, 1024, 4096),
    (1, 2, 512, 4096), (4, 2, 8192, 64), (4, 2, 8192, 128), (1, 2, 2048, 2048),
])
def test_columns_of_layers(npol, layers, nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(nx + ny + layers))
    g = _random(rng, npol, layers, ny, nx)
    cx = rng.uniform(0.5, 2.0, nx).astype(np.float32)
    cy = rng.uniform(0.5, 2.0, ny).astype(np.float32)
    fx, fy, dw = 0.2, 0.3, 55.0
    l = (np.arange(nx) - nx // 2) / nx * fx
    m = (np.arange(ny) - ny // 2) / ny * fy
    nm1 = np.sqrt(1.0 - m[:, None] ** 2 - l ** 2) - 1.0
    ref = sum(_centred(g[:, j]) * np.exp(2j * np.pi * (j - (layers - 1) / 2) * dw * nm1)
              for j in range(layers)) * cx * cy[:, None]
    gd = torch.from_numpy(g).cuda()
    got = api.WStackImager(npol, layers, nx, ny).image(
        gd, torch.from_numpy(cx).cuda(), torch.from_numpy(cy).cuda(), fx, fy, dw).cpu().numpy()
    assert np.array_equal(gd.cpu().numpy(), g)
    err = H.rel_l2(got, ref)
    print(f"[imaging] W-stack {npol} x {layers} x {ny} x {nx}: rel-L2 {err:.2e}", flush=True)
    assert err < TOL
