"""The imaging chain over grid sizes: power-of-two sides (the library's own row
and column transforms, every length and the two orders of unequal sides),
other even sides (the platform library's transform), crops, one to four
polarisations, and W-stacking on both, against numpy's FP64 transform.  The
grid is read only: it holds the same bits afterwards.  Bar: 1e-5 relative L2,
the bar of the other imaging tests (an FP32 transform of 2^24 points is near
5e-7)."""
import numpy as np
import pytest

from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _centred(g):
    ny, nx = g.shape[-2:]
    return np.fft.fftshift(np.fft.ifft2(np.fft.ifftshift(g.astype(np.complex128), axes=(-2, -1))),
                           axes=(-2, -1)) * (nx * ny)


def _random(rng, *shape):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)


@pytest.mark.parametrize("npol,nx,ny,y0,out_ny", [
    (4, 64, 64, 0, 64), (1, 64, 128, 5, 100), (2, 128, 64, 0, 64), (3, 256, 256, 64, 128),
    (1, 512, 256, 0, 256), (4, 256, 512, 128, 256), (1, 1024, 512, 1, 511),
    (2, 512, 1024, 0, 1024), (1, 2048, 1024, 0, 1024), (4, 1024, 2048, 512, 1024),
    (1, 4096, 64, 0, 64), (1, 64, 4096, 1024, 2048), (1, 8192, 128, 0, 128),
    (1, 128, 8192, 0, 8192), (1, 32, 64, 0, 64), (2, 2, 2, 0, 2), (3, 100, 64, 10, 50),
    (1, 64, 102, 0, 102), (4, 486, 746, 0, 746), (2, 1000, 600, 299, 301), (1, 2050, 90, 0, 90),
])
def test_image(npol, nx, ny, y0, out_ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(nx * 7 + ny))
    g = _random(rng, npol, ny, nx)
    cx = rng.uniform(0.5, 2.0, nx).astype(np.float32)
    cy = rng.uniform(0.5, 2.0, out_ny).astype(np.float32)
    ref = _centred(g)[:, y0:y0 + out_ny] * cx * cy[:, None]
    gd = torch.from_numpy(g).cuda()
    cxd, cyd = torch.from_numpy(cx).cuda(), torch.from_numpy(cy).cuda()
    im = api.Imager(npol, nx, ny)
    got = im.image(gd, cxd, cyd, y0=y0, out_ny=out_ny).cpu().numpy()
    assert np.array_equal(gd.cpu().numpy(), g)
    err = H.rel_l2(got, ref)
    print(f"[imaging] {npol} x {ny} x {nx}: rel-L2 {err:.2e}", flush=True)
    assert err < TOL
    if y0 == 0 and out_ny == ny:   # the image may take the scratch's place
        got = im.image(gd, cxd, cyd, out=im.work).cpu().numpy()
        assert H.rel_l2(got, ref) < TOL


@pytest.mark.parametrize("npol,layers,nx,ny", [
    (1, 1, 64, 64), (4, 3, 128, 64), (2, 5, 64, 256), (1, 4, 512, 512), (1, 2, 64, 1024),
    (2, 3, 128, 2048), (1, 2, 64, 4096), (1, 3, 100, 64), (3, 2, 90, 246), (1, 2, 64, 8192),
])
def test_wstack_image(npol, layers, nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(nx * 3 + ny + layers))
    g = _random(rng, npol, layers, ny, nx)
    cx = rng.uniform(0.5, 2.0, nx).astype(np.float32)
    cy = rng.uniform(0.5, 2.0, ny).astype(np.float32)
    fx, fy, dw = 0.3, 0.2, 40.0
    l = (np.arange(nx) - nx // 2) / nx * fx
    m = (np.arange(ny) - ny // 2) / ny * fy
    nm1 = np.sqrt(1.0 - m[:, None] ** 2 - l ** 2) - 1.0
    ref = sum(_centred(g[:, j]) * np.exp(2j * np.pi * (j - (layers - 1) / 2) * dw * nm1)
              for j in range(layers)) * cx * cy[:, None]
    gd = torch.from_numpy(g).cuda()
    im = api.WStackImager(npol, layers, nx, ny)
    got = im.image(gd, torch.from_numpy(cx).cuda(), torch.from_numpy(cy).cuda(), fx, fy,
                   dw).cpu().numpy()
    assert np.array_equal(gd.cpu().numpy(), g)
    err = H.rel_l2(got, ref)
    print(f"[imaging] W-stack {npol} x {layers} x {ny} x {nx}: rel-L2 {err:.2e}", flush=True)
    assert err < TOL
