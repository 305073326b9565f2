"""Grids of more than 2,097,152 tiles (23200^2 cells: 1450^2 tiles of 16): the
records of the first and of the last tile rows, gridded and degridded.  Both
corners are compared with the FP64 oracle on a 256^2 grid of their own: the
coordinates are multiples of 1/64, so the shift between the two grids is exact
and the index rule gives the same taps.  Every other cell stays zero, and every
output of the degridder, filled with NaN beforehand, is written.  Bar: 1e-5
relative L2, the bar of the other parity tests."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5
N, SMALL, BETA, NREC = 23200, 256, 4, 3000


@pytest.mark.parametrize("supports", [(7,), (6, 12, 20, 40)], ids=["separable", "wproj"])
def test_first_and_last_tiles(supports):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    assert (-(-N // 16)) ** 2 > 1 << 21
    rng = np.random.Generator(np.random.PCG64(sum(supports)))
    smax = max(supports)

    def cplx(*shape):
        return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)

    # cells of each corner's own grid: whole footprints, the last tile rows (and
    # columns) up to the edge among them
    lo, hi = smax, SMALL - smax // 2 - 1
    near = rng.integers(64 * lo, 64 * hi, (2, NREC, 2)) / 64.0
    near[:, : NREC // 2, 1] = rng.integers(64 * (hi - 24), 64 * hi, (2, NREC // 2)) / 64.0
    local = near - SMALL // 2                                  # corner's coordinates
    shift = np.array([SMALL // 2 - N // 2, N // 2 - SMALL // 2], np.float64)
    w = rng.uniform(-len(supports) + 0.6, len(supports) - 0.6, (2, NREC, 1))
    small_uvw = np.concatenate([local, w], 2)
    uvw = np.concatenate([local + shift[:, None, None], w], 2).reshape(-1, 3)
    vis = cplx(2 * NREC, 1)
    if len(supports) == 1:
        taps = rng.uniform(-1.0, 1.0, BETA * smax + 1)
        geom = oracle.Geometry(nu=SMALL, nv=SMALL, beta=BETA, scale_u=1.0, scale_v=1.0,
                               support=smax)
        bank = api.KernelBank("separable", torch.from_numpy(taps).float().cuda(), support=smax)
    else:
        sizes = [(BETA * s + 1) ** 2 for s in supports]
        offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
        taps = rng.standard_normal(sum(sizes)) + 1j * rng.standard_normal(sum(sizes))
        taps /= np.abs(taps).max()
        geom = oracle.Geometry(nu=SMALL, nv=SMALL, beta=BETA, scale_u=1.0, scale_v=1.0,
                               kind="wproj", plane_support=np.array(supports, np.int32),
                               plane_offset=offs, inv_dw=1.0)
        bank = api.KernelBank("wproj", torch.from_numpy(taps.astype(np.complex64)).cuda(),
                              plane_support=list(supports), plane_offset=offs.tolist(), inv_dw=1.0)
    taps = H.quantise_taps(taps, "f32")
    spec = api.GridSpec(N, N, 1, BETA, 1.0, 1.0)
    uvw_d = torch.from_numpy(uvw).cuda()
    corner = [slice(0, SMALL), slice(N - SMALL, N)]

    skipped = torch.zeros(1, dtype=torch.int64, device="cuda")
    G = api.grid(spec, bank, uvw_d, torch.from_numpy(vis).cuda(), nskipped=skipped)
    assert int(skipped.item()) == 0
    for i in range(2):
        ref, sk = oracle.grid(geom, taps, small_uvw[i], vis[i * NREC:(i + 1) * NREC])
        assert sk == 0
        err = H.rel_l2(G[:, corner[i], corner[i]].cpu().numpy(), ref)
        print(f"[large] {supports} corner {i}: grid rel-L2 {err:.2e}", flush=True)
        assert err < TOL
        G[:, corner[i], corner[i]] = 0
    assert int(torch.count_nonzero(G).item()) == 0

    out = torch.full((2 * NREC, 1), complex("nan"), dtype=torch.complex64, device="cuda")
    model = cplx(2, 1, SMALL, SMALL)
    for i in range(2):
        G[:, corner[i], corner[i]] = torch.from_numpy(model[i]).cuda()
    V = api.degrid(spec, bank, uvw_d, G, out=out).cpu().numpy()
    for i in range(2):
        ref, _ = oracle.degrid(geom, taps, small_uvw[i], model[i])
        err = H.rel_l2(V[i * NREC:(i + 1) * NREC], ref)
        print(f"[large] {supports} corner {i}: degrid rel-L2 {err:.2e}", flush=True)
        assert err < TOL
