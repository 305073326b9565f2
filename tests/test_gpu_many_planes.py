"""Plans of more planes than one launch's arguments hold (56) and of more bucket
blocks than a workgroup adds up for itself (1024: 128 planes on 3072^2): every
support class, records in every plane, both signs of w, against the FP64 oracle
at 1e-5 relative L2, the bar of the other parity tests."""
import numpy as np
import pytest

import oracle

from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("n,planes,first,last", [
    (300, 56, 4, 36), (300, 57, 4, 36), (280, 113, 3, 34), (300, 128, 8, 40), (3072, 128, 2, 40),
])
def test_many_planes(n, planes, first, last):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(n + planes))
    beta, npol, nrec = 2, 2, 40_000
    supports = np.round(np.linspace(first, last, planes)).astype(np.int32)
    sizes = (beta * supports.astype(np.int64) + 1) ** 2
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    taps = rng.standard_normal(sizes.sum()) + 1j * rng.standard_normal(sizes.sum())
    taps /= np.abs(taps).max()
    uvw = np.concatenate([rng.uniform(-n / 2 - 3, n / 2 + 3, (nrec, 2)),
                          rng.uniform(-planes + 0.6, planes - 0.6, (nrec, 1))], 1)
    vis = rng.standard_normal((nrec, npol)) + 1j * rng.standard_normal((nrec, npol))
    geom = oracle.Geometry(nu=n, nv=n, beta=beta, scale_u=1.0, scale_v=1.0, kind="wproj",
                           plane_support=supports, plane_offset=offs, inv_dw=1.0)
    taps_q = H.quantise_taps(taps, "f32")
    assert len(np.unique(oracle.index(geom, uvw)["plane"])) == planes
    ref, sk = oracle.grid(geom, taps_q, uvw, vis)
    spec = api.GridSpec(n, n, npol, beta, 1.0, 1.0)
    bank = api.KernelBank("wproj", torch.from_numpy(taps.astype(np.complex64)).cuda(),
                          plane_support=supports.tolist(), plane_offset=offs.tolist(), inv_dw=1.0)
    model = (rng.standard_normal((npol, n, n)) + 1j * rng.standard_normal((npol, n, n))
             ).astype(np.complex64)
    vref, _ = oracle.degrid(geom, taps_q, uvw, model)
    with api.Plan(spec, bank, torch.from_numpy(uvw).cuda()) as plan:
        assert plan.nskipped == sk
        G = plan.grid(torch.from_numpy(vis.astype(np.complex64)).cuda()).cpu().numpy()
        V = plan.degrid(torch.from_numpy(model).cuda()).cpu().numpy()
    err, err_d = H.rel_l2(G, ref), H.rel_l2(V, vref)
    print(f"[planes] {planes} planes on {n}^2: grid {err:.2e}, degrid {err_d:.2e}", flush=True)
    assert err < TOL and err_d < TOL
