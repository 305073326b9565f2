"""Unit lists on both sides of the record count from which the groups of supports
above 32 are listed by launches of their own: such groups first, last, between
others and alone, against the FP64 oracle at 1e-5 relative L2, the bar of the
other parity tests."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("supports,nrec", [
    ((5, 33, 12, 34), 1 << 20), ((5, 33, 12, 34), (1 << 20) + 1), ((36,), (1 << 20) + 1),
    ((34, 4, 18), 1_200_000),
])
def test_groups_of_large_supports(supports, nrec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    rng = np.random.Generator(np.random.PCG64(nrec + sum(supports)))
    nu, nv, beta, npol = 333, 290, 2, 1
    sizes = [(beta * s + 1) ** 2 for s in supports]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    taps = rng.standard_normal(sum(sizes)) + 1j * rng.standard_normal(sum(sizes))
    taps /= np.abs(taps).max()
    uvw = np.stack([rng.uniform(-nu / 2 - 2, nu / 2 + 2, nrec),
                    rng.uniform(-nv / 2 - 2, nv / 2 + 2, nrec),
                    rng.uniform(-len(supports) + 0.6, len(supports) - 0.6, nrec)], 1)
    vis = rng.standard_normal((nrec, npol)) + 1j * rng.standard_normal((nrec, npol))
    geom = oracle.Geometry(nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0, kind="wproj",
                           plane_support=np.array(supports, np.int32), plane_offset=offs,
                           inv_dw=1.0)
    taps_q = H.quantise_taps(taps, "f32")
    ref, sk = oracle.grid(geom, taps_q, uvw, vis)
    model = (rng.standard_normal((npol, nv, nu)) + 1j * rng.standard_normal((npol, nv, nu))
             ).astype(np.complex64)
    vref, _ = oracle.degrid(geom, taps_q, uvw, model)
    spec = api.GridSpec(nu, nv, npol, beta, 1.0, 1.0)
    bank = api.KernelBank("wproj", torch.from_numpy(taps.astype(np.complex64)).cuda(),
                          plane_support=list(supports), plane_offset=offs.tolist(), inv_dw=1.0)
    with api.Plan(spec, bank, torch.from_numpy(uvw).cuda()) as plan:
        assert plan.nskipped == sk
        G = plan.grid(torch.from_numpy(vis.astype(np.complex64)).cuda()).cpu().numpy()
        out = torch.full((nrec, npol), complex("nan"), dtype=torch.complex64, device="cuda")
        V = plan.degrid(torch.from_numpy(model).cuda(), out=out).cpu().numpy()
    err, err_d = H.rel_l2(G, ref), H.rel_l2(V, vref)
    print(f"[units] {supports}, {nrec} records: grid {err:.2e}, degrid {err_d:.2e}", flush=True)
    assert err < TOL and err_d < TOL
