"""GPU parity where many records share a tile, a cell and a tap phase: the
paths the gridders and degridders take for dense chunks (a plane's tap table
copied to on-chip memory).  Small grids of a few tiles, records over the whole
grid and slightly beyond it, w of both signs; a third of the records repeat
the coordinates of others exactly.  Grid and degrid against the FP64 oracle at
1e-5 relative L2, the bar of the other parity tests; supports at the edges of
the support classes and of the 64 lanes a wave's slots fill."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5

CASES = [
    # kind, supports, beta, tap type, npol, records
    ("sep", (1,), 2, "f32", 4, 280_000),
    ("sep", (8,), 2, "f32", 1, 280_000),
    ("sep", (9,), 2, "bf16", 3, 280_000),
    ("sep", (16,), 2, "f32", 4, 280_000),
    ("sep", (7,), 4, "f16", 2, 1_100_000),
    ("wproj", (1, 8, 7), 2, "f32", 4, 280_000),
    ("wproj", (9, 16, 8, 15), 2, "f32", 2, 280_000),
    ("wproj", (12, 11), 2, "f16", 4, 280_000),
    ("wproj", (16, 17, 23), 2, "bf16", 1, 280_000),
    ("wproj", (10, 8), 4, "f32", 4, 1_100_000),
    ("wproj", (40,), 2, "f32", 4, 60_000),
]


def _case(kind, supports, beta, npol, nrec):
    rng = np.random.Generator(np.random.PCG64(nrec + 7 * beta + sum(supports) + npol))
    nu, nv = 70, 61
    u = rng.uniform(-nu / 2 - 1, nu / 2 + 1, nrec)
    v = rng.uniform(-nv / 2 - 1, nv / 2 + 1, nrec)
    w = rng.uniform(-len(supports) + 0.6, len(supports) - 0.6, nrec)
    # runs of equal coordinates, some longer than 64, and scattered repeats
    k = nrec // 6
    run = np.sort(rng.integers(0, k // 20, k))
    src = rng.integers(0, nrec, k)
    for x in (u, v, w):
        x[k:2 * k] = x[:k][run]
        x[2 * k:3 * k] = x[src]
    x = rng.integers(0, nrec, 500)
    u[x], v[x], w[x] = u[x[0]], v[x[0]], w[x[0]]
    uvw = np.stack([u, v, w], 1)
    vis = rng.standard_normal((nrec, npol)) + 1j * rng.standard_normal((nrec, npol))
    if kind == "sep":
        taps = rng.uniform(-1.0, 1.0, beta * supports[0] + 1)
        geom = oracle.Geometry(nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0,
                               support=supports[0])
        return nu, nv, uvw, vis, taps, geom, None
    sizes = [(beta * s + 1) ** 2 for s in supports]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    taps = rng.standard_normal(sum(sizes)) + 1j * rng.standard_normal(sum(sizes))
    taps /= np.abs(taps).max()
    geom = oracle.Geometry(nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0, kind="wproj",
                           plane_support=np.array(supports, np.int32), plane_offset=offs,
                           inv_dw=1.0)
    return nu, nv, uvw, vis, taps, geom, offs


@pytest.mark.parametrize("kind,supports,beta,dtype,npol,nrec", CASES)
def test_dense_tiles(kind, supports, beta, dtype, npol, nrec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    nu, nv, uvw, vis, taps, geom, offs = _case(kind, supports, beta, npol, nrec)
    print(f"[dense] {kind} {supports} beta {beta} {dtype} npol {npol} records {nrec}", flush=True)
    taps_q = H.quantise_taps(taps, dtype)
    G_ref, sk = oracle.grid(geom, taps_q, uvw, vis)
    tdt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    spec = api.GridSpec(nu, nv, npol, beta, 1.0, 1.0)
    if kind == "sep":
        bank = api.KernelBank("separable", torch.from_numpy(taps).to(tdt).cuda(),
                              support=supports[0])
    else:
        t = torch.from_numpy(taps.astype(np.complex64)) if dtype == "f32" else \
            torch.from_numpy(np.stack([taps.real, taps.imag], -1)).to(tdt)
        bank = api.KernelBank("wproj", t.cuda(), plane_support=list(supports),
                              plane_offset=offs.tolist(), inv_dw=1.0)
    uvw_d = torch.from_numpy(uvw).cuda()
    vis_d = torch.from_numpy(vis.astype(np.complex64)).cuda()
    rng = np.random.Generator(np.random.PCG64(11))
    Gin = (rng.standard_normal((npol, nv, nu)) + 1j * rng.standard_normal((npol, nv, nu))
           ).astype(np.complex64)
    V_ref, _ = oracle.degrid(geom, taps_q, uvw, Gin)
    with api.Plan(spec, bank, uvw_d) as plan:
        assert plan.nskipped == sk
        G = plan.grid(vis_d).cpu().numpy()
        V = plan.degrid(torch.from_numpy(Gin).cuda()).cpu().numpy()
    one = api.grid(spec, bank, uvw_d, vis_d).cpu().numpy()
    err, err1, err_d = H.rel_l2(G, G_ref), H.rel_l2(one, G_ref), H.rel_l2(V, V_ref)
    print(f"[dense] grid rel-L2 {err:.2e}, one-shot {err1:.2e}, degrid {err_d:.2e}", flush=True)
    assert err < TOL
    assert err1 < TOL
    assert err_d < TOL
