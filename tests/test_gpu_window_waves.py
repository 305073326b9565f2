"""The window gridder of supports 9 to 16 where its taps stay in global memory:
four waves to a workgroup where no chunk of the call can have its table in LDS
(few records, or a large oversampling factor), eight where some can and others
cannot.  Every slot count of the class, chunks of one record up to full ones, one
to four polarisations, a non-finite visibility among them, against the FP64
oracle at 1e-5 relative L2, the bar of the other parity tests."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5


def _case(kind, supports, beta, npol, nrec, clustered):
    rng = np.random.Generator(np.random.PCG64(nrec + 3 * beta + sum(supports)))
    nu, nv = 150, 131
    u = rng.uniform(-nu / 2 - 1, nu / 2 + 1, nrec)
    v = rng.uniform(-nv / 2 - 1, nv / 2 + 1, nrec)
    if clustered:     # a few dense cells beside sparse ones
        k = nrec // 2
        u[:k], v[:k] = rng.normal(3.0, 2.0, k), rng.normal(-5.0, 2.0, k)
    w = rng.uniform(-len(supports) + 0.6, len(supports) - 0.6, nrec)
    uvw = np.stack([u, v, w], 1)
    vis = rng.standard_normal((nrec, npol)) + 1j * rng.standard_normal((nrec, npol))
    if kind == "sep":
        taps = rng.uniform(-1.0, 1.0, beta * supports[0] + 1)
        return nu, nv, uvw, vis, taps, None, oracle.Geometry(
            nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0, support=supports[0])
    sizes = [(beta * s + 1) ** 2 for s in supports]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    taps = rng.standard_normal(sum(sizes)) + 1j * rng.standard_normal(sum(sizes))
    taps /= np.abs(taps).max()
    return nu, nv, uvw, vis, taps, offs, oracle.Geometry(
        nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0, kind="wproj",
        plane_support=np.array(supports, np.int32), plane_offset=offs, inv_dw=1.0)


@pytest.mark.parametrize("kind,supports,beta,dtype,npol,nrec,clustered", [
    ("sep", (9,), 2, "f32", 4, 300, False),
    ("sep", (16,), 30, "bf16", 1, 40_000, True),
    ("sep", (11,), 64, "f16", 3, 700_000, False),
    ("wproj", (9, 10, 11, 12, 13, 14, 15, 16), 4, "f32", 4, 20_000, True),
    ("wproj", (16, 9), 2, "f16", 2, 511_999, True),
    ("wproj", (13, 16), 2, "f32", 1, 530_000, True),
    ("wproj", (12, 9), 8, "f32", 2, 700_000, False),
])
def test_taps_in_global_memory(kind, supports, beta, dtype, npol, nrec, clustered):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    nu, nv, uvw, vis, taps, offs, geom = _case(kind, supports, beta, npol, nrec, clustered)
    taps_q = H.quantise_taps(taps, dtype)
    ref, sk = oracle.grid(geom, taps_q, uvw, vis)
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
    skipped = torch.zeros(1, dtype=torch.int64, device="cuda")
    G = api.grid(spec, bank, uvw_d, vis_d, nskipped=skipped).cpu().numpy()
    err = H.rel_l2(G, ref)
    print(f"[waves] {kind} {supports} beta {beta} {dtype}, {nrec} records: rel-L2 {err:.2e}",
          flush=True)
    assert int(skipped.item()) == sk and err < TOL
    # a non-finite visibility reaches its footprint and no other cell
    ix = oracle.index(geom, uvw)
    r = int(np.flatnonzero(ix["valid"])[7])
    vis_d[r, 0] = complex(float("inf"), 0.0)
    G = api.grid(spec, bank, uvw_d, vis_d).cpu().numpy()
    s = supports[0] if kind == "sep" else supports[int(ix["plane"][r])]
    ku, kv = int(ix["k_lo_u"][r]), int(ix["k_lo_v"][r])
    inside = np.zeros((npol, nv, nu), bool)
    inside[0, kv:kv + s, ku:ku + s] = True
    assert np.isfinite(G[~inside]).all() and not np.isfinite(G[inside]).all()
    keep = np.where(inside, 0.0, ref)
    assert H.rel_l2(np.where(inside, 0.0, G), keep) < TOL
