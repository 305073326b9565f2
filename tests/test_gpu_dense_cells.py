"""Degridding by cell: chunks that hold at least two records for every cell of
their bounding box, so that up to four records of a cell are taken together.  The
records are confined to a few cells of each of several tiles, or spread over whole
tiles with chunks long enough, and the index rule shows on the host that at least
nine tenths of the records lie in such chunks (a full chunk has R records, and its
box cannot exceed that of all records of its tile and plane).  Runs of one to many
records of a cell, w of both signs, every remainder of the footprint's 16-cell
steps, against the FP64 oracle at 1e-5 relative L2, the bar of the other parity
tests."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

TOL = 1e-5
TILE = 16


def _case(kind, supports, beta, npol, nrec, box):
    """Records whose footprint's first cell lies in a box of box x box cells of
    every third tile, at a place of its own in each."""
    rng = np.random.Generator(np.random.PCG64(nrec + 5 * beta + sum(supports) + box))
    smax = max(supports)
    nu, nv = 16 * TILE, 13 * TILE + 3
    tiles = [(tu, tv) for tv in range((nv - smax) // TILE) for tu in range((nu - smax) // TILE)][::3]
    corner = np.array([[TILE * t + rng.integers(0, TILE - box + 1) for t in tile]
                       for tile in tiles])
    which = rng.integers(0, len(tiles), nrec)
    plane = rng.integers(0, len(supports), nrec)
    S = np.asarray(supports)[plane]
    # first cell k and phase o of the footprint: q = beta k + beta S / 2 - 1 - o
    k = corner[which] + rng.integers(0, box, (nrec, 2))
    o = rng.integers(0, beta, (nrec, 2))
    half = beta * S // 2
    q = beta * k - 1 - o + half[:, None]
    u, v = (q / beta - np.array([nu // 2, nv // 2])).T
    w = (plane + rng.uniform(-0.4, 0.4, nrec)) * rng.choice([-1.0, 1.0], nrec)
    uvw = np.stack([u, v, w], 1)
    if kind == "sep":
        taps = rng.uniform(-1.0, 1.0, beta * supports[0] + 1)
        geom = oracle.Geometry(nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0,
                               support=supports[0])
        return nu, nv, uvw, taps, geom, None
    sizes = [(beta * s + 1) ** 2 for s in supports]
    offs = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    taps = rng.standard_normal(sum(sizes)) + 1j * rng.standard_normal(sum(sizes))
    taps /= np.abs(taps).max()
    geom = oracle.Geometry(nu=nu, nv=nv, beta=beta, scale_u=1.0, scale_v=1.0, kind="wproj",
                           plane_support=np.array(supports, np.int32), plane_offset=offs,
                           inv_dw=1.0)
    return nu, nv, uvw, taps, geom, offs


def _dense_share(geom, uvw):
    """Share of the valid records in full chunks that are dense whatever the order."""
    R = H.plan_chunk_records(len(uvw))
    ix = oracle.index(geom, uvw)
    ok = ix["valid"] == 1
    ku, kv = ix["k_lo_u"][ok], ix["k_lo_v"][ok]
    bucket = (np.maximum(ix["plane"][ok], 0) * 4096 + ku // TILE) * 4096 + kv // TILE
    dense = 0
    for b in np.unique(bucket):
        m = bucket == b
        area = (np.ptp(ku[m]) + 1) * (np.ptp(kv[m]) + 1)
        if R >= 2 * area:
            dense += m.sum() // R * R
    return dense / max(1, ok.sum())


@pytest.mark.parametrize("kind,supports,beta,dtype,npol,nrec,box", [
    ("sep", (1,), 2, "f32", 4, 280_000, 5),
    ("sep", (7,), 2, "f32", 1, 280_000, 5),
    ("sep", (8,), 4, "f16", 2, 280_000, 2),
    ("sep", (9,), 2, "bf16", 3, 280_000, 5),
    ("sep", (16,), 2, "f32", 4, 280_000, 5),
    ("sep", (12,), 2, "f32", 4, 2_200_000, 16),
    ("wproj", (7, 8, 3), 2, "f32", 4, 280_000, 5),
    ("wproj", (9, 13, 15, 16), 2, "f32", 2, 280_000, 5),
    ("wproj", (10, 14), 2, "f16", 4, 280_000, 1),
    ("wproj", (11, 16), 2, "bf16", 1, 280_000, 3),
    ("wproj", (6, 7), 2, "f32", 4, 2_200_000, 16),
])
def test_records_of_a_cell_together(kind, supports, beta, dtype, npol, nrec, box):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_04141_amd import api
    nu, nv, uvw, taps, geom, offs = _case(kind, supports, beta, npol, nrec, box)
    share = _dense_share(geom, uvw)
    assert share >= 0.9
    taps_q = H.quantise_taps(taps, dtype)
    rng = np.random.Generator(np.random.PCG64(11))
    model = (rng.standard_normal((npol, nv, nu)) + 1j * rng.standard_normal((npol, nv, nu))
             ).astype(np.complex64)
    ref, sk = oracle.degrid(geom, taps_q, uvw, model)
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
    out = torch.full((nrec, npol), complex("nan"), dtype=torch.complex64, device="cuda")
    V = api.degrid(spec, bank, torch.from_numpy(uvw).cuda(), torch.from_numpy(model).cuda(),
                   out=out).cpu().numpy()
    err = H.rel_l2(V, ref)
    # the largest record error too: a wrong record of many hides in the norm
    worst = np.max(np.linalg.norm(V - ref, axis=1)) / np.sqrt(np.mean(np.sum(np.abs(ref) ** 2, 1)))
    print(f"[cells] {kind} {supports} beta {beta} {dtype} npol {npol}, {nrec} records, "
          f"{share:.2f} dense: rel-L2 {err:.2e}, worst record {worst:.2e}", flush=True)
    assert err < TOL and worst < TOL
